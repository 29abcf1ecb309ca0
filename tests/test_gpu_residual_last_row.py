"""The last row of an odd number of nodes takes the arithmetic of every other row:
one more node that carries no data, which gives it a neighbour in its row pair,
changes no bit of it."""
import numpy as np
import pytest

from workloads import HARD, seeded_complex

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")
from paper_1706_07919_amd import DeviceSurface  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [3, 129, 515])
@pytest.mark.parametrize("k", [np.linspace(1, 9, 16), [0.7, 1.1, 3.9, 4.0]])
def test_last_row_of_odd_n(ctx, n, k):
    rng, k = np.random.default_rng(n), np.asarray(k, dtype=np.float64)
    x, nrm = rng.uniform(-1, 1, (n + 1, 3)), rng.standard_normal((n + 1, 3))
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    w, bc = rng.uniform(0.1, 1, n + 1), np.where(rng.integers(0, 2, n + 1), HARD, 1 - HARD)
    y, xs = (seeded_complex(rng, (len(k), 1, n + 1)) for _ in range(2))
    y[..., n] = xs[..., n] = 0.0
    dg = seeded_complex(rng, (len(k), n + 1, 2))

    def residual(m):
        r = torch.zeros((len(k), 1, m), dtype=torch.complex128, device="cuda")
        kd, yd, xd, dd = (torch.as_tensor(np.ascontiguousarray(a)).cuda()
                          for a in (k, y[..., :m], xs[..., :m], dg[:, :m]))
        native.bem_residual(ctx, DeviceSurface(x[:m], nrm[:m], w[:m], bc[:m]).struct, len(k), kd, 1, yd, xd, dd, r)
        return r.cpu().numpy()

    assert np.array_equal(residual(n), residual(n + 1)[..., :n])
