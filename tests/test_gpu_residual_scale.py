"""The matrix-free residual of bodies far from unit size: with the coordinates times
2^p, the weights times 2^2p and the wavenumbers times 2^-p every term scales by a
power of two, so the residual is that of the unit-size body."""
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


@pytest.mark.parametrize("p", [-80, -64, 64, 80])
@pytest.mark.parametrize("k", [[0.7, 1.1, 3.9, 4.0], np.linspace(1, 9, 16)])
def test_residual_scales(ctx, p, k):
    n, rng = 130, np.random.default_rng(7)
    k = np.asarray(k, dtype=np.float64)
    x, nrm = rng.uniform(-1, 1, (n, 3)), rng.standard_normal((n, 3))
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    w, hard = rng.uniform(0.1, 1, n), rng.integers(0, 2, n).astype(bool)
    y, xs = (seeded_complex(rng, (len(k), 1, n)) for _ in range(2))
    dg = seeded_complex(rng, (len(k), n, 2))

    def residual(s):
        ds = DeviceSurface(x * s, nrm, w * s * s, np.where(hard, HARD, 1 - HARD))
        phi, psi = np.where(hard, xs, y), np.where(hard, y, xs) / s
        r = torch.zeros((len(k), 1, n), dtype=torch.complex128, device="cuda")
        arrays = (k / s, np.where(hard, psi, phi), np.where(hard, phi, psi), dg * np.array([1.0, s]))
        kd, yd, xd, dd = (torch.as_tensor(np.ascontiguousarray(a)).cuda() for a in arrays)
        native.bem_residual(ctx, ds.struct, len(k), kd, 1, yd, xd, dd, r)
        return r.cpu().numpy()

    one, scaled = residual(1.0), residual(2.0 ** p)
    # the same operations on scaled values; a rounding or two where an estimate's
    # table is read at another exponent
    assert np.linalg.norm(scaled - one) <= 1e-14 * np.linalg.norm(one)
