"""The matrix-free residual at the ends of its row pairs, column strides and
wavenumber chunks, for every way of its phases (even grid, scattered, past 2^20
rad), against the sums in NumPy float64."""
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


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [1, 2, 255, 258, 515])
@pytest.mark.parametrize("k", [[2.5], [0.5, 1.0, 1.5], np.linspace(0.3, 6.0, 5), np.linspace(1, 9, 16),
                               np.array([0.7, 1.1, 3.9, 4.0, 5.5, 6.1, 7.0, 8.8, 9.1]), [1.0, 1.5e6]])
def test_residual_rows_and_chunks(ctx, n, k):
    rng = np.random.default_rng(n + len(k))
    k = np.asarray(k, dtype=np.float64)
    x, nrm = rng.uniform(-1, 1, (n, 3)), rng.standard_normal((n, 3))
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    w, hard = rng.uniform(0.1, 1, n), rng.integers(0, 2, n).astype(bool)
    ds = DeviceSurface(x, nrm, w, np.where(hard, HARD, 1 - HARD))
    nr = 2
    y, xs = (seeded_complex(rng, (len(k), nr, n)) for _ in range(2))
    dg = seeded_complex(rng, (len(k), n, 2))
    r = torch.zeros((len(k), nr, n), dtype=torch.complex128, device="cuda")
    native.bem_residual(ctx, ds.struct, len(k), dev(k), nr, dev(y), dev(xs), dev(dg), r)
    r = r.cpu().numpy()
    d = x[None] - x[:, None]                       # x_j - x_i
    rr = np.linalg.norm(d, axis=2) + np.eye(n)
    qn = np.einsum("ijc,jc->ij", d, nrm) / rr ** 3
    off = (1 - np.eye(n)) * w[None]
    for q in range(len(k)):
        E = np.exp(1j * k[q] * rr)
        G, H = off * E / rr, off * qn * E * (1j * k[q] * rr - 1)
        for s in range(nr):
            phi, psi = np.where(hard, xs[q, s], y[q, s]), np.where(hard, y[q, s], xs[q, s])
            ref = -(G @ psi - H @ phi + dg[q, :, 0] * phi + dg[q, :, 1] * psi)
            # rounding of the sums, and of phases k r formed from r with 3 roundings
            # here and at most 4 there
            tol = 1e-12 + 8 * 2.0 ** -53 * k[q] * rr.max()
            assert np.linalg.norm(r[q, s] - ref) <= tol * np.linalg.norm(ref)
