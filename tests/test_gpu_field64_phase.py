"""Phases of the float64 field along an even grid of wavenumbers whose values are
rounded: two nodes and a point on a line at distances that are exact, so nothing but
the kernels' own roundings stands between the field and its 64-bit-mantissa value."""
import numpy as np
import pytest

from workloads import HARD

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


@pytest.mark.parametrize("n_rhs", [1, 3])
@pytest.mark.parametrize("n_k,top", [(8, 11.37), (29, 9.81), (4, 7.77)])
@pytest.mark.parametrize("far", [64.0, 4096.0])
def test_field_phases(ctx, n_rhs, n_k, top, far):
    L = np.longdouble
    k = top * np.arange(1, n_k + 1) / n_k
    x = np.array([[0.0, 0, 0], [far, 0, 0]])
    nrm = np.array([[-1.0, 0, 0], [1.0, 0, 0]])
    w, xp = np.array([1.0, far]), np.array([[-0.5, 0.0, 0.0]])
    rng = np.random.default_rng(5)
    phi, psi = (rng.uniform(0.5, 1.0, (n_k, n_rhs, 2)) * np.exp(1j * rng.uniform(0, 6, (n_k, n_rhs, 2)))
                for _ in range(2))
    ds = DeviceSurface(x, nrm, w, np.full(2, HARD))
    U = torch.zeros((n_rhs, 1, n_k), dtype=torch.complex128, device="cuda")
    i0, inside = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.uint8, device="cuda")
    kd, pd, qd, xd = (torch.as_tensor(a).cuda() for a in (k, phi, psi, xp))
    native.bem_field_eval(ctx, ds.struct, n_k, kd, n_rhs, pd, qd, 1, xd, i0, 0, inside, native.BEM_C128, U)
    assert i0.item() == 0 and inside.item() == 0
    U = U.cpu().numpy()[:, 0]
    s = -L(far)   # n_a . (x_j - x_a), n_a . n_j = -1
    for q in range(n_k):
        kq = L(k[q])
        g, f, gp, fp = np.cos(kq * s), np.sin(kq * s) / kq, kq * np.sin(kq * s), -np.cos(kq * s)
        for c in range(n_rhs):
            pa, qa, pj, qj = (np.clongdouble(v) for v in (*phi[q, c, :1], *psi[q, c, :1], phi[q, c, 1], psi[q, c, 1]))
            total, scale = np.clongdouble(0), L(0)
            for r, sign in ((L(far) + L(0.5), 1), (L(far), -1)):
                G = L(far) / r * (np.cos(kq * r) + 1j * np.sin(kq * r))
                H = G * (1j * kq * r - 1) / r
                total += sign * (pj * H - qj * G - pa * (g * H - gp * G) - qa * (f * H - fp * G))
                scale += abs(pj * H) + abs(qj * G) + abs(pa) * (abs(H) + kq * abs(G)) + abs(qa) * (abs(H) / kq + abs(G))
            want = pa + total / L(12.566370614359172953850573533118)
            # 7 rotations of 3 roundings and some 15 more in every product
            assert abs(U[c, q] - want) <= 40 * 2.0 ** -53 * (abs(pa) + scale / 12.5), (q, c)
