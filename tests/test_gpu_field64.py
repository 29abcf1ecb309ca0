"""Float64 field sums and quadratic rows by wavenumber chunks of 8: a partial
chunk, uneven wavenumbers, phases past the reduction's range (2^20 rad), points
on nodes, several right-hand sides, at the ends of their tiles, against the
float64 oracle."""
import numpy as np
import pytest

from oracle import field as ofield
from oracle import quadratic as Q
from oracle.mesh import Surface
from workloads import Body, HARD, SOFT, seeded_complex

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")
from paper_1706_07919_amd import DeviceQuadSurface, DeviceSurface  # noqa: E402

EVEN = 0.4 * np.arange(1, 12)                       # a whole and a partial chunk
ONE = np.array([2.3])
UNEVEN = np.sort(np.random.default_rng(0).uniform(0.3, 6.0, 9))
WIDE = np.array([0.9, 4.0e5, 4.0e5 + 1.0])


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


# float64 rounding of phases up to k r = 2e6 rad is 2e-10 of a term: 1e-6 leaves room for the
# cancellation of the terms in the sums (as the assembly's own test of wide phases)
@pytest.mark.parametrize("k,tol", [(EVEN, 1e-11), (ONE, 1e-11), (UNEVEN, 1e-11), (WIDE, 1e-6)],
                         ids=["even", "one", "uneven", "wide"])
@pytest.mark.parametrize("n_rhs,m", [(1, 33), (3, 32)])
def test_field_c128_chunks(ctx, k, tol, n_rhs, m):
    bodies = [Body((0.0, 0.0, -1.6), 1.0, 1.0, 2, HARD), Body((0.0, 0.0, 1.6), 0.8, 1.3, 1, SOFT)]
    s, ds = Surface(bodies), DeviceSurface.from_bodies(bodies)
    rng = np.random.default_rng(m)
    xp = rng.uniform(-4.0, 4.0, (m, 3))
    xp[:2] = s.x[[5, 170]]
    phi, psi = seeded_complex(rng, (len(k), n_rhs, s.n)), seeded_complex(rng, (len(k), n_rhs, s.n))
    U = torch.zeros((n_rhs, m, len(k)), dtype=torch.complex128, device="cuda")
    i0, ins = (torch.zeros(m, dtype=t, device="cuda") for t in (torch.int32, torch.uint8))
    native.bem_field_eval(ctx, ds.struct, len(k), dev(k), n_rhs, dev(phi), dev(psi), m, dev(xp), i0, 0,
                          ins, native.BEM_C128, U)
    U = U.cpu().numpy()
    for q, kq in enumerate(k):
        for r in range(n_rhs):
            ref, oi0, oins = ofield.field(s, kq, phi[q, r], psi[q, r], xp)
            assert np.array_equal(i0.cpu().numpy(), oi0) and np.array_equal(ins.cpu().numpy(), oins)
            assert np.array_equal(U[r, :2, q], phi[q, r, [5, 170]])   # a node's own value
            assert np.max(np.abs(U[r, :, q] - ref)) < tol * np.max(np.abs(ref))


@pytest.mark.parametrize("k,tol", [(EVEN, 1e-12), (ONE, 1e-12), (UNEVEN, 1e-12), (WIDE, 1e-6)],
                         ids=["even", "one", "uneven", "wide"])
@pytest.mark.parametrize("n_rhs", [1, 3])
def test_quadratic_chunks(ctx, k, tol, n_rhs):
    body = Body((0.1, -0.2, 0.3), 0.9, 1.4, 0, SOFT)
    qs, ds = Q.QuadSurface(body, 2), DeviceQuadSurface.from_body(body, 2)
    n, m = qs.n, 35
    rng = np.random.default_rng(n_rhs)
    y = seeded_complex(rng, (len(k), n_rhs, n))
    A = torch.zeros((len(k), n, n), dtype=torch.complex128, device="cuda")
    b = torch.zeros((len(k), n_rhs, n), dtype=torch.complex128, device="cuda")
    native.bem_assemble_quadratic(ctx, ds.struct, len(k), dev(k), n_rhs, dev(y), native.BEM_C128, A, n,
                                  b, None)
    phi, psi = y, seeded_complex(rng, y.shape)
    xp = rng.uniform(-3.0, 3.0, (m, 3))
    U = torch.zeros((n_rhs, m, len(k)), dtype=torch.complex128, device="cuda")
    i0, ins = (torch.zeros(m, dtype=t, device="cuda") for t in (torch.int32, torch.uint8))
    native.bem_field_eval_quadratic(ctx, ds.struct, len(k), dev(k), n_rhs, dev(phi), dev(psi), m,
                                    dev(xp), i0, ins, U)
    A, b, U = A.cpu().numpy(), b.cpu().numpy(), U.cpu().numpy()
    for q, kq in enumerate(k):
        for r in range(n_rhs):
            Aref, bref = Q.system(qs, kq, y[q, r])
            scale = np.max(np.abs(Aref), axis=1, keepdims=True)
            assert np.max(np.abs(A[q] - Aref) / scale) < tol
            assert np.linalg.norm(b[q, r] - bref) < tol * np.linalg.norm(bref)
            ref, _, _ = Q.field(qs, kq, phi[q, r], psi[q, r], xp)
            assert np.max(np.abs(U[r, :, q] - ref)) < 10 * tol * np.max(np.abs(ref))
