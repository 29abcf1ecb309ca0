"""Float64 fields at uneven wavenumbers: those of several together are those of each
alone, for every remainder of the groups that share a pair's geometry, and where one
wavenumber's phases pass the range of the short reduction."""
import numpy as np
import pytest

from workloads import Body, HARD

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")
from paper_1706_07919_amd import DeviceSurface  # noqa: E402

K = [0.7, 1.1, 3.9, 4.0, 5.5, 6.1, 7.0, 8.8, 9.1, 10.4]


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_rhs", [1, 3, 5])
@pytest.mark.parametrize("k", [K[:3], K[:4], K[:5], K[:8], K, [0.7, 1.1, 4e5]])
@pytest.mark.parametrize("m", [1, 70])
def test_together_and_alone(ctx, n_rhs, k, m):
    ds = DeviceSurface.from_bodies([Body((0.0, 0.0, 0.0), 1.0, 1.2, 1, HARD)])
    n, n_k, kd = ds.n, len(k), torch.tensor(k, dtype=torch.float64).cuda()
    g = torch.Generator("cuda").manual_seed(n_k)
    phi, psi = (torch.randn((n_k, n_rhs, n), dtype=torch.complex128, device="cuda", generator=g) for _ in range(2))
    xp = torch.rand((m, 3), dtype=torch.float64, device="cuda", generator=g) * 4 + 1.5

    def field(kd, phi, psi):
        U = torch.full((n_rhs, m, len(kd)), 7.0, dtype=torch.complex128, device="cuda")
        i0, ins = (torch.zeros(m, dtype=t, device="cuda") for t in (torch.int32, torch.uint8))
        native.bem_field_eval(ctx, ds.struct, len(kd), kd, n_rhs, phi, psi, m, xp, i0, 0, ins, native.BEM_C128, U)
        return U

    U = field(kd, phi, psi)
    for q in range(n_k):
        one = field(kd[q:q + 1].clone(), phi[q:q + 1].clone(), psi[q:q + 1].clone())[..., 0]
        # the same sums from phases that may differ by a rounding of k r
        tol = (16 + k[q] * 12) * 2.0 ** -53 * np.sqrt(n) * 4
        assert (U[..., q] - one).abs().max() <= tol * one.abs().max()
