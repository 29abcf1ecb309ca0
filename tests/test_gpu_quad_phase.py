"""The quadratic operator of several wavenumbers of an even grid is that of each one
alone: phases advanced along the grid keep the wavenumbers' own roundings, which at
phases of over 1000 rad would show as 1e-13 of every entry."""
import numpy as np
import pytest

from workloads import Body, HARD, SOFT

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")
from paper_1706_07919_amd import DeviceQuadSurface  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_k,top", [(8, 11.37), (13, 9.81), (2, 7.77)])
@pytest.mark.parametrize("bc,n_rhs", [(HARD, 1), (SOFT, 3)])
def test_wavenumbers_together_and_alone(ctx, n_k, top, bc, n_rhs):
    ds = DeviceQuadSurface.from_body(Body((0.0, 0.0, 0.0), 64.0, 1.0, 0, bc), 2)
    n, k = ds.n, torch.as_tensor(top * np.arange(1, n_k + 1) / n_k).cuda()
    g = torch.Generator("cuda").manual_seed(n_k)
    y = torch.randn((n_k, n_rhs, n), dtype=torch.complex128, device="cuda", generator=g)

    def assemble(k, y):
        A = torch.zeros((len(k), n, n), dtype=torch.complex128, device="cuda")
        b = torch.zeros((len(k), n_rhs, n), dtype=torch.complex128, device="cuda")
        native.bem_assemble_quadratic(ctx, ds.struct, len(k), k, n_rhs, y, native.BEM_C128, A, n, b, None)
        return A.clone(), b.clone()

    A, b = assemble(k, y)
    for q in range(n_k):
        A1, b1 = assemble(k[q:q + 1].clone(), y[q:q + 1].clone())
        # up to 4 rotations of 3 roundings, and some 10 in each value
        for a, one in ((A[q], A1[0]), (b[q], b1[0])):
            assert (a - one).norm() <= 24 * 2.0 ** -53 * one.norm(), q
