"""Right-hand sides of the quadratic operator taken together: those of a call with
several are those of calls with one each, on an even and on an uneven grid of
wavenumbers and where a phase passes the range of the rotations."""
import numpy as np
import pytest

from workloads import Body, SOFT

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


@pytest.mark.parametrize("k", [np.linspace(1.0, 4.0, 9), np.array([0.7, 1.1, 3.9, 4.0, 5.5]), np.array([1.0, 1e6])])
@pytest.mark.parametrize("n_rhs", [2, 3, 4, 5, 7])
def test_right_hand_sides_together(ctx, k, n_rhs):
    ds = DeviceQuadSurface.from_body(Body((0.0, 0.0, 0.0), 1.0, 1.0, 0, SOFT), 1)
    n, n_k, kd = ds.n, len(k), torch.as_tensor(k).cuda()
    g = torch.Generator("cuda").manual_seed(n_rhs)
    y = torch.randn((n_k, n_rhs, n), dtype=torch.complex128, device="cuda", generator=g)

    def assemble(y):
        A = torch.zeros((n_k, n, n), dtype=torch.complex128, device="cuda")
        b = torch.full((n_k, y.shape[1], n), 7.0, dtype=torch.complex128, device="cuda")
        native.bem_assemble_quadratic(ctx, ds.struct, n_k, kd, y.shape[1], y, native.BEM_C128, A, n, b, None)
        return A, b

    A, b = assemble(y)
    for r in range(n_rhs):
        A1, b1 = assemble(y[:, r:r + 1].clone())
        # the same sums, only contracted into multiply-adds in another way
        assert (A - A1).norm() <= 1e-15 * A1.norm()
        assert (b[:, r] - b1[:, 0]).norm() <= 1e-14 * b1.norm()
