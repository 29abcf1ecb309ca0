"""Triangular solves with an index of factors and a selection of vectors (several
blocks, and the sweep per vector): fewer sets of factors than wavenumbers, several
right-hand sides, and wavenumbers that leave the refinement one after the other.
And the float32 LU over matrices of two sizes in every launch, at small widths."""
import numpy as np
import pytest

from workloads import Body, HARD

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


def known(ctx, ds, k, n_rhs):
    y = torch.empty((len(k), n_rhs, ds.n), dtype=torch.complex128, device="cuda")
    one = torch.empty((len(k), 1, ds.n), dtype=torch.complex128, device="cuda")
    for r, d in enumerate(((0.0, 0.0, 1.0), (0.6, 0.0, 0.8), (0.0, 1.0, 0.0))[:n_rhs]):
        native.bem_incident(ctx, ds.struct, len(k), k, d, one)
        y[:, r] = one[:, 0]
    return y


def direct(ctx, ds, k, y, mode=native.BEM_FP64_DIRECT, nb=0):
    opts = native.bem_solve_opts_default()
    opts.mode, opts.nb = mode, nb
    x = torch.zeros_like(y)
    native.bem_solve_batched(ctx, [(ds.struct, len(k), k, y.shape[1], y)], opts, [x])
    return x


def close(x, ref, tol):
    return bool((torch.linalg.vector_norm(x - ref, dim=-1) <= tol * torch.linalg.vector_norm(ref, dim=-1)).all())


@pytest.mark.parametrize("n_k,n_rhs", [(9, 1), (9, 2), (9, 3), (130, 3), (330, 1)])
def test_refinement_with_fewer_factors(ctx, n_k, n_rhs):
    ds = DeviceSurface.from_bodies([Body((0.0, 0.0, 0.0), 1.0, 1.2, 3, HARD)])   # 642 nodes
    n, ld, kf = ds.n, ds.n + 6, torch.tensor([0.8, 1.0, 1.2], dtype=torch.float64).cuda()
    # distances from the factors' wavenumbers between 0 and 0.1: from one sweep to several
    k = torch.as_tensor(0.8 + 0.4 * np.linspace(0, 1, n_k) ** 1.5).cuda()
    near = (k[:, None] - kf[None]).abs().argmin(dim=1).to(torch.int32).contiguous()
    y = known(ctx, ds, k, n_rhs)
    LU = torch.zeros((3, n, ld), dtype=torch.complex64, device="cuda")
    b = torch.empty((3, 1, n), dtype=torch.complex128, device="cuda")
    native.bem_assemble(ctx, ds.struct, 3, kf, 1, known(ctx, ds, kf, 1), native.BEM_C64, LU, ld, b, None)
    piv = torch.zeros((3, n), dtype=torch.int32, device="cuda")
    info = torch.ones(3, dtype=torch.int32, device="cuda")
    native.bem_getrf_batched(ctx, native.BEM_C64, n, ld, n * ld, 3, LU, piv, info, 0, native.BEM_GEMM_3M)
    x = torch.zeros_like(y)
    res = native.bem_refine_batched(ctx, ds.struct, n_k, k, n_rhs, y, LU, ld, n * ld, piv, 3, near, 1e-11, 60, x)
    assert len({i.iters for i in res}) > 1 and all(i.converged for i in res)
    # a step below 1e-11 leaves less than that of the solution, times the contraction
    assert close(x, direct(ctx, ds, k, y), 1e-10)


@pytest.mark.parametrize("mode", [native.BEM_FP32_IR_4M, native.BEM_FP32_IR_3M, native.BEM_FP64_DIRECT])
@pytest.mark.parametrize("nb", [24, 40, 72, 136])
def test_two_sizes_in_every_launch(ctx, mode, nb):
    bodies = [Body((0.0, 0.0, 0.0), 1.0, 1.1, level, HARD) for level in (3, 2)]   # 642 and 162 nodes
    ds = [DeviceSurface.from_bodies([b]) for b in bodies]
    k = torch.as_tensor(np.linspace(0.5, 2.5, 5)).cuda()
    y = [known(ctx, d, k, 2) for d in ds]
    x = [torch.zeros_like(v) for v in y]
    opts = native.bem_solve_opts_default()
    opts.mode, opts.nb = mode, nb
    native.bem_solve_batched(ctx, [(d.struct, 5, k, 2, v) for d, v in zip(ds, y)], opts, x)
    for d, v, got in zip(ds, y, x):
        assert close(got, direct(ctx, d, k, v), 1e-10)
