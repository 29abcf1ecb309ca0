"""The f16 split form where it has less than it wants: batches of two sizes packed in
slices, and factorisations recorded in a caller's stream capture, which may hold no
pointer into the packing buffer."""
import numpy as np
import pytest

from workloads import Body, HARD, seeded_complex

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")
from paper_1706_07919_amd import DeviceSurface  # noqa: E402


@pytest.mark.parametrize("spare", [12 << 20, 45 << 20])
def test_two_sizes_in_slices(spare):
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    surfaces = [DeviceSurface.from_bodies([Body((0.0, 0.0, 3.0 * b), 1.0, 1.0, 3, HARD) for b in range(m)])
                for m in (4, 2)]   # 2568 and 1284 nodes
    k = torch.as_tensor(np.linspace(0.5, 3.0, 3)).cuda()
    warm = native.Context(0)
    problems, xs = [], []
    for ds in surfaces:
        y = torch.empty((3, 1, ds.n), dtype=torch.complex128, device="cuda")
        native.bem_incident(warm, ds.struct, 3, k, (0.0, 0.0, 1.0), y)
        problems.append((ds.struct, 3, k, 1, y))
        xs.append(torch.zeros_like(y))

    def solve(ctx, mode):
        opts = native.bem_solve_opts_default()
        # (a loose tolerance keeps the first sweep's solution, which shows the factors' bits)
        opts.mode, opts.nb, opts.tol_step = mode, 256, 1e-2
        native.bem_solve_batched(ctx, problems, opts, xs)
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in xs]

    def calls(ctx, limit):
        ctx.set_workspace_limit(limit)
        ctx.set_profiling(True)
        x = solve(ctx, native.BEM_FP32_IR_3M)
        packed = ctx.kernel_stats("gemm_f16x3")[3]
        ctx.set_profiling(False)
        return x, packed

    for mode in (native.BEM_FP32_IR_4M, native.BEM_FP32_IR_3M):   # (loads every kernel)
        solve(warm, mode)
    warm.close()
    ctx = native.Context(0)
    free = torch.cuda.mem_get_info()[0]
    solve(ctx, native.BEM_FP32_IR_4M)   # one round's workspace
    held = free - torch.cuda.mem_get_info()[0]
    limited, sliced = calls(ctx, held + spare)
    whole, launches = calls(ctx, 0)
    ctx.close()
    assert sliced > launches > 0
    assert all(np.array_equal(a, b) for a, b in zip(limited, whole))


def test_callers_capture_holds_no_packing():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    n, nb = 1290, 256
    rng = np.random.default_rng(3)
    M = torch.as_tensor(seeded_complex(rng, (2, n, n)) + n ** 0.5 * np.eye(n)).to(torch.complex64).cuda()
    A = torch.empty_like(M)
    piv = torch.zeros((2, n), dtype=torch.int32, device="cuda")
    info = torch.ones(2, dtype=torch.int32, device="cuda")
    stream = torch.cuda.Stream()
    ctx = native.Context(0, stream)

    def factor(limit=0):
        ctx.set_workspace_limit(limit)
        native.bem_getrf_batched(ctx, native.BEM_C64, n, n, n * n, 2, A, piv, info, nb, native.BEM_GEMM_3M)

    with torch.cuda.stream(stream):
        A.copy_(M)
        factor()
        split = A.clone()
        A.copy_(M)
        factor(4096)                     # no packing buffer: float32 products
        plain = A.clone()
    stream.synchronize()
    assert not torch.equal(torch.view_as_real(split), torch.view_as_real(plain))
    ctx.set_workspace_limit(0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        factor()
    big = torch.as_tensor(seeded_complex(rng, (6, 1300, 1300)) + 40 * np.eye(1300)).to(torch.complex64).cuda()
    bpiv = torch.zeros((6, 1300), dtype=torch.int32, device="cuda")
    binfo = torch.ones(6, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(stream):
            A.copy_(M)
            info.fill_(7)
            graph.replay()
            got = A.clone()
            # eager work in between, which grows the packing buffer the first time
            W = big.clone()
            native.bem_getrf_batched(ctx, native.BEM_C64, 1300, 1300, 1300 * 1300, 6, W, bpiv, binfo, nb,
                                     native.BEM_GEMM_3M)
        stream.synchronize()
        assert torch.equal(torch.view_as_real(got), torch.view_as_real(plain))
        assert not info.any() and not binfo.any()
    del graph
    ctx.close()
