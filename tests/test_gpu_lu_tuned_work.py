"""A width measured for few matrices is used for few: the tuner tries the default
widths of every amount of work, and its choice at one leaves the default at another."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")


@pytest.fixture()
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


def factor(ctx, A, nb):
    LU, (batch, n, _) = A.clone(), A.shape
    piv = torch.zeros((batch, n), dtype=torch.int32, device="cuda")
    info = torch.ones(batch, dtype=torch.int32, device="cuda")
    native.bem_getrf_batched(ctx, native.BEM_C64, n, n, n * n, batch, LU, piv, info, nb, native.BEM_GEMM_4M)
    assert not info.any()
    return torch.view_as_real(LU)


def test_default_candidates(ctx):
    native.bem_autotune_lu(ctx, native.BEM_C64, 642, 2, native.BEM_GEMM_4M)
    assert {r[0] for r in native.bem_autotune_lu_results(ctx)} == {64, 128, 256, 384, 512, 768, 1024}


def test_width_by_amount_of_work(ctx):
    n = 600
    g = torch.Generator("cuda").manual_seed(1)
    few, some, many = (torch.randn((b, n, n), dtype=torch.complex64, device="cuda", generator=g) +
                       n ** 0.5 * torch.eye(n, device="cuda") for b in (2, 100, 250))   # 0.7, 34, 86 Mi entries
    for A, nb in ((few, 64), (some, 128), (many, 256)):
        assert torch.equal(factor(ctx, A, 0), factor(ctx, A, nb))
        assert not torch.equal(factor(ctx, A, 0), factor(ctx, A, 384))
    native.bem_autotune_lu(ctx, native.BEM_C64, n, 2, native.BEM_GEMM_4M, [384])
    assert native.bem_lu_tuned_plan(ctx, native.BEM_C64, n, native.BEM_GEMM_4M)[0] == 384
    for A, nb in ((few, 384), (some, 128), (many, 256)):
        assert torch.equal(factor(ctx, A, 0), factor(ctx, A, nb))
    native.bem_lu_set_plan(ctx, native.BEM_C64, n, native.BEM_GEMM_4M, 96, 64, 0)
    for A in (few, some, many):
        assert torch.equal(factor(ctx, A, 0), factor(ctx, A, 96))
