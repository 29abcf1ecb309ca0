"""Block rows subtract sums, not single products: with a unit lower triangle whose
products are a quarter of the unknowns' last place each, subtracting them one at a
time would lose every one of them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec,dtype,eps", [(native.BEM_C64, torch.complex64, 2.0 ** -24),
                                            (native.BEM_C128, torch.complex128, 2.0 ** -53)])
@pytest.mark.parametrize("m", [32, 64])
def test_block_row_keeps_small_products(ctx, prec, dtype, eps, m):
    n = m + 70
    # below 1 the last place is eps; right-hand sides of 1 - eps stay below 1
    A = np.eye(n)
    A[:m, :m] += np.tril(np.full((m, m), eps / 4), -1)
    A[:m, m:] = 1.0 - eps
    A[m:, m:] += n * np.eye(n - m)
    LU = torch.as_tensor(A).to(dtype).cuda()
    piv = torch.zeros((1, n), dtype=torch.int32, device="cuda")
    info = torch.ones(1, dtype=torch.int32, device="cuda")
    native.bem_getrf_batched(ctx, prec, n, n, n * n, 1, LU, piv, info, m, native.BEM_GEMM_4M)
    assert info.item() == 0 and piv.cpu().numpy()[0].tolist() == list(range(n))
    U = LU.cpu().numpy()[:m, m:].real.astype(np.float64)
    # row i: (1 - eps) - i eps / 4 up to eps^2, every entry of the row alike; a sum of
    # four products is one last place, so only the last, partial sum is rounded
    off = (U - (1.0 - eps) + eps / 4 * np.arange(m)[:, None]) / eps
    assert np.max(np.abs(off)) <= 0.76
