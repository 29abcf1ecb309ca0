"""Block rows and interchanges of the LU at block widths that leave every size of
triangular solve (up to 16, 32 and 64 rows, and what is left past them), in
matrices of two sizes with odd leading dimensions: backward error of the factors."""
import numpy as np
import pytest

from workloads import seeded_complex

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", [native.BEM_C64, native.BEM_C128])
@pytest.mark.parametrize("nb", [8, 24, 40, 72, 136, 320])
@pytest.mark.parametrize("n,pad", [(323, 0), (400, 1)])
def test_block_rows(ctx, prec, nb, n, pad):
    rng = np.random.default_rng(n + nb)
    batch, ld = 2, n + pad
    cdt = np.complex128 if prec == native.BEM_C128 else np.complex64
    M = seeded_complex(rng, (batch, n, n)).astype(cdt)
    A = torch.zeros((batch, n, ld), dtype=torch.as_tensor(M).dtype)
    A[:, :, :n] = torch.as_tensor(M)
    A = A.cuda()
    piv = torch.zeros((batch, n), dtype=torch.int32, device="cuda")
    info = torch.full((batch,), 7, dtype=torch.int32, device="cuda")
    native.bem_getrf_batched(ctx, prec, n, ld, n * ld, batch, A, piv, info, nb, native.BEM_GEMM_4M)
    A, p = A.cpu().numpy(), piv.cpu().numpy()
    assert info.cpu().tolist() == [0] * batch and np.all(A[:, :, n:] == 0)
    u = 2.0 ** (-53 if prec == native.BEM_C128 else -24)
    for b in range(batch):
        LU = A[b, :, :n].astype(np.complex128)
        L, U = np.tril(LU, -1) + np.eye(n), np.triu(LU)
        perm = np.arange(n)
        for i in range(n):
            perm[[i, p[b, i]]] = perm[[p[b, i], i]]
        # |L U - P A| <= gamma_n |L||U| entry by entry, gamma_n = n u up to a small
        # factor for complex products
        bound = 4 * (n + 4) * u * (np.abs(L) @ np.abs(U))
        assert np.all(np.abs(L @ U - M[b][perm].astype(np.complex128)) <= bound)
