"""LU panels at the ends of their widths, rows per thread and partial last panels
(every factorisation ends in all shorter panels of its precision): backward error,
pivot growth, ties and a column without a pivot."""
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
@pytest.mark.parametrize("n,pad", [(1, 0), (3, 1), (17, 0), (32, 0), (33, 1), (256, 0), (257, 1),
                                   (511, 0), (529, 0), (1055, 1), (2577, 0), (6160, 0)])
def test_panel_sizes(ctx, prec, n, pad):
    rng = np.random.default_rng(n)
    batch, ld = 3 if n < 2000 else 1, n + pad
    cdt = np.complex128 if prec == native.BEM_C128 else np.complex64
    M = seeded_complex(rng, (batch, n, n)).astype(cdt)
    tie = batch == 3 and n > 2
    if tie:
        M[1, :, 0] = 1j ** rng.integers(0, 4, n)   # equal |re|+|im|: the first row stays
        M[2, :, n // 2] = 0                        # no pivot there
    A = torch.zeros((batch, n, ld), dtype=torch.as_tensor(M).dtype)
    A[:, :, :n] = torch.as_tensor(M)
    A = A.cuda()
    piv = torch.zeros((batch, n), dtype=torch.int32, device="cuda")
    info = torch.full((batch,), 7, dtype=torch.int32, device="cuda")
    native.bem_getrf_batched(ctx, prec, n, ld, n * ld, batch, A, piv, info, 0, native.BEM_GEMM_4M)
    A, p, info = A.cpu().numpy(), piv.cpu().numpy(), info.cpu().tolist()
    assert np.all(A[:, :, n:] == 0)
    assert info == ([0, 0, n // 2 + 1] if tie else [0] * batch)
    if tie:
        assert p[1, 0] == 0
    u = 2.0 ** (-53 if prec == native.BEM_C128 else -24)
    for b in range(batch):
        LU = A[b, :, :n].astype(np.complex128)
        L, U = np.tril(LU, -1), np.triu(LU)
        L[np.arange(n), np.arange(n)] = 1
        # the pivot has the largest |re|+|im|, so |l| <= sqrt(2) up to rounding
        assert np.abs(L).max() <= np.sqrt(2) * (1 + 16 * u)
        perm = np.arange(n)
        for i in range(n):
            assert i <= p[b, i] < n
            perm[[i, p[b, i]]] = perm[[p[b, i], i]]
        x = seeded_complex(rng, (n, 3))
        # |L U - P A| <= gamma_n |L||U| entry by entry, gamma_n = n u up to a small
        # factor for complex products; the check's own float64 rounding is below it
        bound = 4 * (n + 4) * u * (np.abs(L) @ (np.abs(U) @ np.abs(x)))
        assert np.all(np.abs(L @ (U @ x) - M[b][perm].astype(np.complex128) @ x) <= bound)
