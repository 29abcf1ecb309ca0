"""An infinite pivot: its column's multipliers are 0 (one infinite part), the other
rows keep their values, and the rest of the factorisation is that of the matrix
without its row and column."""
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


@pytest.mark.parametrize("prec,dtype,eps", [(native.BEM_C64, torch.complex64, 2.0 ** -24),
                                            (native.BEM_C128, torch.complex128, 2.0 ** -53)])
@pytest.mark.parametrize("value", [complex(np.inf, 0.0), complex(0.0, -np.inf), complex(1.0, np.inf)])
@pytest.mark.parametrize("n", [30, 300, 1100])
def test_infinite_pivot(ctx, n, prec, dtype, eps, value):
    rng = np.random.default_rng(n)
    A = seeded_complex(rng, (n, n)) + 4 * n * np.eye(n)   # no interchange
    c = n // 3
    A[c, c] = value
    LU = torch.as_tensor(A).to(dtype).cuda()
    piv = torch.zeros((1, n), dtype=torch.int32, device="cuda")
    info = torch.ones(1, dtype=torch.int32, device="cuda")
    native.bem_getrf_batched(ctx, prec, n, n, n * n, 1, LU, piv, info, 0, native.BEM_GEMM_4M)
    assert info.item() == 0 and piv.cpu().numpy()[0].tolist() == list(range(n))
    F = LU.cpu().numpy().astype(np.complex128)
    assert np.isinf(F[c, c]) and np.all(F[c + 1:, c] == 0)
    keep = np.arange(n) != c
    assert np.all(np.isfinite(F[keep][:, keep])) and np.all(np.isfinite(F[c, keep]))
    L, U = np.tril(F[keep][:, keep], -1) + np.eye(n - 1), np.triu(F[keep][:, keep])
    assert np.all(np.abs(L @ U - A[keep][:, keep]) <= 8 * n * eps * (np.abs(L) @ np.abs(U)))
