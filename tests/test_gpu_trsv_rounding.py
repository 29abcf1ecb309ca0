"""Triangular solves by blocks: with factors whose products over a block of 256
unknowns make a quarter of an unknown's last place, an unknown rounded once per block
would lose all of them.  Also over slices of matrices and of right-hand sides."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")
EPS = 2.0 ** -24   # the last place just below 1


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    c = native.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("n,batch,n_rhs", [(3000, 1, 1), (3000, 2, 3), (1400, 2, 12500), (1400, 30, 500)])
def test_solve_keeps_small_products(ctx, lower, n, batch, n_rhs):
    F = np.tril(np.full((n, n), EPS / 4 / 256), -1)
    LU = np.eye(n) + (F if lower else F.T)
    LU = torch.as_tensor(LU).to(torch.complex64).cuda().repeat(batch, 1, 1).contiguous()
    piv = torch.arange(n, dtype=torch.int32, device="cuda").repeat(batch, 1).contiguous()
    B = torch.full((batch, n_rhs, n), 1.0 - EPS, dtype=torch.complex64, device="cuda")
    X = torch.empty_like(B)
    native.bem_getrs_batched(ctx, native.BEM_C64, n, n, n * n, batch, LU, piv, n_rhs, B, X, n_rhs * n)
    steps = torch.arange(n, device="cuda", dtype=torch.float64)
    want = 1.0 - EPS - (steps if lower else steps.flip(0)) * (EPS / 1024)
    off = max(float(((X[b].real.double() - want) / EPS).abs().max()) for b in range(batch))
    # one rounding of the sum (1/2), and the products of a tile's 64 unknowns that are
    # subtracted one by one (64 / 1024)
    assert off <= 0.5 + 64 / 1024 + 0.01 and float(X.imag.abs().max()) == 0.0
