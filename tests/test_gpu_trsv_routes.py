"""Triangular solves on both sides of every line between solving by blocks and
sweeping with a workgroup per vector: backward stable entry by entry either way."""
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


@pytest.mark.parametrize("prec,n,batch,n_rhs", [
    # float32 on 256 compute units: 256 vectors up to n = 128, 768 up to 320, 320, 256 from 1536 on
    (native.BEM_C64, 127, 2, 128), (native.BEM_C64, 128, 2, 129), (native.BEM_C64, 129, 3, 256),
    (native.BEM_C64, 320, 257, 3), (native.BEM_C64, 321, 319, 1), (native.BEM_C64, 321, 2, 160),
    (native.BEM_C64, 1535, 2, 159), (native.BEM_C64, 1537, 3, 85), (native.BEM_C64, 1536, 2, 128),
    # float64: below n = 960, and 256 vectors below 1200 or of one right-hand side
    (native.BEM_C128, 1, 1, 1), (native.BEM_C128, 959, 1, 2), (native.BEM_C128, 960, 2, 3),
    (native.BEM_C128, 961, 3, 85), (native.BEM_C128, 1199, 2, 128), (native.BEM_C128, 1201, 2, 128),
    (native.BEM_C128, 1281, 1, 1)])
def test_solves_on_both_routes(ctx, prec, n, batch, n_rhs):
    rng = np.random.default_rng(n)
    dt = torch.complex128 if prec == native.BEM_C128 else torch.complex64
    u = 2.0 ** (-53 if prec == native.BEM_C128 else -24)
    sets = min(batch, 3)   # different factors, repeated over the batch
    F = seeded_complex(rng, (sets, n, n)) / np.sqrt(n) + 2.0 * np.eye(n)[None]
    LU = torch.as_tensor(F).to(dt).cuda()[torch.arange(batch) % sets].contiguous()
    perm = np.stack([rng.permutation(n) for _ in range(sets)])
    piv = np.zeros((sets, n), np.int32)   # interchanges that make the permutation
    for s in range(sets):
        order = list(range(n))
        for i in range(n):
            p = order.index(perm[s, i], i)
            order[i], order[p], piv[s, i] = order[p], order[i], p
    pv = torch.as_tensor(piv).cuda()[torch.arange(batch) % sets].contiguous()
    B = torch.as_tensor(seeded_complex(rng, (batch, n_rhs, n))).to(dt).cuda()
    X = torch.full_like(B, 7.0)
    native.bem_getrs_batched(ctx, prec, n, n, n * n, batch, LU, pv, n_rhs, B, X, n_rhs * n)
    for b in range(batch):
        A = LU[b].to(torch.complex128)
        L, U = torch.tril(A, -1) + torch.eye(n, dtype=A.dtype, device="cuda"), torch.triu(A)
        x, rhs = X[b].to(torch.complex128).T, B[b].to(torch.complex128)[:, torch.as_tensor(perm[b % sets]).cuda()].T
        bound = 4 * (n + 4) * u * (L.abs() @ (U.abs() @ x.abs()))
        assert torch.all((L @ (U @ x) - rhs).abs() <= bound), b
