"""Float32 3M factorisations whose large updates run as f16 split products: which
tiles keep the split.  Rows of L with entries below f16's range beside one that
carries the products lose nothing by it; only tiles with entries that could lose more than
the bound on their products take float32 ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
native = pytest.importorskip("paper_1706_07919_amd.native")

N, NB, TILE = 1536, 256, 128


def factor(M, limit, pad):
    ctx = native.Context(0)
    if limit:
        ctx.set_workspace_limit(limit)
    batch = len(M)
    A = torch.zeros((batch, N, N + pad), dtype=torch.complex64)
    A[:, :, :N] = torch.as_tensor(M)
    A = A.cuda()
    piv = torch.zeros((batch, N), dtype=torch.int32, device="cuda")
    info = torch.ones(batch, dtype=torch.int32, device="cuda")
    native.bem_getrf_batched(ctx, native.BEM_C64, N, N + pad, N * (N + pad), batch, A, piv, info,
                             NB, native.BEM_GEMM_3M)
    assert info.cpu().numpy().tolist() == [0] * batch
    assert np.array_equal(piv.cpu().numpy(), np.broadcast_to(np.arange(N), (batch, N)))
    out = A.cpu().numpy()[:, :, :N]
    ctx.close()
    return out


def matrix(rng, rows):
    """[[I], [L]] [I, U] plus a dominant diagonal in the trailing block: off that diagonal
    the factors there are the rounding of C - L U.  Every row of L has one large entry;
    in the given ones it meets zeros of U."""
    def c(*shape):
        return rng.uniform(-0.5, 0.5, shape) + 1j * rng.uniform(-0.5, 0.5, shape)
    m = N - NB
    L, U = c(m, NB) * 2.0 ** -20, 0.25 + 0.25j + 0.5 * c(NB, m)
    at = rng.integers(1, NB, m)
    at[list(rows)] = 0
    L[:, 0] = 0.0
    L[np.arange(m), at] = 0.5
    L[list(rows)] *= 2.0 ** -12
    L[list(rows), 0] = 0.5
    U[0] = 0.0
    A = np.zeros((N, N), np.complex128)
    A[:NB, :NB], A[NB:, :NB], A[:NB, NB:] = np.eye(NB), L, U
    A[NB:, NB:] = L @ U + np.diag(np.full(m, 4.0 * N))
    return A.astype(np.complex64)


@pytest.mark.parametrize("pad", [0, 1])   # rows 16-byte aligned, or not
def test_tiles_that_lose_nothing_keep_the_split(pad):
    rng = np.random.default_rng(0)
    M = np.stack([matrix(rng, ()), matrix(rng, (3, 5 * TILE + 100))])
    split, plain = factor(M, 0, pad), factor(M, 1 << 20, pad)   # (a limit without room to pack)
    # the first block row of the trailing part has seen one update only: by tiles
    same = (split == plain)[:, NB:2 * NB, 2 * NB:].reshape(2, 2, TILE, -1, TILE).mean(axis=(2, 4))
    assert np.all(same[0] < 0.5) and np.all(same[1, 1] < 0.5), same
    assert np.all(same[1, 0] == 1.0), same
    for b in range(2):
        L = np.tril(split[b].astype(np.complex128), -1) + np.eye(N)
        U = np.triu(split[b].astype(np.complex128))
        # n roundings of 2^-24, four real products each
        assert np.all(np.abs(L @ U - M[b]) <= 4 * N * 2.0 ** -24 * (np.abs(L) @ np.abs(U)))
