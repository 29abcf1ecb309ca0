"""Float32 3M factorisations whose large updates run as f16 split products: the
factors stay within the float32 error of the products |L||U| entry by entry,
also for rows and columns scaled over 2^+-30 (the split's scales follow them), at
the edges of its tiles, depths and packing slices."""
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


@pytest.mark.parametrize("n,pad,nb,limit,scaled", [
    (1089, 0, 64, 0, False),               # one update just above the threshold, ragged tiles
    (1152, 0, 128, 0, True),               # exactly 1024 x 1024: whole tiles, one depth range
    (1200, 1, 100, 0, True),               # odd leading dimension, partial last 8-k block
    (1300, 0, 264, 0, True),               # three depth ranges, the last 8 deep
    (1290, 2, 256, 24 << 20, True),        # packed in slices of one matrix
    (1290, 0, 256, 4096, False),           # no packing buffer: float32 MFMA
])
def test_split_update_entrywise_error(ctx, n, pad, nb, limit, scaled):
    rng = np.random.default_rng(n + nb)
    batch, ld = 2, n + pad
    M = seeded_complex(rng, (batch, n, n)) + 0.5 * np.sqrt(n) * np.eye(n)[None]
    if scaled:
        M *= 2.0 ** rng.integers(-30, 31, (batch, n, 1)) * 2.0 ** rng.integers(-30, 31, (batch, 1, n))
    M = M.astype(np.complex64)
    A = torch.zeros((batch, n, ld), dtype=torch.complex64)
    A[:, :, :n] = torch.as_tensor(M)
    A = A.cuda()
    piv = torch.zeros((batch, n), dtype=torch.int32, device="cuda")
    info = torch.ones(batch, dtype=torch.int32, device="cuda")
    ctx.set_workspace_limit(limit)
    try:
        native.bem_getrf_batched(ctx, native.BEM_C64, n, ld, n * ld, batch, A, piv, info, nb,
                                 native.BEM_GEMM_3M)
    finally:
        ctx.set_workspace_limit(0)
    assert info.cpu().numpy().tolist() == [0] * batch
    LU, p = A.cpu().numpy()[:, :, :n].astype(np.complex128), piv.cpu().numpy()
    # entrywise backward error: n roundings of 2^-24 bound it by n 2^-24 |L||U|
    # (7e-5); as they are random it stays near sqrt(n) 2^-24 (2e-6), and the
    # largest of n^2 entries within a few times that
    for b in range(batch):
        L, U = np.tril(LU[b], -1) + np.eye(n), np.triu(LU[b])
        PA = M[b].astype(np.complex128)
        for i in range(n):
            PA[[i, p[b, i]]] = PA[[p[b, i], i]]
        assert np.max(np.abs(L @ U - PA) / (np.abs(L) @ np.abs(U))) < 4 * np.sqrt(n) * 2.0 ** -24
