"""Dense layers of the surrogate at the edges of their GEMM's tiles and depth
parts: forward, dW, db and dx against float64, within the rounding of a float32
sum of that length, with aligned and unaligned operands."""
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


@pytest.mark.parametrize("B,n_in,n_out,shift", [
    (1, 1, 1, 0), (33, 7, 65, 0), (64, 64, 64, 0), (256, 10, 512, 0), (31, 515, 2050, 0),
    (256, 1025, 4100, 0), (65, 512, 1028, 1), (130, 96, 33, 0)])
def test_dense_layer_against_float64(ctx, B, n_in, n_out, shift):
    rng = np.random.default_rng(B + n_in + n_out)

    def put(*shape):   # `shift` floats past an aligned address
        a = rng.standard_normal(shape).astype(np.float32)
        t = torch.empty(a.size + shift, dtype=torch.float32, device="cuda")[shift:].reshape(shape)
        t.copy_(torch.as_tensor(a))
        return a.astype(np.float64), t

    x, xd = put(B, n_in)
    W, Wd = put(n_in, n_out)
    b, bd = put(n_out)
    dy, dyd = put(B, n_out)
    y, dW, db, dx = (torch.full(s, np.nan, dtype=torch.float32, device="cuda")
                     for s in ((B, n_out), (n_in, n_out), (n_out,), (B, n_in)))
    native.bem_mlp_dense_fwd(ctx, B, n_in, n_out, xd, Wd, bd, 0, None, y)
    native.bem_mlp_dense_bwd(ctx, B, n_in, n_out, xd, Wd, None, 0, dyd, dW, db, dx, None)
    for got, ref, mag, terms in ((y, x @ W + b, np.abs(x) @ np.abs(W) + np.abs(b), n_in + 1),
                                 (dW, x.T @ dy, np.abs(x).T @ np.abs(dy), B),
                                 (db, dy.sum(0), np.abs(dy).sum(0), B),
                                 (dx, dy @ W.T, np.abs(dy) @ np.abs(W).T, n_out)):
        # n roundings of a sum of n terms: at most n 2^-24 sum |terms|
        assert np.all(np.abs(got.cpu().numpy() - ref) <= (terms + 1) * 2.0 ** -24 * mag)
