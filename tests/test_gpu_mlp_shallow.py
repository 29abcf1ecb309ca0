"""Dense layers on both sides of the lines between the shallow and the deep product
(depth 128, 256 with four tiles per compute unit; tiles that fill the chip), against
float64 sums."""
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


@pytest.mark.parametrize("B,n_in,n_out", [
    (1, 1, 1), (1025, 1, 1025), (1000, 128, 1030), (1000, 129, 1030), (33, 130, 16321),
    (2050, 256, 2040), (2050, 257, 2040), (127, 2040, 530), (16321, 7, 65)])
def test_dense_layer(ctx, B, n_in, n_out):
    g = torch.Generator("cuda").manual_seed(B + n_in)
    x, W, b, dy = (torch.randn(s, device="cuda", generator=g) for s in
                   ((B, n_in), (n_in, n_out), (n_out,), (B, n_out)))
    z, y, dz, dx = (torch.full(s, 7.0, device="cuda") for s in ((B, n_out), (B, n_out), (B, n_out), (B, n_in)))
    dW, db = torch.full_like(W, 7.0), torch.full_like(b, 7.0)
    native.bem_mlp_dense_fwd(ctx, B, n_in, n_out, x, W, b, 1, z, y)
    native.bem_mlp_dense_bwd(ctx, B, n_in, n_out, x, W, z, 1, dy, dW, db, dx, dz)
    u = 2.0 ** -24
    X, V, Z = x.double(), W.double(), z.double()

    def near(got, want, depth, size):   # a sum of depth products and its rounding
        assert torch.all((got.double() - want).abs() <= (depth + 4) * u * size)
    near(z, X @ V + b.double(), n_in, X.abs() @ V.abs() + b.double().abs())
    s = torch.sigmoid(Z)
    near(y, Z * s, 8, Z.abs())
    D = dz.double()
    near(dz, dy.double() * s * (1 + Z * (1 - s)), 8, dy.double().abs() * (1 + Z.abs()))
    near(dW, X.T @ D, B, X.T.abs() @ D.abs())
    near(db, D.sum(0), B, D.abs().sum(0))
    near(dx, D @ V.T, n_out, D.abs() @ V.T.abs())
