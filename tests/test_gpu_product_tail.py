"""The FP32 product's last few columns on the vector units: every remainder, and the
passes of 64 columns, at the bound of the product's parity tests; the product of the
same columns in whole blocks gives the same bits for the columns before them."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("cols", [16, 17, 18, 19, 20, 21, 33, 50, 65, 68, 69, 131])
@pytest.mark.parametrize("n", [200, 4999])
def test_product_tail(n, cols):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] product tail", n, cols, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + cols)
    px, py = (0.02 * n ** 0.5 * torch.rand(2, n, device="cuda", generator=g)).unbind(0)
    V = torch.randn(cols, n, device="cuda", generator=g)
    k = G.Kernel(0.04, 0.3)
    Y = G.ops.kernel_mvm(k, px, py, V, prec="fp32")
    x, y = px.double(), py.double()
    K = 0.09 * torch.exp(-((x[:, None] - x) ** 2 + (y[:, None] - y) ** 2) / (2 * 0.04 ** 2))
    assert ((Y.double() - V.double() @ K).abs() <= 1e-5 * (V.double().abs() @ K)).all()
    whole = cols - cols % 16
    assert torch.equal(Y[:whole], G.ops.kernel_mvm(k, px, py, V[:whole].contiguous(), prec="fp32"))
    out = torch.randn(cols, n + 3, device="cuda", generator=g)[:, :n]
    want = Y + 0.5 * out
    G.ops.kernel_mvm(k, px, py, V, prec="fp32", out=out, beta=0.5)
    assert ((out - want).abs() <= 1e-6 * (want.abs() + Y.abs())).all()
