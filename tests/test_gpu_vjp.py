"""The product's backward pass over one plan: bit for bit the product, and the
gradients of the adjoint's own entry (same pairs and sums, split over the waves
by another cost in the precision form, so FP64 sums in another order); errors as
there."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["f16x3", "fp32"])
@pytest.mark.parametrize("n,cols", [(1, 1), (65, 17), (1600, 19), (4097, 2), (9000, 37)])
def test_vjp(n, cols, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] vjp", n, cols, prec, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    px, py = (0.02 * n ** 0.5 * torch.rand(2, n, device="cuda", generator=g)).unbind(0)
    V, U = (torch.randn(cols, n + 5, device="cuda", generator=g)[:, :n] for _ in range(2))  # strided columns
    k = G.Kernel(0.04, 0.3)
    gx, gy, gV, gh = G.ops.kernel_mvm_vjp(k, px, py, V, U, prec=prec)
    assert torch.equal(gV, G.ops.kernel_mvm(k, px, py, U, prec=prec))
    wx, wy, wh = G.ops.kernel_mvm_backward(k, px, py, U, V, [1.0] * cols)
    for a, b in ((gx, wx), (gy, wy), (gh, wh)):
        assert (a - b).abs().max() <= 1e-6 * b.abs().max()
    with pytest.raises(Exception):
        G.ops.kernel_mvm_vjp(G.Kernel(0.04, 0.0), px, py, V, U, prec=prec)
    with pytest.raises(ValueError):
        G.ops.kernel_mvm_vjp(k, px, py, V, U[:, :-1], prec=prec)


def test_products_over_stale_memory():
    """Results the caller has not given are not cleared: every entry is written."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    g = torch.Generator(device="cuda").manual_seed(3)
    n = 700
    px, py = torch.rand(2, n, device="cuda", generator=g).unbind(0)
    V = torch.randn(3, n, device="cuda", generator=g)
    grid, psf = G.Grid(n=13, ss=2, pix_scale=0.05), G.PSF(0.1)
    img = torch.randn(2, grid.N, device="cuda", generator=g)
    z = torch.zeros(0, device="cuda")

    def run():
        a = [G.ops.kernel_mvm(G.Kernel(0.04, 0.3), px, py, V, prec=p) for p in ("f16x3", "fp32")]
        a += [G.ops.gauss_product(0.01, 1.0, px, py, px, py, V), G.ops.psf_conv(grid, psf, img, False),
              G.ops.psf_conv(grid, psf, img[:, :grid.n_pix].contiguous(), True),
              G.ops.gauss_product(0.01, 1.0, px, py, z, z, torch.zeros(3, 0, device="cuda"))]
        return a
    first = [t.clone() for t in run()]
    assert (first[-1] == 0).all()
    del g
    for _ in range(3):
        dirt = [torch.full_like(t, float("nan")) for t in first]
        del dirt
        for a, b in zip(run(), first):
            assert torch.equal(a, b)
