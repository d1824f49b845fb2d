"""`autograd.KernelMVM` over points held in any shape and stride: the gradients have
the points' own shape and the values of the same points in one row."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("form", ["row", "grid", "transposed", "strided"])
def test_gradients_take_the_points_shape(form):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    from paper_2105_09465_amd.autograd import KernelMVM
    print("[case] autograd points", form, flush=True)
    m = 9
    g = torch.Generator(device="cuda").manual_seed(8)
    row = torch.rand(2, m * m, device="cuda", generator=g)
    V = torch.randn(3, m * m, device="cuda", generator=g)
    U = torch.randn(3, m * m, device="cuda", generator=g)
    hyper = torch.tensor([0.1, 0.5], dtype=torch.float64, device="cuda")

    def held(v):
        if form == "row":
            return v.clone()
        if form == "grid":
            return v.view(m, m).clone()
        if form == "transposed":
            return v.view(m, m).T.contiguous().T
        return torch.stack([v, v], 1)[:, 0]

    px, py = (held(v).detach().requires_grad_() for v in row)
    h = hyper.clone().requires_grad_()
    Vg = V.clone().requires_grad_()
    Y = KernelMVM.apply(px, py, Vg, h, "fp32")
    Y.backward(U)
    wx, wy, wV, wh = G.ops.kernel_mvm_vjp(G.Kernel(0.1, 0.5), row[0].clone(), row[1].clone(), V, U)
    for p, w in ((px, wx), (py, wy)):
        assert p.grad.shape == p.shape and torch.equal(p.grad.reshape(-1), w)
    assert torch.equal(Vg.grad, wV) and torch.equal(h.grad, wh)
    # each its own memory: what is done to one does not keep or touch the other's
    assert px.grad.untyped_storage().data_ptr() != py.grad.untyped_storage().data_ptr()
