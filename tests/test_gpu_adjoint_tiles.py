"""The product's adjoint at the column counts where its passes and MFMA steps
change and at ragged point counts, against the closed form in FP64."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    return G


@pytest.mark.parametrize("pairs", [1, 2, 3, 4, 5, 8, 9, 16, 17, 18, 19, 37])
@pytest.mark.parametrize("n", [1, 63, 700, 4097])
def test_adjoint_columns(G, pairs, n):
    """Point gradients: every term is FP32 (kernel value, contraction of 2 x pairs
    products) with FP64 sums, so an entry is within a few 2^-24 of the sum of its
    terms' magnitudes: 4e-6 of it. The hyperparameter sums likewise."""
    print("[case] adjoint", pairs, n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(31 + n)
    side = 0.02 * n ** 0.5
    p = side * (torch.rand(2, n, device="cuda", generator=g) - 0.5) + 1.3
    A = torch.randn(pairs, n, device="cuda", generator=g)
    B = torch.randn(pairs, n, device="cuda", generator=g)
    w = [0.5 - 0.3 * (c % 4) for c in range(pairs)]
    gx0 = torch.randn(2, n, device="cuda", generator=g)
    ell, amp = 0.04, 0.3
    gpx, gpy, hyp = G.ops.kernel_mvm_backward(G.Kernel(ell, amp), p[0].contiguous(), p[1].contiguous(), A, B, w,
                                              gx0[0].clone(), gx0[1].clone())
    x, y = p[0].double(), p[1].double()
    dx, dy = x[:, None] - x[None], y[:, None] - y[None]
    d2 = dx * dx + dy * dy
    K = amp ** 2 * torch.exp(-d2 / (2 * ell ** 2))
    wA, Bd = torch.tensor(w, device="cuda", dtype=torch.float64)[:, None] * A.double(), B.double()
    F = wA.T @ Bd
    S, M = F + F.T, wA.abs().T @ Bd.abs()
    M = M + M.T
    for got, d, g0 in ((gpx, dx, gx0[0]), (gpy, dy, gx0[1])):
        want = -(K * S * d).sum(1) / ell ** 2
        bound = 4e-6 * (K * M * d.abs()).sum(1) / ell ** 2
        assert torch.all((got.double() - g0.double() - want).abs() <= bound + 1e-6 * (want.abs() + g0.double().abs()))
    want = torch.stack([0.5 * (K * S * d2).sum() / ell ** 3, (K * S).sum() / amp])
    scale = torch.stack([0.5 * (K * M * d2).sum() / ell ** 3, (K * M).sum() / amp])
    assert torch.all((hyp - want).abs() <= 4e-6 * scale)
