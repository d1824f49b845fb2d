"""The tile plan at the sizes where its kernels change: the one-workgroup plan
and the first size past it, ragged tiles, the sort's second workgroup, and the
point counts past the split that one workgroup holds. The product over the plan
is compared with FP64 on sampled rows, and the plan's work with a direct count."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    return G


def _cloud(kind, n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    side = 0.02 * n ** 0.5  # about the density of a ray-traced image
    p = side * (torch.rand(2, n, device="cuda", generator=g) - 0.5)
    if kind == "clumped":  # half of the points in one cell of the curve
        p[:, ::2] = 0.25 * side + 1e-6 * p[:, ::2]
    if kind == "line":
        p[1] = 0.0
    return p[0].contiguous(), p[1].contiguous()


@pytest.mark.parametrize("kind", ["uniform", "clumped", "line"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1025, 4095, 4096, 4097, 5000, 70001])
@pytest.mark.parametrize("prec", ["f16x3", "fp32"])
def test_product_over_plan(G, kind, n, prec):
    """Per entry within 1e-5 of |K||V|, the bound of the product's parity tests."""
    print("[case] plan", kind, n, prec, flush=True)
    if kind == "clumped" and n > 5000:
        n = 9001  # every pair of the clump is evaluated
    _check(G, kind, n, prec, 3, min(n, 200))


def test_product_past_the_folded_split(G):
    """More row tiles than one workgroup splits (n > 262,144)."""
    print("[case] plan 263000", flush=True)
    _check(G, "uniform", 263000, "f16x3", 17, 100)


def _check(G, kind, n, prec, cols, rows):
    px, py = _cloud(kind, n, 21)
    ell, amp = 0.04, 0.3
    V = torch.randn(cols, n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(22))
    Y = G.ops.kernel_mvm(G.Kernel(ell, amp), px, py, V, prec=prec)
    at = torch.randperm(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(23))[:rows]
    x, y = px.double(), py.double()
    K = amp ** 2 * torch.exp(-((x[at, None] - x[None]) ** 2 + (y[at, None] - y[None]) ** 2) / (2 * ell ** 2))
    want, scale = V.double() @ K.T, V.double().abs() @ K.T
    assert torch.all((Y[:, at].double() - want).abs() <= 1e-5 * scale)


@pytest.mark.parametrize("n", [700, 4096, 4097])
def test_plan_work(G, n):
    """Evaluated subtiles cover every pair above the cutoff: at least as many
    kernel values as pairs with k > 2^-36, and no more than all pairs of tiles."""
    print("[case] plan work", n, flush=True)
    px, py = _cloud("uniform", n, 24)
    tiles, sub, lo = G.ops.kernel_mvm_live_tiles(G.Kernel(0.04, 0.3), px, py, prec="f16x3", with_lo=True)
    d2 = (px[:, None].double() - px[None].double()) ** 2 + (py[:, None].double() - py[None].double()) ** 2
    live = int((d2 * (1.4426950408889634 / (2 * 0.04 ** 2)) < 36).sum())
    nrt = (n + 63) // 64
    assert live <= 512 * sub and tiles <= nrt * 2 * nrt and sub <= 4 * tiles and lo <= sub
