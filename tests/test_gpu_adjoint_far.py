"""The product's adjoint where a 64-point tile spans far against the lengthscale: one
finite far point, first or last along the curve, or two clusters that share a tile,
against the closed form in FP64."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ELL, AMP, N = 0.04, 0.3, 701


def _points(where, far):
    g = torch.Generator(device="cuda").manual_seed(5)
    p = 0.5 * (torch.rand(2, N, device="cuda", generator=g) - 0.5)
    if where == "first":  # lower left of all: the curve starts there
        p[:, 300] = -far
    elif where == "last":  # lower right: the curve ends there
        p[0, 300] = far
    else:  # clusters of 331 and 370 points: neither fills its tiles
        p[0, 331:] += far
    return p


@pytest.mark.parametrize("where", ["first", "last", "clusters"])
@pytest.mark.parametrize("far", [25.0, 1e2, 1e4, 1e6, 1e7, 1e12, 1e25])
@pytest.mark.parametrize("entry", ["backward", "vjp"])
def test_adjoint_wide_tile(where, far, entry):
    """FP32 terms with FP64 sums: 4e-6 of the sum of the terms' magnitudes, as on a
    compact cloud; a point on its own has no gradient."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] adjoint far", where, far, entry, flush=True)
    p = _points(where, far)
    px, py = p[0].contiguous(), p[1].contiguous()
    g = torch.Generator(device="cuda").manual_seed(6)
    A, B = (torch.randn(17, N, device="cuda", generator=g) for _ in range(2))
    k = G.Kernel(ELL, AMP)
    if entry == "vjp":
        gpx, gpy, _, hyp = G.ops.kernel_mvm_vjp(k, px, py, B, A)
    else:
        gpx, gpy, hyp = G.ops.kernel_mvm_backward(k, px, py, A, B, [1.0] * 17)
    x, y = p.double()
    dx, dy = x[:, None] - x[None], y[:, None] - y[None]
    d2 = dx * dx + dy * dy
    K = AMP ** 2 * torch.exp(-d2 / (2 * ELL ** 2))
    F, M = A.double().T @ B.double(), A.double().abs().T @ B.double().abs()
    KS, KM = K * (F + F.T), K * (M + M.T)
    for got, d in ((gpx, dx), (gpy, dy)):
        want = -(KS * d).sum(1) / ELL ** 2
        assert torch.all((got.double() - want).abs() <= 4e-6 * (KM * d.abs()).sum(1) / ELL ** 2)
    want = torch.stack([0.5 * (KS * d2).sum() / ELL ** 3, KS.sum() / AMP])
    scale = torch.stack([0.5 * (KM * d2).sum() / ELL ** 3, KM.sum() / AMP])
    assert torch.all((hyp - want).abs() <= 4e-6 * scale), (hyp - want) / scale
