"""What the sorted Gaussian products leave out is exactly zero: two clusters of points
whose pairs all lie near the end of FP32's exponent, along the axes and the diagonals,
with long and round shapes in every direction, against the all-pairs product."""
import math

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tshape,sshape", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("angle", [0.0, 0.25, 0.5, 0.75, 0.1])
def test_far_terms_are_kept(tshape, sshape, angle):
    """Sums of at most 2,000 positive FP32 terms in another order: 2e-4 relative, where
    the sum is above the smallest normal number by the terms' own rounding."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import ctypes as C

    import paper_2105_09465_amd as G
    print("[case] gauss cull", tshape, sshape, angle, flush=True)
    n, base = 6000, 0.0016
    g = torch.Generator(device="cuda").manual_seed(int(100 * angle) + 2 * tshape + sshape)
    u = lambda *s: torch.rand(*s, device="cuda", generator=g)  # noqa: E731
    c, s = math.cos(math.pi * angle), math.sin(math.pi * angle)

    def side(shapes, sign):
        # exponents of 100 to 126 at the base covariance for most pairs
        along, across = sign * (0.264 - 0.03 * u(n)), 0.3 * (u(n) - 0.5)
        z = None
        if shapes:
            t, a, b = 2 * math.pi * u(n), 0.03 * u(n) ** 4, 0.002 * u(n)
            ct, st = torch.cos(t), torch.sin(t)
            z = torch.stack([a * ct * ct + b * st * st, (a - b) * ct * st, a * st * st + b * ct * ct]).contiguous()
        return (c * along - s * across).contiguous(), (s * along + c * across).contiguous(), z

    T, S = side(tshape, 1), side(sshape, -1)
    V = 0.5 + u(1, n)
    Y = G.ops.gauss_product(base, 1.0, T[0], T[1], S[0], S[1], V, tz=T[2], sz=S[2])
    want = torch.empty_like(Y)
    p, par = G.ops._ptr, G._lib.gpl_gauss(base, 1.0)
    G._lib.call("gpl_gauss_product", C.byref(par), n, p(T[0]), p(T[1]), p(T[2]), None, n, p(S[0]), p(S[1]), p(S[2]),
                None, 1, p(V), n, p(want), n, 0.0, G.ops._stream())
    assert (want > 0).float().mean() > 0.3
    live = want > 1e-33  # each of the terms left is a normal number with a thousandth of its own rounding
    assert live.any()
    assert ((Y - want).abs()[live] <= 2e-4 * want[live]).all()
    assert ((Y - want).abs()[~live] <= 2e-37 * n).all()
