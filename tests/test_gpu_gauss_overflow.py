"""Sorted Gaussian products over points so far apart that the squared gap of their boxes
overflows: a non-finite column value or weight still reaches every target, as in the
all-pairs product (0 times it is not a number), and finite ones give the same sums."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tshape,sshape", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("what", ["none", "value", "weight"])
def test_overflowing_gap(tshape, sshape, what):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] gauss overflow", tshape, sshape, what, flush=True)
    n = 20480
    g = torch.Generator(device="cuda").manual_seed(2)
    u = lambda *s: torch.rand(*s, device="cuda", generator=g)  # noqa: E731
    tx, ty, sx, sy, sw = u(n), u(n), u(n), u(n), 0.5 + u(n)
    sx[n // 2:] += 2e20  # half of the sources: several whole chunks
    V = 0.5 + u(1, n)
    z = [torch.stack([0.02 * u(n), torch.zeros(n, device="cuda"), 0.02 * u(n)]) if s else None
         for s in (tshape, sshape)]
    if what == "value":
        V[0, n - 9] = float("nan")
    if what == "weight":
        sw[n - 9] = float("inf")
    Y = G.ops.gauss_product(0.0016, 1.0, tx, ty, sx, sy, V, tz=z[0], sz=z[1], sw=sw)
    want, par, p = torch.empty_like(Y), G._lib.gpl_gauss(0.0016, 1.0), G.ops._ptr
    G._lib.call("gpl_gauss_product", C.byref(par), n, p(tx), p(ty), p(z[0]), None, n, p(sx), p(sy), p(z[1]), p(sw), 1,
                p(V), n, p(want), n, 0.0, G.ops._stream())
    assert torch.equal(torch.isnan(Y), torch.isnan(want))
    if what == "none":  # positive terms: two orders of 10,240 FP32 additions
        assert ((Y - want).abs() <= 2e-5 * want).all()
    else:
        assert torch.isnan(want).all()
