"""The sorted Gaussian products (large products through ops.gauss_product, which
gives them a workspace) against plain FP64 torch: shapes on neither side, one
side or both, column counts around the passes of 1, 2, 4 and 8, ragged sizes,
shapes that reach across the whole field, and non-finite inputs."""
import math

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BASE, NORM = 0.5 * 0.04 ** 2, 1.0 / (2 * math.pi)


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    return G


def _side(n, seed, shapes, spread=1.5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = lambda *s: torch.rand(*s, device="cuda", generator=g)  # noqa: E731
    x, y = spread * (2 * u(n) - 1), spread * (2 * u(n) - 1)
    z = None
    if shapes:
        a, b = 0.02 * (2 * u(2, n) - 1), 0.02 * (2 * u(2, n) - 1)
        z = torch.stack([a[0] ** 2 + b[0] ** 2, a[0] * a[1] + b[0] * b[1], a[1] ** 2 + b[1] ** 2])
        z[:, n // 3] = torch.tensor([0.09, 0.02, 0.05], device="cuda")  # reaches across the field
    return x, y, z, 0.5 + u(n)


def _dense(T, S, V):
    """(product, its scale |M||V|) in FP64, and the mask of targets whose terms are all representable."""
    (tx, ty, tz, tw), (sx, sy, sz, sw) = ([None if v is None else v.double() for v in s] for s in (T, S))
    dx, dy = tx[:, None] - sx[None], ty[:, None] - sy[None]
    cxx = torch.full_like(dx, float(torch.tensor(BASE, dtype=torch.float32)))
    cyy, cxy = cxx.clone(), torch.zeros_like(dx)
    for z, at in ((tz, lambda v: v[:, None]), (sz, lambda v: v[None])):
        if z is not None:
            cxx, cxy, cyy = cxx + at(z[0]), cxy + at(z[1]), cyy + at(z[2])
    det = cxx * cyy - cxy ** 2
    M = NORM * tw[:, None] * sw[None] * torch.exp(-0.5 * (cyy * dx * dx - 2 * cxy * dx * dy + cxx * dy * dy) / det)
    M = M / det.sqrt()
    V = V.double()
    return V @ M.T, V.abs() @ M.abs().T


@pytest.mark.parametrize("tshape,sshape", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("nt,ns,cols", [(6000, 6001, 1), (40000, 1600, 2), (1601, 33000, 3), (6143, 6145, 5),
                                        (5800, 5800, 9)])
def test_sorted_product_vs_dense(G, tshape, sshape, nt, ns, cols):
    """Within 1e-5 of |M||V| per entry, the bound of the dense products (FP32
    terms and sums), plus 1e-12 of the largest scale for targets all of whose
    terms underflow FP32."""
    print("[case] sorted gauss product", tshape, sshape, nt, ns, cols, flush=True)
    assert G._lib.lib.gpl_gauss_product_workspace(nt, ns, cols) > 0
    T, S = _side(nt, 1, tshape), _side(ns, 2, sshape)
    if nt == ns:
        S = (T[0], T[1]) + S[2:]  # one set of points
    V = torch.randn(cols, ns, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    Y0 = torch.randn(cols, nt, device="cuda", generator=torch.Generator(device="cuda").manual_seed(4))
    Y = G.ops.gauss_product(BASE, NORM, T[0], T[1], S[0], S[1], V, tz=T[2], tw=T[3], sz=S[2], sw=S[3])
    Yb = G.ops.gauss_product(BASE, NORM, T[0], T[1], S[0], S[1], V, tz=T[2], tw=T[3], sz=S[2], sw=S[3],
                             out=Y0.clone(), beta=-0.5)
    want, scale = _dense(T, S, V)
    bound = 1e-5 * scale + 1e-12 * scale.max()
    assert torch.all((Y.double() - want).abs() <= bound)
    assert torch.all((Yb.double() - (want - 0.5 * Y0.double())).abs() <= bound + 1e-6 * Y0.double().abs())


def test_sorted_product_keeps_non_finite_inputs(G):
    """A non-finite column value, weight, shape or position reaches the same
    targets as in the all-pairs product (entry without a workspace)."""
    print("[case] sorted gauss product, non-finite", flush=True)
    nt, ns = 6001, 6002
    C, lib = __import__("ctypes"), G._lib
    for what in ("V", "sw", "sz", "sx", "tx", "tz"):
        T, S = list(_side(nt, 5, True)), list(_side(ns, 6, False))
        if what == "sz":
            T, S = list(_side(nt, 5, False)), list(_side(ns, 6, True))
        V = torch.randn(1, ns, device="cuda", generator=torch.Generator(device="cuda").manual_seed(7))
        bad = {"V": V[0], "sw": S[3], "sz": None if S[2] is None else S[2][0], "sx": S[0], "tx": T[0],
               "tz": None if T[2] is None else T[2][1]}[what]
        bad[1234] = float("nan")
        Y = G.ops.gauss_product(BASE, NORM, T[0], T[1], S[0], S[1], V, tz=T[2], tw=T[3], sz=S[2], sw=S[3])
        want = torch.zeros_like(Y)
        g = lib.gpl_gauss(BASE, NORM)
        p = G.ops._ptr
        lib.call("gpl_gauss_product", C.byref(g), nt, p(T[0]), p(T[1]), p(T[2]), p(T[3]), ns, p(S[0]), p(S[1]),
                 p(S[2]), p(S[3]), 1, p(V), ns, p(want), nt, 0.0, G.ops._stream())
        assert torch.equal(torch.isnan(Y), torch.isnan(want)), what
        ok = ~torch.isnan(want)
        if ok.any():
            assert torch.allclose(Y[ok], want[ok], rtol=1e-4, atol=1e-6 * float(want[ok].abs().max())), what
