"""The adjoint entry of the Gaussian product (`gpl_gauss_product_backward`) against its
closed form in FP64, at the sizes where its workgroups change from eight waves to sixteen
(the steps of 64 points they sum over) and back (more than 16,384 points of their own)."""
import ctypes as C
import math

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BASE, NORM = 0.5 * 0.04 ** 2, 1.0 / (2 * math.pi)


@pytest.mark.parametrize("shapes,weights", [(True, True), (False, False)])
@pytest.mark.parametrize("nt,ns", [(1, 1), (70, 512), (513, 65), (1600, 1100), (2500, 2561), (16384, 513), (16385, 600),
                                   (600, 16385), (40961, 600)])
def test_adjoint_vs_closed_form(nt, ns, shapes, weights):
    """FP32 terms summed in FP32 over at most 16,385 points in 8 or 16 parts of 64-point
    runs: 1e-5 of the sum of the terms' magnitudes (the product's own bound)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] gauss adjoint", nt, ns, shapes, weights, flush=True)
    g = torch.Generator(device="cuda").manual_seed(nt + ns)
    u = lambda *s: torch.rand(*s, device="cuda", generator=g)  # noqa: E731
    T, S = 0.4 * u(2, nt), 0.4 * u(2, ns)
    tz = None
    if shapes:
        a, b = 0.03 * (2 * u(2, nt) - 1), 0.03 * (2 * u(2, nt) - 1)
        tz = torch.stack([a[0] ** 2 + b[0] ** 2, a[0] * a[1] + b[0] * b[1], a[1] ** 2 + b[1] ** 2])
    tw, sw = (0.5 + u(nt), 0.5 + u(ns)) if weights else (None, None)
    V, U = 2 * u(ns) - 1, 2 * u(nt) - 1
    g0 = [2 * u(5, nt) - 1, 2 * u(3, ns) - 1]
    gt, gs = (v.clone() for v in g0)
    p, par = G.ops._ptr, G._lib.gpl_gauss(BASE, NORM)
    G._lib.call("gpl_gauss_product_backward", C.byref(par), nt, p(T[0]), p(T[1]), p(tz), p(tw), ns, p(S[0]), p(S[1]),
                p(sw), p(V), p(U), p(gt[0]), p(gt[1]), p(gt[2:]) if shapes else None, p(gs[0]), p(gs[1]), p(gs[2]),
                G.ops._stream())
    d = lambda v: v.double()  # noqa: E731
    base = float(torch.tensor(BASE, dtype=torch.float32))
    z = d(tz) if shapes else torch.zeros(3, nt, dtype=torch.float64, device="cuda")
    cxx, cxy, cyy = z[0] + base, z[1], z[2] + base
    det = cxx * cyy - cxy ** 2
    inv = [(c / det)[:, None] for c in (cyy, -cxy, cxx)]
    dx, dy = d(T[0])[:, None] - d(S[0]), d(T[1])[:, None] - d(S[1])
    ux, uy = inv[0] * dx + inv[1] * dy, inv[1] * dx + inv[2] * dy
    w = (NORM * d(U) * (d(tw) if weights else 1.0) / det.sqrt())[:, None] * torch.exp(-0.5 * (dx * ux + dy * uy))
    e = w * (d(sw) if weights else 1.0) * d(V)  # every pair's share of F
    rows = [(-e * ux, (e * ux).abs()), (-e * uy, (e * uy).abs())]
    if shapes:
        for a, b, i in ((ux, ux, 0), (ux, uy, 1), (uy, uy, 2)):
            rows.append((0.5 * e * (a * b - inv[i]), 0.5 * e.abs() * ((a * b).abs() + inv[i].abs())))
    for k, (term, mag) in enumerate(rows):
        err = (d(gt[k]) - d(g0[0][k]) - term.sum(1)).abs()
        assert torch.all(err <= 1e-5 * mag.sum(1) + 1e-6 * (d(g0[0][k]).abs() + term.sum(1).abs())), k
    if not shapes:
        assert torch.equal(gt[2:], g0[0][2:])
    for k, (term, mag) in enumerate(((e * ux, (e * ux).abs()), (e * uy, (e * uy).abs()), (w * d(V), (w * d(V)).abs()))):
        err = (d(gs[k]) - d(g0[1][k]) - term.sum(0)).abs()
        assert torch.all(err <= 1e-5 * mag.sum(0) + 1e-6 * (d(g0[1][k]).abs() + term.sum(0).abs())), k
