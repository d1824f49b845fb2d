"""The variational step at sizes around its tiles (16-target subtiles, 64-point
tiles, shares of the sources): the smallest images the k-NN weights allow,
ragged ones, and a grid larger than the image's points, against the oracle with
the bounds of the step's own test."""
import numpy as np
import pytest

from oracle import vigp as ov
from test_gpu_vigp import LAYERS, _rel, _setup, t64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    return G


@pytest.mark.parametrize("n,ss,gn,layers", [(5, 1, 5, LAYERS), (8, 1, 40, LAYERS), (23, 1, 9, LAYERS[:2]),
                                            (40, 1, 21, LAYERS), (27, 2, 16, (("sp", 0.1), ("ip", 0.01)))])
def test_vigp_elbo_and_gradient_sizes(G, n, ss, gn, layers):
    print("[case] vigp sizes", n, ss, gn, len(layers), flush=True)
    w, d, prob, om, P, eps, v, e64, e32 = _setup(G, n, ss, gn, 0.04, 190 + n, layers)
    out = t64(v.elbo(e64, e32))
    pts = G.ops.lens_raytrace(prob.grid, G.Lens(*out[5:13]))
    E, pc, g = ov.elbo(om, P, eps, d, want_grad=True, points=(t64(pts[0]), t64(pts[1])))
    mag = abs(pc["loglik"]) + abs(pc["logprior_y"]) + abs(pc["logprior_theta"]) + abs(pc["neg_logq"])
    for a, b in zip(out[:5], (E, pc["loglik"], pc["logprior_y"], pc["logprior_theta"], pc["neg_logq"])):
        assert a == b or abs(a - b) <= 1e-6 * mag
    G64, G32 = t64(v.G64), t64(v.G32)
    assert _rel(G64[0:7], g["lens_mean"]) <= 1e-4
    o = 0
    if "sp_mean" in g:
        want = np.concatenate([g["sp_mean"], g["sp_logs"], g["sp_cross"].T.ravel()])
        o = want.size
        assert _rel(G32[:o], want) <= 1e-4
    for gm, gl in zip(g["ip_mean"], g["ip_logs"]):
        assert _rel(G32[o:o + om.N], gm) <= 1e-4 and _rel(G32[o + om.N:o + 2 * om.N], gl) <= 1e-4
        o += 2 * om.N
