"""The variational step where the pixels' shapes lie on the line from which a target is
taken by workgroups of its own (largest eigenvalue above 8 l^2 / 2): undeflected square
pixels, all of the same shape up to rounding, at lengthscales just on either side of the
line and on it, where rounding divides them. Against the oracle with the bounds of the
step's own test."""
import math

import numpy as np
import pytest

from oracle import vigp as ov
from test_gpu_vigp import _rel, _setup, t64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("off", [-1e-3, -1e-5, -3e-6, 0.0, 1e-3])
@pytest.mark.parametrize("n", [9, 21])
def test_far_line(n, off):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] vigp far", n, off, flush=True)
    ell = 0.5 * 0.05 / math.sqrt(4 * math.pi) * math.sqrt(1.00001) * (1 + off)  # lambda = pixel^2 / (4 pi) = 4 l^2
    w, d, prob, om, P, eps, v, e64, e32 = _setup(G, n, 1, 5, 0.04, 40 + n, (("ip", ell), ("ip", 0.05)))
    assert w.pix_scale == 0.05
    P["lens_mean"] = np.array([1e-9, 0.8, 1.0, 0.0, 0.0, 0.0, 0.0])
    P["lens_raw"] = np.diag(np.full(7, -30.0))
    v.lens_mean.copy_(torch.as_tensor(P["lens_mean"]))
    v.lens_raw.copy_(torch.as_tensor(P["lens_raw"]))
    out = t64(v.elbo(e64, e32))
    pts = G.ops.lens_raytrace(prob.grid, G.Lens(*out[5:13]))
    E, pc, g = ov.elbo(om, P, eps, d, want_grad=True, points=(t64(pts[0]), t64(pts[1])))
    assert abs(out[1] - pc["loglik"]) <= 1e-6 * (abs(pc["loglik"]) + abs(pc["logprior_y"]) + abs(pc["neg_logq"]))
    G32 = t64(v.G32)  # (the lens gradient is not unique here: the k-th neighbours are ties)
    o = 0
    for gm, gl in zip(g["ip_mean"], g["ip_logs"]):
        assert _rel(G32[o:o + om.N], gm) <= 1e-4 and _rel(G32[o + om.N:o + 2 * om.N], gl) <= 1e-4
        o += 2 * om.N
