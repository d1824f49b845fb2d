"""The adjoint of the k-NN weights where a point's shares cancel: pairs of mutual nearest
neighbours with opposite parameters, whose shares are opposite numbers bit for bit, and a
third point of 2^-16 of them whose nearest neighbour is one of the pair. A lengthscale
far beyond the image leaves no other gradient. Each point's shares are summed in FP64 and
rounded once: what is left is good to FP32 (1e-4 with the differences of the lens
Jacobian across a pixel), where a share rounded by itself is off by 2^16 times that."""
import dataclasses

import numpy as np
import pytest

from helpers import gpu_problem
import synth
from oracle import vigp as ov

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,count", [(24, 12), (32, 1)])
def test_cancelling_shares(n, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] vigp shares", n, count, flush=True)
    w = synth.workload(1).replace(n=n, ss=1)
    prob = gpu_problem(w)
    prob = prob.replace(source=dataclasses.replace(prob.source, peak=0.0))
    lens = np.array([1.1, 0.8, 1.0, 2.0, 0.05, -0.03, 0.0, 0.0])
    px, py = (v.double().cpu().numpy() for v in G.ops.lens_raytrace(prob.grid, G.Lens(*lens)))
    d2 = (px[:, None] - px) ** 2 + (py[:, None] - py) ** 2
    np.fill_diagonal(d2, np.inf)
    near = np.sort(d2, 1)
    clear, nn = near[:, 1] > near[:, 0] * (1 + 1e-4), d2.argmin(1)
    mean, used = np.zeros(n * n), set()
    for j in range(n * n):
        o = nn[j]
        if nn[o] != j or not (clear[j] and clear[o]) or len(used) == 3 * count:
            continue
        for t in np.flatnonzero(nn == j):
            if t != o and clear[t] and not {j, o, t} & used:
                mean[j], mean[o], mean[t] = 1.0, -1.0, 2.0 ** -16
                used |= {j, o, t}
                break
    assert len(used) == 3 * count
    layers = (("ip", 1e6),)
    d = np.ones(n * n)
    src = (0.0, w.source.R_e, w.source.n_sersic, w.source.xs, w.source.ys)
    om = ov.Model(n, 1, w.pix_scale, lens[3], src, w.noise_sigma, w.psf_fwhm, layers, knn_k=1)
    P = dict(lens_mean=lens[list(ov.FREE)], lens_raw=np.zeros((7, 7)), log_amp=np.zeros(1), ip_mean=[mean],
             ip_logs=[np.zeros(n * n)])
    eps = dict(e_l=np.zeros(7), e_ip=[np.zeros(n * n)])
    v = G.vigp.Vigp(G.vigp.VigpModel(layers, lens[3], knn_k=1), prob, torch.ones(n * n, device="cuda"))
    v.lens_mean.copy_(torch.as_tensor(P["lens_mean"]))
    v.ip[0]["mean"].copy_(torch.as_tensor(mean))
    v.elbo(torch.zeros(7, dtype=torch.float64, device="cuda"), torch.zeros(n * n, device="cuda"))
    want = ov.elbo(om, P, eps, d, want_grad=True, points=(px, py))[2]["lens_mean"]
    got = v.G64[:7].cpu().numpy()
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    print("relative error", err)
    assert err <= 1e-4
