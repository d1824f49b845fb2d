"""Conjugate gradients with everything between two products in one workgroup a column
(images of up to 64 x 64 pixels and 4,096 fine points) and in five launches (the
others), against the same recurrence in FP64 around the library's product with A: a
few steps, so that the FP32 vectors' rounding stays far below the bound."""
import numpy as np
import pytest

import synth
from helpers import gpu_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,ss,prec,fwhm", [(2, 1, "fp32", 0.1), (31, 1, "f16x3", 0.1), (33, 1, "fp32", 0.1),
                                            (64, 1, "f16x3", 0.3), (65, 1, "f16x3", 0.1), (32, 2, "fp32", 0.1),
                                            (33, 2, "f16x3", 0.1), (5, 3, "f16x3", 0.0), (16, 4, "f16x3", 0.1)])
@pytest.mark.parametrize("check_every", [0, 2])
def test_cg_steps(n, ss, prec, fwhm, check_every):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] cg column", n, ss, prec, fwhm, check_every, flush=True)
    prob = gpu_problem(synth.workload(1).replace(n=n, ss=ss, psf_fwhm=fwhm))
    px, py = G.ops.lens_raytrace(prob.grid, prob.lens)
    npix, steps, tol = n * n, 5, 0.2
    rng = np.random.default_rng(n)
    B = rng.standard_normal((4, npix)).astype(np.float32)
    B[1] = 0
    B[3] = 1e-3 * np.abs(B[3])
    res = G.ops.cg_solve(prob, px, py, torch.as_tensor(B, device="cuda"), tol=tol, max_iter=steps, n_lanczos=steps,
                         check_every=check_every, prec=prec)
    X, R = np.zeros_like(B, dtype=np.float64), B.astype(np.float64)
    P, iters = R.copy(), np.zeros(4, int)
    ab = np.zeros((4, steps, 2))
    rr, active = (R * R).sum(1), (R * R).sum(1) > 0
    bb = rr.copy()
    for it in range(steps):
        AP = G.ops.apply_A(prob, px, py, torch.as_tensor(P.astype(np.float32), device="cuda"),
                           prec=prec).double().cpu().numpy()
        for c in np.flatnonzero(active):
            a = rr[c] / (P[c] @ AP[c])
            X[c] += a * P[c]
            R[c] -= a * AP[c]
            new = R[c] @ R[c]
            ab[c, it] = a, new / rr[c]
            P[c] = R[c] + new / rr[c] * P[c]
            rr[c], iters[c] = new, it + 1
            active[c] = np.sqrt(new) > tol * np.sqrt(bb[c])
    assert (res["iters"].cpu().numpy() == iters).all(), (res["iters"], iters)
    got = res["X"].double().cpu().numpy()
    assert np.linalg.norm(got - X) <= 1e-4 * np.linalg.norm(X)
    assert (got[1] == 0).all()
    # alpha, and beta where it is not the rounding of a solved system (four pixels take three steps)
    gab = res["ab"].cpu().numpy()
    solved = ab[..., 1] < 1e-6
    assert np.allclose(gab[..., 0], ab[..., 0], rtol=1e-3, atol=0)
    assert np.allclose(gab[..., 1][~solved], ab[..., 1][~solved], rtol=1e-3, atol=0) and (gab[..., 1][solved] < 1e-6).all()
    live = rr > 1e-6 * bb
    assert np.allclose(res["relres"].cpu().numpy()[live], np.sqrt(rr[live] / bb[live]), rtol=1e-3)
