"""The operator A with B^T X (and the pixel shapes of the windowed kernel) formed beside
the tile plan's kernels, against its parts called one by one: around the size of the
one-workgroup plan, with a ragged last tile, several columns and no PSF, where the
windowed product changes from all pairs to sorted ones, and past the plan's split that
one workgroup holds. The parts see the same numbers in the same order, so the product
has the same bits and two FP32 roundings of the last sum are left."""
import pytest

import synth
from helpers import gpu_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,ss,cols,prec,kind,fwhm", [
    (64, 1, 3, "f16x3", 0, 0.1), (65, 1, 17, "f16x3", 0, 0.1), (65, 1, 19, "fp32", 0, 0.1), (33, 2, 1, "f16x3", 0, 0.3),
    (66, 1, 65, "f16x3", 0, 0.0), (130, 1, 2, "fp32", 0, 0.1), (513, 1, 1, "f16x3", 0, 0.1),
    (40, 1, 2, "fp32", 1, 0.1), (46, 1, 3, "fp32", 1, 0.1), (64, 1, 2, "fp32", 1, 0.1), (33, 2, 9, "fp32", 1, 0.1),
    (65, 1, 1, "fp32", 1, 0.0)])
def test_operator_against_its_parts(n, ss, cols, prec, kind, fwhm):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] operator", n, ss, cols, prec, kind, fwhm, flush=True)
    prob = gpu_problem(synth.workload(1).replace(n=n, ss=ss, psf_fwhm=fwhm))
    prob = prob.replace(kernel=G.Kernel(0.04, 0.3, kind=kind))
    px, py = G.ops.lens_raytrace(prob.grid, prob.lens)
    X = torch.randn(cols, n * n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    X[0] *= 1e-4
    for _ in range(2):  # a second call finds the first one's numbers in its scratch memory
        Y = G.ops.apply_A(prob, px, py, X, prec=prec)
        T1 = G.ops.psf_conv(prob.grid, prob.psf, X, adjoint=True)
        T2 = G.ops.kernel_mvm(prob.kernel, px, py, T1, prec=prec, grid=prob.grid)
        BT2 = G.ops.psf_conv(prob.grid, prob.psf, T2, adjoint=False).double()
        s2X = float(torch.tensor(prob.noise_sigma ** 2, dtype=torch.float32)) * X.double()
        assert torch.all((Y.double() - (BT2 + s2X)).abs() <= 2 ** -23 * (BT2.abs() + s2X.abs()))
        X = X.flip(1).contiguous()
