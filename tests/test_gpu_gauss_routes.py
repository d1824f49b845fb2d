"""Gaussian products around the sizes from which they are sorted first (with shapes on
both sides 2^22 pairs, else 3 * 2^25), on both routes: within the sorted products'
bounds of FP64, and equal to the all-pairs entry up to the order of the sums."""
import ctypes as C

import pytest

import test_gpu_gauss_tiles as tiles
from test_gpu_gauss_tiles import G, test_sorted_product_vs_dense as check  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tshape,sshape", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("nt,ns,cols", [(10033, 10034, 1), (10034, 10034, 3), (39000, 2600, 2), (2047, 2049, 4),
                                        (2047, 2051, 1)])
def test_routes(G, tshape, sshape, nt, ns, cols):  # noqa: F811
    if G._lib.lib.gpl_gauss_product_workspace(nt, ns, cols) > 0:
        check(G, tshape, sshape, nt, ns, cols)
    T, S = tiles._side(nt, 1, tshape), tiles._side(ns, 2, sshape)
    V = torch.rand(cols, ns, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    Y = G.ops.gauss_product(tiles.BASE, tiles.NORM, T[0], T[1], S[0], S[1], V, tz=T[2], tw=T[3], sz=S[2], sw=S[3])
    want, par, p = torch.empty_like(Y), G._lib.gpl_gauss(tiles.BASE, tiles.NORM), G.ops._ptr
    G._lib.call("gpl_gauss_product", C.byref(par), nt, p(T[0]), p(T[1]), p(T[2]), p(T[3]), ns, p(S[0]), p(S[1]),
                p(S[2]), p(S[3]), cols, p(V), ns, p(want), nt, 0.0, G.ops._stream())
    # positive terms: two orders of at most 39,000 FP32 additions, 2e-5 of the sum
    assert ((Y - want).abs() <= 2e-5 * want + 1e-30).all()
