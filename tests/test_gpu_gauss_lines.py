"""Gaussian products on both sides of the lines from which they are sorted first and from
which all pairs go by sixteen waves instead of eight: many targets and few sources, few
and many, one set of points, against FP64 with the sorted products' bound."""
import pytest

import test_gpu_gauss_tiles as tiles

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tshape,sshape", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("nt,ns,cols", [
    (20011, 20011, 1), (13001, 16385, 3), (16385, 8193, 2), (100003, 4097, 9),  # sorted with any shapes or with both
    (16384, 512, 3), (16384, 513, 3), (16385, 1024, 2), (40960, 700, 1), (40961, 700, 1), (70, 2561, 8),
    (33, 17000, 1)])
def test_lines(tshape, sshape, nt, ns, cols):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    print("[case] gauss lines", tshape, sshape, nt, ns, cols, flush=True)
    T, S = tiles._side(nt, 1, tshape), tiles._side(ns, 2, sshape)
    if nt == ns:
        S = (T[0], T[1]) + S[2:]
    V = torch.randn(cols, ns, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    Y = G.ops.gauss_product(tiles.BASE, tiles.NORM, T[0], T[1], S[0], S[1], V, tz=T[2], tw=T[3], sz=S[2], sw=S[3])
    for i0 in range(0, nt, 8192):  # FP64 in parts
        part = [None if v is None else v[..., i0:i0 + 8192] for v in T]
        want, scale = tiles._dense(part, S, V)
        assert torch.all((Y[:, i0:i0 + 8192].double() - want).abs() <= 1e-5 * scale + 1e-12 * scale.max())
