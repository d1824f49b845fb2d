"""Which Gaussian products ask for the workspace of the sorted route: none whose sorts cost
more than its pairs (many targets and few sources), all large ones."""
import pytest


@pytest.mark.parametrize("nt,ns,cols,sorts", [
    (400000, 300, 1, False), (400000, 256, 17, False), (16384, 257, 8, False), (4200000, 1, 3, False),
    (65, 65000, 1, True), (2500, 2500, 1, True), (40000, 40000, 1, True), (40000, 10000, 3, True), (1600, 40000, 2, True),
    (2000000, 2000000, 8, True), (2000, 2000, 1, False), (0, 100, 1, False), (100, 0, 1, False)])
def test_sorted_where_it_pays(nt, ns, cols, sorts):
    L = pytest.importorskip("paper_2105_09465_amd._lib")
    assert (L.lib.gpl_gauss_product_workspace(nt, ns, cols) > 0) == sorts
