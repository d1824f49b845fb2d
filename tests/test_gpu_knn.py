"""The k-NN density at the edges of its kernel's tiles: point counts around the
32-point chunks and 64-point tiles, the smallest and largest k, many equal
distances, and points far from all others."""
import numpy as np
import pytest

from oracle import window as owin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2105_09465_amd as G
    return G


def _points(kind, n):
    rng = np.random.default_rng(110 + n)
    if kind == "grid":  # equal distances in every neighbourhood
        i = np.arange(n)
        return np.stack([i % 17, i // 17]).astype(np.float32) * np.float32(0.03125)
    q = rng.uniform(-1, 1, (2, n)).astype(np.float32)
    if kind == "clumps":  # tight clumps far apart: neighbours across the curve's ends
        q = (q * 0.01 + rng.integers(0, 4, (2, n)) * 3.0).astype(np.float32)
    return q


@pytest.mark.parametrize("kind", ["uniform", "grid", "clumps"])
@pytest.mark.parametrize("n,k", [(2, 1), (33, 32), (63, 20), (64, 1), (65, 32), (129, 20), (2047, 32)])
def test_knn_density_tile_edges(G, kind, n, k):
    """rho = k / (pi r_k^2). FP32 differences and squares put a relative error of
    at most 3 x 2^-24 on each squared distance (an order statistic moves by no
    more than that), the quotient and its product two roundings more: 5e-7."""
    print("[case] knn", kind, n, k, flush=True)
    q = _points(kind, n)
    dev = [torch.as_tensor(v, device="cuda") for v in q]
    rho = G.ops.knn_density(dev[0], dev[1], k).double().cpu().numpy()
    want = owin.knn_density(q[0].astype(np.float64), q[1].astype(np.float64), k)
    assert np.max(np.abs(rho - want) / want) <= 5e-7
