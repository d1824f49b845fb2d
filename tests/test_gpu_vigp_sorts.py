"""The variational step where its two point sets are sorted apart, together, or a
small one beside a large one (up to 4,096 points a set is sorted by one workgroup),
against the oracle with the bounds of the step's own test."""
import pytest

from test_gpu_vigp import LAYERS
from test_gpu_vigp_sizes import G, test_vigp_elbo_and_gradient_sizes as check  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,gn", [(66, 7), (9, 66), (65, 65)])
def test_vigp_sorts(G, n, gn):  # noqa: F811
    check(G, n, 1, gn, LAYERS)
