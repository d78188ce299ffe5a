"""Search and row pattern on both sides of the size up to which the kernels
find their own offsets (67,584 slave elements or nodes) at a third of it, and at
the size up to which a slave element has eight lanes (32,768), with lists longer
than the short fill holds on either side, against the oracle bit for bit."""

import numpy as np
import pytest

from tests.test_gpu_candidate_lists import test_lists as check_lists
from tests.test_gpu_search_sizes import test_search as check_search

pytestmark = pytest.mark.gpu

LONG = (33, 2, 49, 48, 32, 1, 40)


# elements / nodes: 20,480 / 20,769; 20,193 / 20,480; 20,608; 32,768; 32,896;
# 67,584 / 68,105; 67,065 / 67,584; 67,840
@pytest.mark.parametrize("nx,ny", [(160, 128), (159, 127), (161, 128), (256, 128), (257, 128), (264, 256), (263, 255),
                                   (265, 256)])
def test_sizes(nx, ny):
    check_search(nx, ny, 0.0)


@pytest.mark.parametrize("n", [20480, 20481, 32768, 32769, 67584, 67585])
def test_long_lists(n):
    rng = np.random.default_rng(n)
    counts = np.ones(n, dtype=int)
    counts[rng.permutation(n)[:200]] = rng.choice(LONG, 200)
    check_lists(tuple(counts.tolist()))
