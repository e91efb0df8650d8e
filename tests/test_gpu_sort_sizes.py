"""The key sort's three forms (one workgroup in LDS, tiles whose histograms the
scatter sums itself, scanned tiles) at the sizes where they change over and at
tile remainders: keys and permutation against the oracle's, bit for bit, with
runs of equal keys across tile and wave boundaries (stability)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1706_06989_amd import workloads as W
from tests.gpu_util import say, tree_parts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 64, 65, 1000, 8191, 8192, 8193, 9217, 40000, 131071, 131072, 131073, 266241])
def test_keys_and_permutation(n):
    say("sort", n)
    x, y, z, m = W.plummer(n, seed=n)
    # a third of the particles on 50 points, in no order
    rng = np.random.default_rng(n)
    pick = rng.choice(n, n // 3, replace=False)
    at = rng.integers(0, min(50, n), len(pick))
    x[pick], y[pick], z[pick] = x[at], y[at], z[at]
    s, _ = tree_parts(x, y, z, m)
    g = s.get_tree()
    k, p = orc.Tree(x, y, z, m).keys()
    assert np.array_equal(g["keys"], k)
    assert np.array_equal(g["perm"], p)
