"""The cells of all levels from one pass over the sorted keys, against the
oracle's level-by-level tree: particle counts around the kernels' tile of 1024,
leaf sizes from one particle to the largest, coincident particles (leaves at
the deepest level) and clusters that make deep, narrow trees; and the upward
pass over their few- and many-celled levels."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1706_06989_amd import workloads as W
from tests.gpu_util import say, tree_parts

pytestmark = pytest.mark.gpu


def clustered(n, seed):
    """Plummer spheres of ever smaller scale (deep trees) with copies of one
    point across a tile boundary."""
    x, y, z, m = W.plummer(n, seed=seed)
    k = np.arange(n) % 5
    s = 10.0 ** (-1.5 * k)
    x, y, z = x * s, y * s, z * s
    c = slice(n // 2, n // 2 + min(60, n // 4))
    x[c], y[c], z[c] = x[n // 2], y[n // 2], z[n // 2]
    return x, y, z, m


@pytest.mark.parametrize("n,n_crit", [(1, 1), (2, 1), (63, 1), (1023, 25), (1024, 25), (1025, 25), (2049, 1), (5000, 2),
                                      (4097, 31), (4096, 32), (9000, 63), (4096, 4096), (4097, 4096), (12289, 4095),
                                      (70001, 25), (70001, 4096)])
@pytest.mark.parametrize("shape", ["uniform", "clustered"])
def test_tree_and_moments_match_the_oracle(shape, n, n_crit):
    say("tree levels", shape, n, n_crit)
    x, y, z, m = W.uniform_cube(n, seed=n) if shape == "uniform" else clustered(n, seed=n)
    s, _ = tree_parts(x, y, z, m, n_crit=n_crit)
    g = s.get_tree()
    t = orc.Tree(x, y, z, m, n_crit=n_crit)
    c = t.cells()
    for f in ("level", "begin", "count", "parent", "child0", "nchild"):
        assert np.array_equal(g[f], c[f]), f
    assert s.get_counts()["leaves"] == int(np.sum(c["nchild"] == 0))
    s.compute_moments()
    t.compute_moments()
    gm, om = s.get_moments(), t.moments()
    # mass, centre of mass and R_max decide the walk: bit for bit
    assert np.array_equal(gm[:, :5], om[:, :5])
    M, R = om[:, 0:1], om[:, 4:5]
    assert np.all(np.abs(gm[:, 5:11] - om[:, 5:11]) <= 1e-12 * M * R**2 + 1e-300)
    assert np.all(np.abs(gm[:, 11:21] - om[:, 11:21]) <= 1e-12 * M * R**3 + 1e-300)
