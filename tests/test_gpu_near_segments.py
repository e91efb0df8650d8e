"""Near-field lists cut into segments: a few wide leaves around a compact core
face the whole core in direct summation, so that their lists are cut, beside
thousands of short lists that are not.  Leaves of one and of several blocks of
64 targets, entries far larger than the staging buffer and lists of many small
ones, both precisions, against the oracle (FP64 to 1e-12 of the sum of
magnitudes; mixed to its bars, 2e-6 at the 99th percentile and 1e-4)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1706_06989_amd import amfmm
from tests.gpu_util import gpu_solve, say

pytestmark = pytest.mark.gpu


def core_and_halo(n, halo, seed):
    """n - 7 halo particles in a unit ball inside one octant of a box of side
    20, `halo` spread over each of the seven others."""
    rng = np.random.default_rng(seed)
    k = n - 7 * halo
    v = rng.standard_normal((k, 3))
    v *= (rng.random(k) ** (1 / 3) / np.linalg.norm(v, axis=1))[:, None]
    parts = [v + 3.0]
    for o in range(7):
        sign = np.array([o & 1, (o >> 1) & 1, (o >> 2) & 1]) * 2 - 1
        parts.append(rng.uniform(0.5, 10.0, (halo, 3)) * sign)
    x = np.concatenate(parts)
    x[-1], x[-2] = -10.0, 10.0  # the box
    return (*(np.ascontiguousarray(x[:, i]) for i in range(3)), rng.uniform(0.5, 1.5, n) / n)


@pytest.mark.parametrize("n,halo,n_crit,theta", [(16000, 3, 25, 0.5), (16000, 25, 25, 0.3), (12001, 100, 128, 0.4),
                                                 (9000, 150, 200, 0.3), (20011, 24, 25, 0.1), (5000, 1, 1, 0.3)])
@pytest.mark.parametrize("precision", [amfmm.FP64, amfmm.MIXED])
def test_cut_lists_match_the_oracle(n, halo, n_crit, theta, precision):
    say("near segments", n, halo, n_crit, theta, precision)
    x, y, z, m = core_and_halo(n, halo, seed=n)
    acc, pot, s = gpu_solve(x, y, z, m, theta, precision=precision, n_crit=n_crit)
    t = orc.Tree(x, y, z, m, n_crit=n_crit)
    t.compute_moments()
    t.walk(theta)
    oacc, opot = t.evaluate(amfmm.TC)
    _, _, gabs = orc.direct(x, y, z, m)
    err = np.linalg.norm(acc - oacc, axis=0) / gabs
    perr = np.abs(pot - opot) / np.abs(opot)
    if precision == amfmm.FP64:
        assert err.max() <= 1e-12 and perr.max() <= 1e-12, (err.max(), perr.max())
    else:
        assert np.percentile(err, 99) <= 2e-6 and err.max() <= 1e-4, (np.percentile(err, 99), err.max())
        assert np.percentile(perr, 99) <= 1e-6, np.percentile(perr, 99)
    # the directed particle interactions of the lists, i != j
    c = t.cells()["count"].astype(np.int64)
    _, near = t.lists()
    a, b = near[:, 0], near[:, 1]
    want = np.where(a == b, c[a] * (c[a] - 1), 2 * c[a] * c[b]).sum()
    assert s.get_counts()["near_interactions"] == want
