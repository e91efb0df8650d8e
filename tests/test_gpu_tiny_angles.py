"""Opening angles whose squares leave the normal range: two particles a
distance of 2e-139 apart and single ones at distances around r / theta, where
the geometric decision takes its stated form.  Lists against the oracle's, bit
for bit."""
import numpy as np
import pytest

from oracle import oracle as orc
from tests.gpu_util import say, tree_parts

pytestmark = pytest.mark.gpu

R = 1e-139


def pair_and_far(theta):
    """The pair at the origin, and particles at r / theta times 1 -+ k / 10^4
    in the box's corners' directions."""
    k = np.arange(-20, 21) * 1e-4
    d = R / theta * (1.0 + k)
    s = np.array([[i & 1, (i >> 1) & 1, (i >> 2) & 1] for i in range(8)])[np.arange(len(k)) % 8] * 2.0 - 1.0
    x = np.concatenate([[[0.0, 0.0, 0.0], [2 * R, 0.0, 0.0]], s / np.sqrt(3.0) * d[:, None]])
    return (*(np.ascontiguousarray(x[:, i]) for i in range(3)), np.full(len(x), 1.0 / len(x)))


@pytest.mark.parametrize("theta", [1e-140, 1e-150, 3e-153, 1e-154, 1e-158, 1e-160, 1e-161, 1e-165])
def test_lists_bit_exact(theta):
    say("tiny angle", theta)
    p = pair_and_far(theta)
    s, _ = tree_parts(*p, n_crit=1)
    s.compute_moments()
    s.walk(theta)
    far, near = s.get_lists()
    t = orc.Tree(*p, n_crit=1)
    t.compute_moments()
    t.walk(theta)
    ofar, onear = t.lists()
    pair = np.flatnonzero(t.moments()[:, 4] == R)  # the pair's leaf and the chain of cells above it
    assert np.isin(ofar, pair).any() and np.isin(onear, pair).any()  # the angle divides the particles
    assert np.array_equal(far, ofar)
    assert np.array_equal(near, onear)
