"""The geometric decision taken first without root and division, against the
oracle's lists where it is closest: regular lattices, whose cells repeat a few
radii and distances, at opening angles that put many pairs at d = r / theta to
the last bit, and at scales whose squares leave the normal range."""
import numpy as np
import pytest

from oracle import oracle as orc
from tests.gpu_util import say, tree_parts

pytestmark = pytest.mark.gpu

# r / d of lattice cells of equal size: sqrt(3) to sqrt(1/8) over small integers
ANGLES = [np.sqrt(3.0) / 4, np.sqrt(3.0) / 6, np.sqrt(3.0 / 8), np.sqrt(3.0 / 20), 0.5, 1.0]


def lattice(k, scale):
    g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) * scale
    return (*(np.ascontiguousarray(g[:, i]) for i in range(3)), np.full(len(g), 1.0 / len(g)))


@pytest.mark.parametrize("scale", [1.0, 0.1, 1e-151])
@pytest.mark.parametrize("theta", ANGLES)
def test_lattice_lists_bit_exact(theta, scale):
    say("lattice lists", theta, scale)
    p = lattice(16, scale)
    s, _ = tree_parts(*p, n_crit=1)
    s.compute_moments()
    s.walk(float(theta))
    far, near = s.get_lists()
    t = orc.Tree(*p, n_crit=1)
    t.compute_moments()
    t.walk(float(theta))
    ofar, onear = t.lists()
    assert np.array_equal(far, ofar)
    assert np.array_equal(near, onear)
