"""Lengths and masses scaled by powers of two, which round nothing: every output
of the FP64 far field scales exactly, bit for bit, in any units in which the
particles, the cells' moments and the outputs are themselves in range
(cosmology in metres and kilograms among them: 10^27 and 10^48)."""
import numpy as np
import pytest
import torch

from paper_1706_06989_amd import amfmm
from paper_1706_06989_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

# exponents of the unit of length and of mass
UNITS = [(60, -640), (60, 320), (75, 160), (90, 160), (90, -320), (120, -480), (120, 80), (135, -160), (30, -480), (15, 480),
         (-15, -480), (-30, 480), (-60, 640), (-60, -320), (-120, 320), (-135, 160)]


def solve(lengths, masses, noalloc, softening, kw):
    x, y, z, m = W.plummer(3000, seed=5)
    p = to_dev(*(np.ldexp(v, lengths) for v in (x, y, z)), np.ldexp(m, masses))
    s = amfmm.Solver(softening=float(np.ldexp(softening, lengths)), **kw)
    out = s._outputs(3000, True)
    (s.solve_gravity_noalloc if noalloc else s.solve_gravity)(*p, 0.5, out=out)
    ax, ay, az, pot = (v.cpu().numpy() for v in out)
    s.close()
    return np.stack([*(np.ldexp(v, 2 * lengths - masses) for v in (ax, ay, az)), np.ldexp(pot, lengths - masses)])


@pytest.mark.parametrize("order,variant,softening,noalloc", [
    (3, amfmm.UC, 0.0, False), (3, amfmm.TC, 0.0, False), (3, amfmm.TC, 0.0, True), (4, amfmm.UC, 0.0, False),
    (4, amfmm.TC, 0.0, False), (4, amfmm.TC, 0.125, False), (4, amfmm.TC, 64.0, False)])
def test_outputs_scale_exactly(order, variant, softening, noalloc):
    say("units", order, variant, softening, noalloc)
    kw = dict(order=order, variant=variant)
    ref = solve(0, 0, noalloc, softening, kw)
    assert np.isfinite(ref).all()
    for lengths, masses in UNITS:
        # the moments of order P (in mass length^P), their shifts and the
        # outputs' coefficients (mass / length^(P+1)) within 2^-960 .. 2^960
        low, high = sorted([masses + (order + 1) * lengths, masses - (order + 2) * lengths])
        if not (low > -880 and high < 880):
            continue
        got = solve(lengths, masses, noalloc, softening, kw)
        assert np.array_equal(got, ref), (lengths, masses, np.abs(got / ref - 1).max())


@pytest.mark.parametrize("order,variant", [(3, amfmm.UC), (3, amfmm.TC), (4, amfmm.TC)])
def test_a_softening_far_beyond_the_box(order, variant):
    """The unit of length follows the larger of the two."""
    a = solve(0, 0, False, 2.0 ** 40, dict(order=order, variant=variant))
    b = solve(0, 0, False, 2.0 ** 41, dict(order=order, variant=variant))
    assert np.isfinite(a).all()
    # potentials M / eps, accelerations by eps^3
    assert np.abs(a[3] / b[3] / 2 - 1).max() < 1e-12
    assert np.linalg.norm(a[:3] - 8 * b[:3]) <= 1e-12 * np.linalg.norm(a[:3])
