"""Phase times from the device clock: every phase of a solve is there, in range
of the wall clock, with whole and batched walks, staged calls and repeats."""
import time

import pytest
import torch

from paper_1706_06989_amd import amfmm
from paper_1706_06989_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def check(t, wall_ms, least):
    assert set(t) == set(amfmm.PHASES)
    assert all(v >= 0.0 for v in t.values()), t
    phases = [t[k] for k in amfmm.PHASES[:8]]
    assert abs(sum(phases) - t["total"]) <= 1e-9 * max(1.0, t["total"])
    assert t["walk-pass"] <= t["walk"]
    assert all(t[k] > 0.0 for k in least), t
    assert t["total"] <= wall_ms, (t, wall_ms)


@pytest.mark.parametrize("n,order,list_bytes", [(1, 3, 0), (4096, 3, 0), (100003, 3, 0), (60000, 4, 0), (100003, 3, 1 << 20)])
def test_solve(n, order, list_bytes):
    say("phase times", n, order, list_bytes)
    p = to_dev(*W.plummer(n, seed=n))
    s = amfmm.Solver(order=order, list_bytes=list_bytes)
    for _ in range(2):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        s.solve_gravity(*p, 0.5)
        torch.cuda.synchronize()
        wall = 1e3 * (time.perf_counter() - t0)
        check(s.get_phase_times(), wall, [k for k in amfmm.PHASES[:8] if n > 1 or k not in ("push-down", "far")])


def test_staged_calls():
    p = to_dev(*W.plummer(30000, seed=4))
    s = amfmm.Solver()
    t0 = time.perf_counter()
    s.build_tree(*p)
    first = s.get_phase_times()
    assert first["tree"] > 0.0 and first["walk"] == 0.0 and first["near+eval"] == 0.0
    s.compute_moments()
    s.walk(0.5)
    s.evaluate()
    torch.cuda.synchronize()
    check(s.get_phase_times(), 1e3 * (time.perf_counter() - t0), amfmm.PHASES[:8])
