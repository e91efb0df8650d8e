"""A timeline longer than the device's clock words: many evaluations of one walk
go on adding to the phases that they run."""
import pytest
import torch

from paper_1706_06989_amd import amfmm
from paper_1706_06989_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [3, 4])
def test_many_evaluations(order):
    p = to_dev(*W.plummer(2000, seed=4))
    s = amfmm.Solver(order=order)
    s.build_tree(*p)
    s.compute_moments()
    s.walk(0.5)
    start = s.get_phase_times()
    out = s.evaluate()

    def run(k):
        before = s.get_phase_times()
        for _ in range(k):
            s.evaluate(out=out)
        after = s.get_phase_times()
        return {q: (after[q] - before[q]) / k for q in ("far", "push-down", "near+eval", "total")}

    run(1000)
    few = run(2000)  # within the words: three to ten marks an evaluation
    say("ms an evaluation", few)
    many = run(40000)
    say("ms an evaluation", many)
    for q, v in few.items():
        assert 0.5 * v <= many[q] <= 2.0 * v, (q, v, many[q])
    # what came before is still there, and a new tree starts anew
    t = s.get_phase_times()
    for q in ("validate+bbox", "keys+sort", "tree", "moments"):
        assert t[q] == pytest.approx(start[q], abs=1e-9), q
    s.build_tree(*p)
    torch.cuda.synchronize()
    t = s.get_phase_times()
    assert t["near+eval"] == 0.0 and 0.0 < t["total"] < 10.0
    s.close()
