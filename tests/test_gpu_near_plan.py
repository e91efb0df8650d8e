"""Which near-field lists are cut into segments, and what comes of them: the
room for the segments' partial sums holds every request (leaves of far more
particles than n_crit, at the deepest level, among them), so the choice depends
on the lists alone and repeated solves agree bit for bit; and cut lists under
softening, at order 4, in batches of subtrees, in the allocation-free solve and
with the other variants, against the oracle (FP64 to 1e-12 of the sum of
magnitudes; mixed to its bars, 2e-6 at the 99th percentile and 1e-4)."""
import re

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_1706_06989_amd import amfmm
from paper_1706_06989_amd import workloads as W
from tests.gpu_util import say, to_dev
from tests.test_gpu_near_segments import core_and_halo

pytestmark = pytest.mark.gpu


def clump(n, cells, seed):
    """All but eight of n particles in cells^3 neighbouring cells of the deepest
    level (2^-21 of a box of side 1), the eight at its corners."""
    rng = np.random.default_rng(seed)
    h = 2.0 ** -21
    x = 0.3 + np.floor(rng.random((n, 3)) * cells) * h + rng.random((n, 3)) * 0.9 * h
    x[:8] = [[i & 1, (i >> 1) & 1, (i >> 2) & 1] for i in range(8)]
    return (*(np.ascontiguousarray(x[:, i]) for i in range(3)), rng.uniform(0.5, 1.5, n) / n)


def plans(capfd):
    """(cut blocks, segments, room, partial sums, room) of every near-field call."""
    err = capfd.readouterr().err
    return [tuple(map(int, g)) for g in
            re.findall(r"cut blocks (\d+) segments (\d+) of (\d+) partial sums (\d+) of (\d+)", err)]


def host(o):
    torch.cuda.synchronize()
    return np.stack([v.cpu().numpy() for v in o])


def check(got, ref, gabs, precision):
    err = np.linalg.norm(got[:3] - ref[:3], axis=0) / gabs
    perr = np.abs(got[3] - ref[3]) / np.abs(ref[3])
    say("  ", err.max(), perr.max())
    if precision == amfmm.FP64:
        assert err.max() <= 1e-12 and perr.max() <= 1e-12, (err.max(), perr.max())
    else:
        assert np.percentile(err, 99) <= 2e-6 and err.max() <= 1e-4, (np.percentile(err, 99), err.max())
        assert np.percentile(perr, 99) <= 1e-6, np.percentile(perr, 99)


# (60000 and 200000 particles: leaves enough for several workgroups to ask at once)
@pytest.mark.parametrize("n,cells,n_crit", [(20000, 3, 25), (20000, 2, 25), (9001, 3, 1), (20000, 3, 100),
                                            (60000, 8, 25), (200000, 12, 25)])
@pytest.mark.parametrize("precision", [amfmm.FP64, amfmm.MIXED])
def test_every_request_has_room(n, cells, n_crit, precision, monkeypatch, capfd):
    say("near plan", n, cells, n_crit, precision)
    p = clump(n, cells, seed=n + cells)
    P = to_dev(*p)
    # order 4: its moments keep the dipole that rounding leaves about a centre
    # of mass, here 1e-10 of a cell's size (at order 3 parents leave it out, and
    # the oracle, which sums over particles, does not)
    s = amfmm.Solver(n_crit=n_crit, precision=precision, order=4)
    first = host(s.solve_gravity(*P, 0.5))
    monkeypatch.setenv("AMFMM_DEBUG_NEAR", "1")
    capfd.readouterr()
    for _ in range(4):
        assert np.array_equal(host(s.solve_gravity(*P, 0.5)), first)
    seen = plans(capfd)
    assert len(seen) == 4 and len(set(seen)) == 1
    cut, segments, units, parts, room = seen[0]
    assert 0 < cut <= segments <= units and segments <= parts <= room, seen[0]
    s.close()
    if n > 20000:
        return
    oacc, opot = orc.solve(*p, theta=0.5, n_crit=n_crit, variant=amfmm.TC, order=4)
    i = np.arange(0, n, 37)
    _, _, gabs = orc.direct(*p, i)
    check(first[:, i], np.vstack([oacc, opot[None]])[:, i], gabs, precision)


@pytest.mark.parametrize("variant,order,softening,precision", [
    (amfmm.TC, 3, 0.05, amfmm.FP64), (amfmm.TC, 3, 0.05, amfmm.MIXED), (amfmm.UC, 3, 0.0, amfmm.FP64),
    (amfmm.TCO, 3, 0.0, amfmm.MIXED), (amfmm.TC, 4, 0.0, amfmm.FP64), (amfmm.TC, 4, 0.05, amfmm.MIXED)])
@pytest.mark.parametrize("how", ["solve", "batched", "noalloc"])
def test_cut_lists_in_every_solve(variant, order, softening, precision, how, monkeypatch, capfd):
    if how == "noalloc" and order == 4:
        pytest.skip("the allocation-free solve takes order 3 only")
    say("cut lists", how, variant, order, softening, precision)
    n, n_crit, theta = 16000, 25, 0.4
    p = core_and_halo(n, 25, seed=5)
    P = to_dev(*p)
    s = amfmm.Solver(n_crit=n_crit, variant=variant, order=order, softening=softening, precision=precision,
                     list_bytes=1 << 20 if how == "batched" else 0)
    out = tuple(torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(4))

    def solve():
        if how == "noalloc":
            return host(s.solve_gravity_noalloc(*P, theta, out))
        return host(s.solve_gravity(*P, theta, out=out))

    first = solve()
    assert s.get_counts()["near_launches"] > (1 if how == "batched" else 0)
    monkeypatch.setenv("AMFMM_DEBUG_NEAR", "1")
    capfd.readouterr()
    assert np.array_equal(solve(), first)
    seen = plans(capfd)
    if how != "noalloc":  # (which prints nothing)
        assert any(c[0] > 0 for c in seen) and all(c[1] <= c[2] and c[3] <= c[4] for c in seen), seen
    s.close()
    oacc, opot = orc.solve(*p, theta=theta, n_crit=n_crit, variant=variant, softening=softening, order=order)
    _, _, gabs = orc.direct(*p, softening=softening)
    check(first, np.vstack([oacc, opot[None]]), gabs, precision)


@pytest.mark.parametrize("n,n_crit", [(1, 1), (300, 128), (1000, 64), (4096, 25)])
def test_room_follows_the_problem(n, n_crit, monkeypatch, capfd):
    """A partial sum takes 48 bytes, a segment 40: a few thousand particles do
    not hold tens of megabytes for lists that they cannot have."""
    rng = np.random.default_rng(n)
    P = to_dev(*rng.standard_normal((3, n)), np.full(n, 1.0 / n))
    s = amfmm.Solver(n_crit=n_crit)
    monkeypatch.setenv("AMFMM_DEBUG_NEAR", "1")
    capfd.readouterr()
    s.solve_gravity(*P, 0.5)
    (cut, segments, units, parts, room), = plans(capfd)
    s.close()
    assert segments <= units and parts <= room
    # every list costs less than 0.4 a target and source, a share at least 4000
    most = 1.01 * 0.4 * n * n / 4000
    assert units <= 3 * most + 64 and room <= 1.5 * 64 * most + 64, (units, room)


@pytest.mark.parametrize("order", [3, 4])
def test_one_near_phase_a_batch(order):
    """One near-field phase for the top levels and one a batch of subtrees, where
    the far field takes one for the top and one for each of a batch's levels (two
    at least here)."""
    p = W.plummer(1 << 17, seed=12)
    P = to_dev(*p)
    outs = []
    for list_bytes in (0, 1 << 20):
        s = amfmm.Solver(order=order, list_bytes=list_bytes)
        outs.append(host(s.solve_gravity(*P, 0.7)))
        c = s.get_counts()
        if list_bytes:
            assert c["near_launches"] > 1 and 2 * (c["near_launches"] - 1) <= c["far_launches"] - 1, c
        s.close()
    i = W.sample_targets(1 << 17, 256, seed=99)
    _, _, gabs = orc.direct(*p, i)
    check(outs[1][:, i], outs[0][:, i], gabs, amfmm.FP64)
