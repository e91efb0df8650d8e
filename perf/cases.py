"""Performance cases: the work a user of the library has it do, through its
public entry points (``paper_1706_06989_amd.amfmm.Solver``).

``listed()`` names twelve cases, ``draw(rng)`` gives more of the same ranges.
A case is a dict of plain values: ``kind`` (which calls are made), the particle
set (``shape``, ``n``) and the solver's options.  ``prepare`` puts the inputs
on the GPU and makes the solver a program keeps, ``run`` makes one pass,
``work`` is what the path cannot do without and ``exact`` is the same result
in plain float64 (direct summation) at the sizes where that takes seconds.
"""
import math
import weakref

import numpy as np
import torch

from paper_1706_06989_amd import amfmm
from paper_1706_06989_amd import learned
from paper_1706_06989_amd import workloads as W

VARIANTS = {"UC": amfmm.UC, "TC": amfmm.TC, "TCO": amfmm.TCO}
PRECISIONS = {"fp64": amfmm.FP64, "mixed": amfmm.MIXED}
SHAPES = {"uniform": W.uniform_cube, "plummer": W.plummer, "two_plummer": W.two_plummer}

# the benchmark's pilot solve and error tolerances (order 3, order 4)
PILOT = dict(variant=amfmm.UC, precision=amfmm.MIXED, n_crit=128)
PILOT_THETA = 1.0
EPS = {3: 9e-8, 4: 1.75e-5}
NCRIT = {3: 25, 4: 64}
TRAIN_ROWS = 120000  # pairs of the learned criterion's training set


def _solve(name, n, shape="plummer", theta=0.5, variant="TC", precision="fp64", n_crit=25, softening=0.0,
           kind="solve"):
    return dict(name=name, kind=kind, n=n, shape=shape, theta=theta, variant=variant, precision=precision,
                n_crit=n_crit, softening=softening)


def listed():
    return [
        # the smallest everyday call: the 4096-particle cube with the solver's
        # defaults, where launches and read-backs are the time
        _solve("solve_uniform_4096", 4096, shape="uniform"),
        # a run in time: the two-sphere binary of the angular-momentum study,
        # eight leapfrog steps a call
        dict(name="leapfrog_binary_65536", kind="leapfrog", n=65536, theta=0.5, variant="TC", precision="fp64",
             dt=0.02, steps=8),
        # an ordinary solve at an odd size
        _solve("solve_plummer_100003", 100003),
        # the million-particle Plummer sphere at the paper's settings
        _solve("solve_plummer_1m", 1 << 20),
        # the paper's accuracy sweep over opening angles on two spheres
        _solve("sweep_two_plummer_4m", 1 << 22, shape="two_plummer", theta=0.35),
        # softened N-body production: mixed precision, odd size
        _solve("softened_mixed_300007", 300007, theta=0.6, precision="mixed", softening=0.01),
        # callers that cannot allocate, with the alternative correction
        _solve("noalloc_tco_50021", 50021, theta=0.7, variant="TCO", kind="noalloc"),
        # a force step at a p99 error of 1e-4 (pilot solve for the field
        # scale, then the multipole criterion): a quarter million particles
        dict(name="step_plummer_256k", kind="step", n=1 << 18, shape="plummer", order=3),
        # the benchmark: the same step at 16.8 million
        dict(name="step_plummer_16m", kind="step", n=1 << 24, shape="plummer", order=3),
        # the same accuracy through the order-4 expansion
        dict(name="step_order4_4m", kind="step", n=1 << 22, shape="plummer", order=4),
        # error truth: direct sums at sampled targets
        dict(name="direct_4096_of_1m", kind="direct", n=1 << 20, targets=4096),
        # training of the learned criterion: Adam steps on batches of 4096
        dict(name="train_batch_4096", kind="train", batch=4096, steps=50),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["step"] * 3 + ["noalloc", "leapfrog", "direct", "train"])
    if kind in ("solve", "noalloc"):
        n = _log_int(rng, 1000, 4000000 if kind == "solve" else 150000)
        c = _solve("", n, shape=rng.choice(sorted(SHAPES)),
                   theta=round(rng.uniform(0.5 if kind == "noalloc" else 0.3 if n < 1000000 else 0.4, 1.0), 2),
                   variant=rng.choice(["UC", "TC", "TC", "TC", "TCO"]), precision=rng.choice(["fp64", "fp64", "mixed"]),
                   n_crit=rng.choice([16, 25, 25, 25, 64, 128]), softening=rng.choice([0.0, 0.0, 0.0, 0.01, 0.05]),
                   kind=kind)
        del c["name"]
        return c
    if kind == "step":
        order = rng.choice([3, 3, 4])
        return dict(kind="step", n=_log_int(rng, 20000, 2500000 if order == 3 else 8000000),
                    shape=rng.choice(["plummer", "two_plummer"]), order=order)
    if kind == "leapfrog":
        return dict(kind="leapfrog", n=_log_int(rng, 4096, 150000), theta=round(rng.uniform(0.4, 0.8), 2),
                    variant=rng.choice(["UC", "TC", "TC"]), precision="fp64", dt=0.02, steps=rng.randint(1, 8))
    if kind == "direct":
        n = _log_int(rng, 4096, 2000000)
        return dict(kind="direct", n=n, targets=min(n, _log_int(rng, 256, 16384)))
    return dict(kind="train", batch=_log_int(rng, 256, 16384), steps=rng.randint(10, 50))


# One solver per set of options while any state of it is alive: a program
# keeps its solver and hands it new particles.
_solvers = weakref.WeakValueDictionary()


def _solver(**options):
    key = tuple(sorted(options.items()))
    s = _solvers.get(key)
    if s is None:
        s = _solvers[key] = amfmm.Solver(**options)
    return s


def _options(case):
    o = dict(variant=VARIANTS[case["variant"]], precision=PRECISIONS[case["precision"]])
    if case["kind"] in ("solve", "noalloc"):
        o.update(n_crit=case["n_crit"], softening=case["softening"])
    return o


def _cuda(arrays):
    return [torch.from_numpy(np.ascontiguousarray(a, np.float64)).cuda() for a in arrays]


def _targets(case, seed):
    return torch.from_numpy(W.sample_targets(case["n"], case["targets"], seed=seed)).cuda()


def _training_set(seed):
    """Rows like the ones learned.collect draws from far-field lists: the eight
    features in their ranges, labels near the multipole estimate."""
    rng = np.random.default_rng(seed)
    u = rng.random((TRAIN_ROWS, 8))
    f = np.empty((TRAIN_ROWS, 8), np.float32)
    f[:, 0] = 0.08 + 0.42 * u[:, 0] ** 2  # (R_A + R_B) / d
    f[:, 1] = u[:, 1]  # |R_A - R_B| / (R_A + R_B)
    for i in (2, 3, 4, 5):  # traceless norm levels, held to 1/256 and 1/128
        f[:, i] = np.floor(64.0 * u[:, i] ** 2) / 128.0
    f[:, 6] = u[:, 6]  # |M_A - M_B| / (M_A + M_B)
    f[:, 7] = 10.0 + 10.0 * u[:, 7]  # plog2 of N_A N_B
    lab = 0.6 * f[:, 0] - 0.4 * f[:, 1] + f[:, 3] + 0.35 * rng.standard_normal(TRAIN_ROWS)
    return f, lab.astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        f, lab = _training_set(seed)
        P = torch.from_numpy(learned.init_model(f, seed)).cuda()
        m = torch.zeros(amfmm.MLP_PARAMS, dtype=torch.float32, device="cuda")
        return dict(case=case, s=_solver(), feats=torch.from_numpy(f).cuda(), labels=torch.from_numpy(lab).cuda(),
                    model=P, m=m, v=torch.zeros_like(m), step=0)
    n = case["n"]
    st = dict(case=case)
    if kind == "leapfrog":
        *p, vx, vy, vz = W.two_plummer_binary(n, seed=seed)
        st["p"] = _cuda(p)
        st["v"] = _cuda((vx, vy, vz))
        st["s"] = _solver(**_options(case))
        st["acc"] = st["s"].solve_gravity(*st["p"], case["theta"], pot=False)[:3]
        return st
    if kind == "direct":
        st.update(p=_cuda(W.plummer(n, seed=seed)), t=_targets(case, seed), s=_solver())
        return st
    st["p"] = _cuda(SHAPES[case["shape"]](n, seed=seed))
    st["out"] = tuple(torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(4))
    if kind == "step":
        order = case["order"]
        st["pilot"] = _solver(**PILOT)
        st["pilot_out"] = tuple(torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(3)) + (None,)
        st["s"] = _solver(precision=amfmm.MIXED, criterion=amfmm.MULTIPOLE, error_tol=EPS[order], theta_max=0.5,
                          order=order, n_crit=NCRIT[order])
    else:
        st["s"] = _solver(**_options(case))
    return st


def run(st):
    case, s = st["case"], st["s"]
    kind = case["kind"]
    if kind == "solve":
        return s.solve_gravity(*st["p"], case["theta"], out=st["out"])
    if kind == "noalloc":
        return s.solve_gravity_noalloc(*st["p"], case["theta"], st["out"])
    if kind == "step":
        g = st["pilot"].solve_gravity(*st["p"], PILOT_THETA, out=st["pilot_out"])
        s.set_field_estimate(*g[:3])
        return s.solve_gravity(*st["p"], 0.5, out=st["out"])
    if kind == "leapfrog":
        x, y, z, m = st["p"]
        s.leapfrog(x, y, z, *st["v"], m, case["theta"], case["dt"], case["steps"], st["acc"])
        return [x, y, z, *st["v"], *st["acc"]]
    if kind == "direct":
        return s.direct(*st["p"], st["t"])
    loss = s.mlp_train(st["feats"], st["labels"], st["model"], st["m"], st["v"], st["step"], case["steps"],
                       case["batch"], 2e-3)
    st["step"] += case["steps"]
    return dict(model=st["model"], m=st["m"], v=st["v"], loss=loss)


# Interactions per particle the method makes (measured on these particle sets):
# near-field particle pairs and far-field cell pairs, both directed.
def _interactions(case):
    n, kind = case["n"], case["kind"]
    if kind == "step":
        # over log2 n at the benchmark's tolerances
        at = (18.0, 20.0, 22.0, 24.0)
        near = {3: (78670.0, 40014.0, 22597.0, 19312.0), 4: (9093.0, 6200.0, 4235.0, 2983.0)}[case["order"]]
        far = {3: (1694.0, 2361.0, 1713.0, 1075.0), 4: (88.0, 56.0, 36.0, 30.0)}[case["order"]]
        return (min(n, float(np.interp(math.log2(n), at, near))), float(np.interp(math.log2(n), at, far)))
    t = 0.5 / case["theta"]
    size = case.get("n_crit", 25) / 25.0
    near, far = (450.0, 30.0) if case.get("shape") == "uniform" else (1000.0, 47.0)
    return min(n, near * t**3.3 * size), min(0.15 * n, far * t**2.8) / size


def work(case):
    kind = case["kind"]
    if kind == "train":
        # forward and two backward products of 8 -> 64 -> 64 -> 1, Adam's state
        return dict(bytes=case["steps"] * (36.0 * case["batch"] + 28.0 * amfmm.MLP_PARAMS),
                    flops=case["steps"] * case["batch"] * 6.0 * amfmm.MLP_PARAMS)
    n = case["n"]
    if kind == "direct":
        return dict(bytes=32.0 * n + 48.0 * case["targets"], flops=22.0 * n * case["targets"])
    near, far = _interactions(case)
    # 20 flop a particle interaction; an unordered cell pair 357 flop at order
    # 3 (derivatives once, both cells' coefficients, the correction once), 900
    # at order 4
    flops = n * (20.0 * near + (450.0 if case.get("order") == 4 else 178.5) * far)
    moved = 64.0 * n  # x, y, z, m in, three components and the potential out
    if kind == "step":
        flops += n * 20.0 * 300.0  # the pilot's near field
        moved += 80.0 * n  # its pass over the particles, its field out and in
    if kind == "leapfrog":
        flops *= case["steps"]
        moved = case["steps"] * n * (32.0 + 24.0) + 2 * n * 72.0
    return dict(bytes=moved, flops=flops)


def _direct64(x, y, z, m, softening=0.0, targets=None):
    """Plain float64 direct sums at all particles (or the targets): ax, ay, az,
    potential and sum m / r^2; pairs at r = 0 are skipped."""
    n = x.numel()
    t = torch.arange(n, device=x.device) if targets is None else targets
    outs = [torch.empty(t.numel(), dtype=torch.float64, device=x.device) for _ in range(5)]
    rows = max(1, (1 << 27) // n)
    for a in range(0, t.numel(), rows):
        i = t[a:a + rows]
        dx, dy, dz = (q[None, :] - q[i][:, None] for q in (x, y, z))
        r2 = dx * dx + dy * dy + dz * dz
        w = torch.where(r2 > 0, (r2 + softening * softening).rsqrt(), 0.0)
        del r2
        mw = m[None, :] * w
        outs[3][a:a + rows] = -mw.sum(1)
        mw *= w
        outs[4][a:a + rows] = mw.sum(1)
        mw *= w
        for o, d in zip(outs, (dx, dy, dz)):
            o[a:a + rows] = (mw * d).sum(1)
    return outs


def _train64(case, seed):
    """The training steps in float64, weights, inputs and hidden activations
    rounded to BF16 where the model defines it."""
    f, lab = _training_set(seed)
    P = torch.from_numpy(learned.init_model(f, seed)).cuda().double()
    f, lab = torch.from_numpy(f).cuda().double(), torch.from_numpy(lab).cuda().double()
    b16 = lambda v: v.bfloat16().double()  # noqa: E731
    m = torch.zeros(amfmm.MLP_PARAMS, dtype=torch.float64, device="cuda")
    v, B, tau = torch.zeros_like(m), case["batch"], learned.TAU
    for s in range(case["steps"]):
        rows = (s * B + torch.arange(B, device="cuda")) % len(lab)
        X = b16(f[rows] * P[4801:4809] + P[4809:4817])
        W1, b1, W2, b2 = b16(P[:512]).view(64, 8), P[512:576], b16(P[576:4672]).view(64, 64), P[4672:4736]
        w3, b3 = b16(P[4736:4800]), P[4800]
        H1 = b16((X @ W1.T + b1).clamp(min=0))
        H2 = b16((H1 @ W2.T + b2).clamp(min=0))
        res = lab[rows] - (H2 @ w3 + b3)
        loss = torch.where(res < 0, (tau - 1) * res, tau * res).mean()
        dy = torch.where(res < 0, 1 - tau, -tau).double() / B
        d2 = (dy[:, None] * w3) * (H2 > 0)
        d1 = (d2 @ W2) * (H1 > 0)
        g = torch.cat([(d1.T @ X).flatten(), d1.sum(0), (d2.T @ H1).flatten(), d2.sum(0), dy @ H2, dy.sum()[None]])
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        P[:amfmm.MLP_PARAMS] -= 2e-3 * (m / (1 - 0.9 ** (s + 1))) / ((v / (1 - 0.999 ** (s + 1))).sqrt() + 1e-8)
    return dict(model=P, m=m, v=v, loss=float(loss))


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _train64(case, seed)
    n = case["n"]
    if kind == "direct":
        p = _cuda(W.plummer(n, seed=seed))
        return _direct64(*p, targets=_targets(case, seed)) if n * case["targets"] < 4e10 else None
    if kind == "leapfrog":
        if n * n * (case["steps"] + 1) > 6e10:
            return None
        *p, vx, vy, vz = W.two_plummer_binary(n, seed=seed)
        x, v = _cuda(p), _cuda((vx, vy, vz))
        acc = _direct64(*x)
        for _ in range(case["steps"]):
            for k in range(3):
                v[k] += 0.5 * case["dt"] * acc[k]
                x[k] += case["dt"] * v[k]
            acc = _direct64(*x)
            for k in range(3):
                v[k] += 0.5 * case["dt"] * acc[k]
        return [*x[:3], *v, *acc[:3]]
    if n * n > 8e10:
        return None  # direct sums would take minutes
    return _direct64(*_cuda(SHAPES[case["shape"]](n, seed=seed)), softening=case.get("softening", 0.0))[:4]
