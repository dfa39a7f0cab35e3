"""The work that a user of this library has it do, as cases that can be timed.

A pass is one of the library's public calls on device-resident inputs: a step of a simulation
(``Plan.rebuild`` for new positions and ``Plan.execute`` for their masses), an evaluation of new
masses on a tree that stays, a one-shot ``solve``, a batch of independent solves on the serving
runtime, or the direct sum that force errors are measured against. Sizes, distributions, tree
rules and gridlet orders are those of the benchmark and the tests; ``draw`` takes more from the
same ranges.
"""
from __future__ import annotations

import math

import torch

from paper_1906_10734_amd import hpm

SOFTENING = 1e-3   # of the unit box, in every workload of the benchmark
SCREENING = 0.05   # the benchmark's screened kernel


def listed():
    return [
        # one small solve with everything counted: the benchmark's latency workload, where
        # launches and the one host synchronisation of a tree build are the cost
        dict(name="small_uniform_f64", call="step", n=4096, kind="uniform", precision="f64", ng=4,
             route="grid", uniform_depth=3),
        # a script's first call on a small set: plan, tables, tree and evaluation in one call
        dict(name="oneshot_small_f32", call="solve", n=3000, kind="plummer", precision="f32", ng=4,
             route="grid", leaf=16),
        # the benchmark's headline: one step of a 2^18-particle Plummer sphere on the padded grid
        dict(name="plummer_256k_f32", call="step", n=1 << 18, kind="plummer", precision="f32",
             ng=6, route="grid", leaf=64),
        # the same step in double precision
        dict(name="plummer_256k_f64", call="step", n=1 << 18, kind="plummer", precision="f64",
             ng=6, route="grid", leaf=64),
        # the same set on the route that the autotuner picks for it
        dict(name="plummer_256k_f32_shared", call="step", n=1 << 18, kind="plummer",
             precision="f32", ng=6, route="shared", leaf=64),
        # new masses on a tree that stays (an iterative solver's matrix-vector product), odd size
        dict(name="masses_150k_f64_cells", call="masses", n=150001, kind="plummer",
             precision="f64", ng=6, route="cells", leaf=64),
        # the largest requests of the served stream: clustered sets at a 1e-4 force tolerance,
        # which the server answers with extended gridlets on the cell route
        dict(name="served_1m_f32_extended", call="step", n=1000003, kind="clustered",
             precision="f32", ng=6, route="cells", leaf=64, extended=True),
        # the largest single solve of the benchmark: 2^24 clustered particles, low order, on its
        # fastest route
        dict(name="clustered_16m_f32", call="step", n=1 << 24, kind="clustered", precision="f32",
             ng=4, route="cells", leaf=32),
        # the screened interaction (plasmas, modified gravity), ragged size
        dict(name="screened_100k_f32", call="step", n=100003, kind="plummer", precision="f32",
             ng=6, route="grid", leaf=64, kernel="yukawa"),
        # high accuracy: the highest gridlet order in double, on the largest set that it takes
        dict(name="accurate_64k_f64", call="step", n=1 << 16, kind="plummer", precision="f64",
             ng=8, route="grid", leaf=64),
        # many independent solves in one call of the serving runtime, sizes from 2^10 to 2^18
        dict(name="batch_32_f32", call="batch", count=32, lo=1 << 10, hi=1 << 18, precision="f32",
             route="shared", leaf=64),
        # the force-error reference: a direct sum at 4096 of 2^18 particles
        dict(name="direct_4k_of_256k", call="direct", n=1 << 18, targets=4096, kind="plummer",
             precision="f64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))


def draw(rng):
    """A case of the same ranges: particle counts log-uniform over the sizes that the benchmark
    and the served stream use, every route, precision, distribution and gridlet order of theirs."""
    call = rng.choice(["step", "step", "step", "step", "masses", "masses", "solve", "batch",
                       "direct"])
    precision = rng.choice(["f32", "f32", "f64"])
    kind = rng.choice(["uniform", "plummer", "clustered"])
    if call == "direct":
        n = _log_int(rng, 1 << 12, 1 << 20)
        return dict(call=call, n=n, targets=min(n, _log_int(rng, 64, 4096)), kind=kind,
                    precision=precision)
    if call == "batch":
        lo = _log_int(rng, 1 << 10, 1 << 13)
        return dict(call=call, count=rng.randint(4, 32), lo=lo, hi=lo * rng.choice([4, 16, 32]),
                    precision=precision, route=rng.choice(["grid", "cells", "shared"]),
                    leaf=rng.choice([32, 64]))
    ng = rng.choice([4, 6, 4, 6, 4, 6, 8])
    case = dict(call=call, kind=kind, precision=precision, ng=ng)
    if ng == 8:
        case.update(n=_log_int(rng, 1 << 10, 1 << 16), route="grid", leaf=64)
    else:
        leaf = rng.choice([16, 32, 64])  # the cells, and so the cost, grow as n / leaf
        hi = 1 << 16 if call == "solve" else (1 << 20) * leaf // 64
        case.update(n=_log_int(rng, 1 << 10, hi), route=rng.choice(["grid", "cells", "shared"]),
                    leaf=leaf)
        if case["route"] != "shared" and rng.random() < 0.3:
            case["extended"] = True
    if kind == "uniform" and rng.random() < 0.3:
        # a uniform tree of about 16 to 128 particles per leaf
        case.pop("leaf")
        case["uniform_depth"] = max(2, min(5, int(math.log(case["n"] / 16.0, 8))))
    if rng.random() < 0.2:
        case["kernel"] = "yukawa"
    if precision == "f32" and ng in (4, 6) and case["route"] == "grid" and rng.random() < 0.2 \
            and call != "solve":
        case["strict"] = True
    return case


# ---- inputs ---------------------------------------------------------------------------------
def _plummer_offsets(gen, scale, r_t=0.5):
    """Offsets from the centre of Plummer spheres truncated at r_t, one per element of scale."""
    n = scale.numel()
    u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    u = (u * (r_t * r_t / (r_t * r_t + scale * scale)) ** 1.5).clamp_min(1e-300)
    r = scale / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
    mu = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * 2.0 - 1.0
    ph = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * (2.0 * math.pi)
    s = torch.sqrt((1.0 - mu * mu).clamp_min(0.0))
    return torch.stack([r * s * torch.cos(ph), r * s * torch.sin(ph), r * mu], 1)


def _positions(kind, n, gen):
    """(n, 3) positions in the unit box in float64: a uniform cube, a Plummer sphere of scale 0.05
    in its middle, or 8 spheres (32 from 2^22 particles on) on a 10% uniform background."""
    if kind == "uniform":
        return torch.rand(n, 3, generator=gen, device="cuda", dtype=torch.float64)
    if kind == "plummer":
        a = torch.full((n,), 0.05, device="cuda", dtype=torch.float64)
        return (_plummer_offsets(gen, a) + 0.5).clamp(0.0, math.nextafter(1.0, 0.0))
    k = 32 if n >= 1 << 22 else 8
    a_k = torch.rand(k, generator=gen, device="cuda", dtype=torch.float64)
    a_k = torch.exp(math.log(0.005) + a_k * math.log(10.0))
    c_k = torch.rand(k, 3, generator=gen, device="cuda", dtype=torch.float64)
    w_k = torch.exp(torch.rand(k, generator=gen, device="cuda", dtype=torch.float64) * math.log(10.0))
    pos = torch.rand(n, 3, generator=gen, device="cuda", dtype=torch.float64)
    edges = torch.cumsum(w_k, 0) / w_k.sum()
    pick = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    sphere = torch.searchsorted(edges, pick).clamp_max(k - 1)
    todo = torch.arange(n // 10, n, device="cuda")  # the first tenth stays uniform
    while todo.numel():  # samples outside the box are drawn again
        p = _plummer_offsets(gen, a_k[sphere[todo]]) + c_k[sphere[todo]]
        pos[todo] = p
        todo = todo[((p < 0.0) | (p >= 1.0)).any(1)]
    return pos[torch.randperm(n, generator=gen, device="cuda")].contiguous()


def _particles(kind, n, precision, gen, masses="equal"):
    dt = torch.float32 if precision == "f32" else torch.float64
    pos = _positions(kind, n, gen)
    x, y, z = (pos[:, k].to(dt).contiguous() for k in range(3))
    if masses == "equal":
        m = torch.full((n,), 1.0 / n, device="cuda", dtype=dt)
    else:
        m = ((torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) + 0.5) / n).to(dt)
    return x, y, z, m


def _problem(case, ng):
    tree = dict(uniform_depth=case["uniform_depth"]) if case.get("uniform_depth") else \
        dict(leaf_capacity=case["leaf"], max_depth=10)
    kernel = case.get("kernel", "newton")
    return hpm.Problem(ng=ng, precision=case["precision"], softening=SOFTENING, m2l=case["route"],
                       extended=bool(case.get("extended")), kernel=kernel,
                       screening=SCREENING if kernel == "yukawa" else 0.0, **tree)


def _batch(case):
    """(particles, kind, gridlet order) of each solve: sizes log-uniform from lo to hi, uniform
    cubes and Plummer spheres in turn, orders 4 and 6."""
    k = case["count"]
    sizes = [int(round(case["lo"] * (case["hi"] / case["lo"]) ** ((i + 0.5) / k))) for i in range(k)]
    return [(n, "uniform" if i % 2 == 0 else "plummer", 4 if i % 4 < 2 else 6)
            for i, n in enumerate(sizes)]


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["call"] == "batch":
        return [_particles(kind, n, case["precision"], gen) for n, kind, _ in _batch(case)]
    masses = "random" if case["call"] == "masses" else "equal"
    return _particles(case["kind"], case["n"], case["precision"], gen, masses)


def _targets(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1)
    pick = torch.randperm(case["n"], generator=gen, device="cuda")[:case["targets"]]
    return pick.to(torch.int32).contiguous()


def prepare(case, seed):
    inputs = _inputs(case, seed)
    state = dict(call=case["call"], inputs=inputs)
    if case["call"] == "direct":
        state["targets"] = _targets(case, seed)
        return state
    dt = torch.float32 if case["precision"] == "f32" else torch.float64
    if case["call"] == "batch":
        total = sum(p[0].numel() for p in inputs)
        out = [torch.empty(total, dtype=dt, device="cuda") for _ in range(4)]
        at = [0]
        for p in inputs:
            at.append(at[-1] + p[0].numel())
        state.update(server=hpm.Server(slots=8, hbm_budget=64 << 30), out=out,
                     problems=[_problem(case, ng) for _, _, ng in _batch(case)],
                     parts=[tuple(o[a:b] for o in out) for a, b in zip(at, at[1:])])
        return state
    problem = _problem(case, case["ng"])
    if case["call"] == "solve":
        state["problem"] = problem
        return state
    x, y, z, _ = inputs
    plan = hpm.Plan(problem, x, y, z)
    if case.get("strict"):
        plan.set_fp32_strict(True)
    state.update(plan=plan, out=[torch.empty_like(x) for _ in range(4)])
    return state


def run(state):
    call = state["call"]
    if call == "batch":
        status, _ = state["server"].run_batch(state["problems"], state["inputs"], state["parts"])
        if any(s != "HPM_OK" for s in status):
            raise RuntimeError("a solve of the batch failed: " + ", ".join(status))
        return state["out"]
    x, y, z, m = state["inputs"]
    if call == "direct":
        return hpm.direct_sum(x, y, z, m, state["targets"], softening=SOFTENING)
    if call == "solve":
        return hpm.solve(state["problem"], x, y, z, m)
    if call == "step":
        state["plan"].rebuild(x, y, z)
    state["plan"].execute(m, *state["out"])
    return state["out"]


# ---- what a pass cannot do without ------------------------------------------------------------
def _solve_flops(n, ng, extended, leaf=0, uniform_depth=0):
    """Near-zone pairs at 20 operations, and the interaction zones as one pointwise complex
    product per cell pair (189 per target, C^2 (C/2 + 1) modes, C = 2 N_g or 2 N_g + 2): the
    fewest operations that a transform-based step is known to need. Adaptive trees have about
    4 n / leaf targets and 15 n leaf near pairs on the benchmark's sets."""
    c = 2 * ng + (2 if extended else 0)
    product = 189 * 8.0 * c * c * (c // 2 + 1)
    if uniform_depth:
        leaves = 8.0 ** uniform_depth
        return 20.0 * 27.0 * n * n / leaves + product * min(leaves, n) * 8.0 / 7.0
    return 20.0 * 15.0 * n * min(leaf, n) + product * 4.0 * n / leaf


def work(case):
    elem = 4 if case["precision"] == "f32" else 8
    if case["call"] == "direct":
        t = case["targets"]
        return {"bytes": 4.0 * case["n"] * elem + t * (4.0 + 4 * 8), "flops": 20.0 * case["n"] * t}
    if case["call"] == "batch":
        solves = _batch(case)
        return {"bytes": 8.0 * elem * sum(n for n, _, _ in solves),
                "flops": sum(_solve_flops(n, ng, False, case["leaf"]) for n, _, ng in solves)}
    return {"bytes": 8.0 * elem * case["n"],
            "flops": _solve_flops(case["n"], case["ng"], case.get("extended"), case.get("leaf", 0),
                                  case.get("uniform_depth", 0))}


# ---- the same in plain torch, 64 bits -----------------------------------------------------------
MOST_PAIRS = 2.1e11


def _direct(x, y, z, m, kernel, targets=None):
    """Potential and acceleration of every particle (or the targets) by summing every pair."""
    x, y, z, m = (v.double() for v in (x, y, z, m))
    n = x.numel()
    at = torch.arange(n, device="cuda") if targets is None else targets.long()
    out = [torch.empty(at.numel(), dtype=torch.float64, device="cuda") for _ in range(4)]
    rows = max(1, (1 << 26) // n)
    for a in range(0, at.numel(), rows):
        t = at[a:a + rows]
        d = [v[t][:, None] - v[None, :] for v in (x, y, z)]
        s = d[0] * d[0]
        s.addcmul_(d[1], d[1]).addcmul_(d[2], d[2]).add_(SOFTENING * SOFTENING)
        inv = s.rsqrt_()
        inv[torch.arange(t.numel(), device="cuda"), t] = 0.0  # no particle acts on itself
        if kernel == "yukawa":  # exp(-s/l)/s and exp(-s/l) (1/s^3 + 1/(l s^2))
            w = torch.exp(-1.0 / (inv * SCREENING)) * inv
            c = w * (inv * inv + inv / SCREENING)
        else:
            w, c = inv, inv * inv * inv
        out[0][a:a + rows] = -(w @ m)
        for k in range(3):
            out[1 + k][a:a + rows] = -(d[k].mul_(c) @ m)
    return out


def exact(case, seed):
    """The sums that every solve stands for, pair by pair; None above about 20 seconds of them."""
    if case["call"] == "batch":
        pairs = sum(float(n) * n for n, _, _ in _batch(case))
    else:
        pairs = float(case["n"]) * (case["targets"] if case["call"] == "direct" else case["n"])
    if pairs > MOST_PAIRS:
        return None
    inputs = _inputs(case, seed)
    if case["call"] == "batch":
        parts = [_direct(*p, "newton") for p in inputs]
        return [torch.cat([p[k] for p in parts]) for k in range(4)]
    if case["call"] == "direct":
        return tuple(_direct(*inputs, "newton", _targets(case, seed)))
    return _direct(*inputs, case.get("kernel", "newton"))
