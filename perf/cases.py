"""The work that users of this library have it do, as measurable cases.

Every case goes through the public entry points of ``paper_1405_2255_amd.fmm``
on particle sets from ``paper_1405_2255_amd.workloads``:

listed()            the cases
draw(rng)           one more case of the same ranges
prepare(case, seed) the inputs on the GPU and the context a program keeps
run(state)          one pass
work(case)          bytes and operations one pass cannot do without
exact(case, seed)   the outputs by plain FP64 sums in torch
"""
import math

import numpy as np
import torch

from paper_1405_2255_amd import fmm, workloads

DEV = "cuda:0"

# the fields a case may leave out
DEFAULTS = {"profile": "plummer", "masses": "equal", "eps": 1e-7, "p": -1, "leaf": 0,
            "factor": 0.0, "centre": "auto", "precision": "fp64", "mac": "a", "sinks": 0,
            "clusters": 0, "size_seed": 0, "lo": 1000, "hi": 100000}


def listed():
    return [
        # the smallest evaluation an N-body program makes each step: a few
        # thousand bodies with the library's defaults; launches and
        # synchronisations count, not arithmetic
        {"name": "forces_2e3", "call": "forces", "n": 2000, "eps": 1e-7},
        # the paper's table of costs (criterion f, p = 10, eps = 10^-6.25) at its
        # smallest size
        {"name": "forces_f_1e4", "call": "forces", "n": 10000, "mac": "f", "p": 10,
         "eps": 10.0 ** -6.25},
        # an ordinary cluster with the defaults, an odd size
        {"name": "forces_1e5", "call": "forces", "n": 100003, "eps": 1e-7},
        # the headline workload: 10^6 equal-mass Plummer particles, rms 1e-7, FP64,
        # the committed tuned parameters
        {"name": "forces_1e6", "call": "forces", "n": 1000000, "p": 15, "eps": 6e-8, "leaf": 80,
         "factor": 2.0, "centre": "midpoint"},
        # a cuspy galaxy with a mass spectrum in mixed precision, a deep tree
        {"name": "mixed_cusp_1e6", "call": "forces", "profile": "dehnen1", "masses": "salpeter",
         "n": 1000000, "eps": 5e-8, "precision": "mixed"},
        # a drift step of a served request: tree and previous |a| recycled, mixed
        # precision, target 1e-6
        {"name": "refit_mixed_3e5", "call": "refit", "profile": "dehnen1.5", "n": 300007,
         "eps": 5e-7, "precision": "mixed"},
        # block time steps: the innermost 10^4 of 10^6 on the recycled tree
        {"name": "active_1e6", "call": "active", "n": 1000000, "sinks": 10000, "p": 15,
         "eps": 6e-8, "leaf": 80, "factor": 2.0, "centre": "midpoint"},
        # a shared step of a Hermite integrator: forces and jerks
        {"name": "jerk_2e5", "call": "jerk", "n": 200003, "p": 15, "eps": 6e-8, "leaf": 80,
         "factor": 2.0, "centre": "midpoint"},
        # individual accuracies: the inner tenth at 1e-7, the rest at 1e-5
        {"name": "eps_2e5", "call": "eps", "profile": "dehnen0", "masses": "salpeter",
         "n": 200000, "eps": 1e-7},
        # many independent clusters in one call, sizes log-uniform in [1e3, 1e5], tuned
        {"name": "batched_64", "call": "batched", "clusters": 64, "size_seed": 78, "n": 0,
         "p": 14, "eps": 9e-8, "leaf": 96, "factor": 1.0, "centre": "enclosing"},
        # exact forces of a small system (integrators without a tree, references)
        {"name": "direct_3e4", "call": "direct", "n": 30011, "profile": "uniform",
         "masses": "salpeter"},
        # exact forces of sampled sinks: the accuracy check of a large run
        {"name": "direct_sinks_1e6", "call": "direct_sinks", "n": 1000000, "sinks": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(10.0 ** rng.uniform(math.log10(lo), math.log10(hi))))


def draw(rng):
    call = rng.choice(["forces", "forces", "forces", "refit", "active", "jerk", "eps", "batched",
                       "direct", "direct_sinks"])
    profile = rng.choice(["plummer", "plummer", "dehnen0", "dehnen1", "dehnen1.5", "uniform"])
    case = {"call": call, "profile": profile, "masses": rng.choice(["equal", "salpeter"])}
    if call == "direct":
        case["n"] = _log_int(rng, 500, 100000)
        return case
    if call == "direct_sinks":
        case["n"] = _log_int(rng, 5000, 1000000)
        case["sinks"] = min(case["n"], _log_int(rng, 64, 16384))
        return case
    case["eps"] = float("%.3g" % 10.0 ** rng.uniform(math.log10(6e-8), -5.0))
    case["leaf"] = rng.choice([0, 0, 16, 48, 80, 96])
    case["factor"] = rng.choice([0.0, 1.0, 2.0])
    case["centre"] = rng.choice(["auto", "midpoint", "enclosing"])
    if call in ("forces", "refit", "active", "batched"):
        case["precision"] = rng.choice(["fp64", "fp64", "mixed"])
    if call in ("forces", "eps", "jerk"):
        case["mac"] = rng.choice(["a", "a", "a", "f"])
    if call == "batched":
        case["clusters"] = rng.randint(2, 96)
        case["size_seed"] = rng.randrange(1 << 20)
        case["lo"], case["hi"] = 100, _log_int(rng, 2000, 40000)
        case["n"] = 0
        return case
    case["n"] = _log_int(rng, 500, 300000 if call in ("jerk", "eps") else 500000)
    if call == "active":
        case["sinks"] = max(1, int(case["n"] * 10.0 ** rng.uniform(-3.0, -0.3)))
    return case


def _sizes(c):
    return workloads.log_uniform_sizes(c["clusters"], c["size_seed"], c["lo"], c["hi"])


def _inputs(c, seed):
    """The particle arrays of a case (float64 CUDA tensors), from the seed alone."""
    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)

    if c["call"] == "batched":
        sizes = _sizes(c)
        parts = [workloads.cluster(c["profile"], int(s), seed + 131 * i, masses=c["masses"])
                 for i, s in enumerate(sizes)]
        return {"offsets": np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64),
                "pos": dev(np.concatenate([q[0] for q in parts])),
                "mass": dev(np.concatenate([q[1] for q in parts]))}
    n = c["n"]
    pos, mass = workloads.cluster(c["profile"], n, seed, masses=c["masses"])
    d = {"pos": dev(pos), "mass": dev(mass)}
    r = np.sqrt(np.einsum("ij,ij->i", pos, pos))
    if c["call"] in ("refit", "active"):
        d["start"] = d["pos"]
        vel = workloads.drift_velocities(c["profile"], pos, seed + 17)
        d["pos"] = dev(pos + 1e-3 * vel)
    if c["call"] == "jerk":
        d["vel"] = dev(workloads.drift_velocities(c["profile"], pos, seed + 17))
    if c["call"] == "eps":
        inner = r <= np.quantile(r, 0.1)
        d["eps"] = dev(np.where(inner, c["eps"], max(c["eps"], 1e-5)))
    if c["call"] == "active":     # the innermost particles, as block time steps take them
        d["sinks"] = dev(np.argsort(r, kind="stable")[:c["sinks"]].astype(np.int64))
    if c["call"] == "direct_sinks":
        pick = np.random.default_rng(seed + 29).choice(n, c["sinks"], replace=False)
        d["sinks"] = dev(np.sort(pick).astype(np.int64))
    return d


def prepare(case, seed):
    c = {**DEFAULTS, **case}
    d = _inputs(c, seed)
    recycled = c["call"] in ("refit", "active")
    d["ctx"] = fmm.Context(device=0, leaf_size=c["leaf"], p2p_factor=c["factor"], mac=c["mac"],
                           precision=c["precision"], centre=c["centre"],
                           scale_source="previous" if recycled else "estimate")
    d["case"] = c
    if recycled:      # the step before: a full evaluation that builds the tree
        d["ctx"].forces(d.pop("start"), d["mass"], 1.0, c["p"], c["eps"])
    return d


def run(state):
    c, ctx = state["case"], state["ctx"]
    pos, mass, p, eps = state["pos"], state["mass"], c["p"], c["eps"]
    call = c["call"]
    if call == "forces":
        return ctx.forces(pos, mass, 1.0, p, eps)
    if call == "refit":
        return ctx.forces(pos, mass, 1.0, p, eps, refit=True)
    if call == "active":
        return ctx.forces_active(pos, mass, state["sinks"], 1.0, p, eps, refit=True)
    if call == "jerk":
        return ctx.forces_jerk(pos, state["vel"], mass, 1.0, p, eps)
    if call == "eps":
        return ctx.forces_eps(pos, mass, state["eps"], 1.0, p)
    if call == "batched":
        return ctx.forces_batched(state["offsets"], pos, mass, 1.0, p, eps)
    if call == "direct":
        return ctx.direct(pos, mass)
    return ctx.direct_sinks(pos, mass, state["sinks"])


def work(case):
    c = {**DEFAULTS, **case}
    n = int(_sizes(c).sum()) if c["call"] == "batched" else c["n"]
    sinks = c["sinks"] or n
    # particles in (x, y, z, m), potential and acceleration out
    nbytes = 32.0 * n + 32.0 * sinks
    if c["call"] in ("active", "direct_sinks"):
        nbytes += 8.0 * sinks
    if c["call"] == "jerk":
        nbytes += 48.0 * n
    if c["call"] == "eps":
        nbytes += 8.0 * n
    if c["call"] == "direct":
        return {"bytes": nbytes, "flops": 20.0 * n * n}
    if c["call"] == "direct_sinks":
        return {"bytes": nbytes, "flops": 20.0 * n * sinks}
    # The multipole method's direct pairs and M2L of one sink: 1.47e4 pairs of
    # 20 operations and 1.9 M2L of 8 sum (n+1)(p-n+1)^2 at N = 10^6 and
    # eps = 6e-8, falling as error^-0.18 (Dehnen 2014, Sec. 6.2); never more than
    # the direct sum.
    per_sink = min(20.0 * n, 4.0e5 * (c["eps"] / 6e-8) ** -0.18)
    if c["call"] == "jerk":
        per_sink *= 1.9
    if c["call"] == "eps":
        per_sink *= 0.5
    return {"bytes": nbytes, "flops": per_sink * sinks}


def _direct(pos, mass, sinks, vel=None):
    """Potential, acceleration (and jerk) of the listed sinks by plain sums."""
    n, k = pos.shape[0], sinks.shape[0]
    pot = torch.empty(k, dtype=torch.float64, device=pos.device)
    acc = torch.empty((k, 3), dtype=torch.float64, device=pos.device)
    jerk = torch.empty((k, 3), dtype=torch.float64, device=pos.device)
    step = max(1, (1 << 26) // max(n, 1))
    for s in range(0, k, step):
        idx = sinks[s:s + step]
        d = [pos[None, :, a] - pos[idx][:, a, None] for a in range(3)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        r2.scatter_(1, idx[:, None], math.inf)       # no self term
        ri = torch.rsqrt(r2)
        q = mass[None, :] * ri
        pot[s:s + step] = -q.sum(1)
        q *= ri * ri
        for a in range(3):
            acc[s:s + step, a] = (q * d[a]).sum(1)
        if vel is not None:
            dv = [vel[None, :, a] - vel[idx][:, a, None] for a in range(3)]
            rv = (d[0] * dv[0] + d[1] * dv[1] + d[2] * dv[2]) * (ri * ri)
            for a in range(3):
                jerk[s:s + step, a] = (q * (dv[a] - 3.0 * rv * d[a])).sum(1)
    return (pot, acc) if vel is None else (pot, acc, jerk)


def exact(case, seed):
    c = {**DEFAULTS, **case}
    pairs = float(c["sinks"] or c["n"]) * c["n"]
    if c["call"] == "batched":
        pairs = float((_sizes(c).astype(np.float64) ** 2).sum())
    if pairs > 1.5e11:
        return None
    d = _inputs(c, seed)
    if c["call"] == "batched":
        off = d["offsets"]
        parts = [_direct(d["pos"][a:b], d["mass"][a:b], torch.arange(b - a, device=DEV))
                 for a, b in zip(off[:-1].tolist(), off[1:].tolist())]
        return tuple(torch.cat(x) for x in zip(*parts))
    sinks = d["sinks"] if "sinks" in d else torch.arange(c["n"], device=DEV)
    return _direct(d["pos"], d["mass"], sinks, d.get("vel"))
