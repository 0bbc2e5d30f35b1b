"""Near field whose list entries are taken in several parts (split.h): leaves of
one body have hundreds of entries each, and those of all leaves together pass
the bound of one part.  A call for a few listed sinks has one part only, and sums
each of them in the same order, so the results agree bit for bit."""
import os
import re

import numpy as np
import pytest

from paper_1405_2255_amd import workloads

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BEGIN = (1 << 40) - 1


def _bound():
    text = open(os.path.join(ROOT, "paper_1405_2255_amd", "csrc", "split.h")).read()
    return 1 << int(re.search(r"NEAR_ENTRIES = int64_t\(1\) << (\d+);", text).group(1))


def _entries(ctx):
    """The merged ranges of every cell, once for each leaf below it, and a
    closing entry per leaf."""
    import torch
    q, c = (torch.from_numpy(a).cuda() for a in (ctx.export_p2p(), ctx.export_cells()))
    new = torch.ones(len(q), dtype=torch.bool, device="cuda")
    new[1:] = (q[1:, 0] != q[:-1, 0]) | (q[1:, 1] != q[:-1, 2])
    sink, count = torch.unique(q[new, 0], return_counts=True)
    c = c[torch.argsort(c[:, 0])]
    i = torch.searchsorted(c[:, 0].contiguous(), sink)
    beg, end = c[i, 0] & BEGIN, c[i, 1]
    # a leaf begins wherever a cell begins
    leaf = torch.zeros(int(c[:, 1].max()) + 1, dtype=torch.int64, device="cuda")
    leaf[c[:, 0] & BEGIN] = 1
    before = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), leaf.cumsum(0)])
    return int((count * (before[end] - before[beg])).sum()) + int(leaf.sum())


def test_leaves_of_one_body(gpu_lib):
    import torch
    n, p, eps = 700000, 8, 1e-6
    pos, m = workloads.cluster("plummer", n, 5)
    vel = np.random.default_rng(6).standard_normal(pos.shape)
    s = np.random.default_rng(7).choice(n, 20000, replace=False).astype(np.int64)
    P, V, M, S = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (pos, vel, m, s))
    ctx = gpu_lib.Context(leaf_size=1)
    pot, acc = ctx.forces(P, M, 1.0, p, eps)
    assert _entries(ctx) > _bound()
    pj, aj, jerk = ctx.forces_jerk(P, V, M, 1.0, p, eps)
    pl, al, jl = ctx.forces_jerk_active(P, V, M, S, 1.0, p, eps)
    assert torch.equal(pot, pj) and torch.equal(acc, aj)
    assert torch.equal(pl, pot[S]) and torch.equal(al, acc[S]) and torch.equal(jl, jerk[S])
    # (errors of the method at this accuracy: a few 1e-5 at the worst body)
    p0, a0 = ctx.direct_sinks(P, M, S[:256].contiguous())
    assert ((pot[S[:256]] - p0) / p0).abs().max().item() < 1e-3
    assert ((acc[S[:256]] - a0).norm(dim=1) / a0.norm(dim=1)).max().item() < 1e-3
