"""Exact sums of few sinks of a large system, whose sources are cut into many
rows, against plain FP64 sums.

Tolerance: a term has a relative error of a few 1e-16 (the jerk's, with its
longer expression, below 1e-14), and a sink's terms are added by lanes, rows of
a few hundred sources and up to a few thousand rows, so a sum is within 1e-12 of
the sum of its terms' sizes."""
import numpy as np
import pytest

from paper_1405_2255_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(1000000, 64), (1000000, 100), (1000000, 1), (500000, 64)])
def test_few_sinks_of_many_sources(gpu_lib, n, k):
    import torch
    pos, m = workloads.cluster("plummer", n, 3, masses="salpeter")
    vel = np.random.default_rng(4).standard_normal(pos.shape)
    sinks = np.random.default_rng(5).choice(n, k, replace=False).astype(np.int64)
    sinks[-1] = n - 1
    P, V, M, S = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
                  for a in (pos, vel, m, sinks))
    ctx = gpu_lib.Context()
    pot, acc = ctx.direct_sinks(P, M, S, 1.0)
    pot2, acc2 = ctx.direct_sinks(P, M, S, 1.0, noalloc=True)
    jerk = ctx.direct_jerk_sinks(P, V, M, S, 1.0)
    assert torch.equal(pot, pot2) and torch.equal(acc, acc2)
    for j, i in enumerate(sinks.tolist()):
        d, dv = P - P[i], V - V[i]
        r2 = (d * d).sum(1)
        r2[i] = float("inf")
        ri = r2.rsqrt()
        q = M * ri
        p0, q = -q.sum(), q * ri * ri
        a0 = (q[:, None] * d).sum(0)
        rv = 3.0 * (d * dv).sum(1) * ri * ri
        t = q[:, None] * (dv - rv[:, None] * d)
        size_a = (q * d.norm(dim=1)).sum()
        size_j = (q * (dv.norm(dim=1) + rv.abs() * d.norm(dim=1))).sum()
        assert ((pot[j] - p0) / p0).abs().item() < 1e-12
        assert ((acc[j] - a0).norm() / size_a).item() < 1e-12
        assert ((jerk[j] - t.sum(0)).norm() / size_j).item() < 1e-12
