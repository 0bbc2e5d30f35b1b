"""Rates of the multipoles at the orders where their kernel's layout changes (lanes
per particle: degree p - 1 up to 3, 7, 15 and above; even and odd middle columns;
registers from 16), against the oracle at the jerk's parity bound of 1e-9."""
import numpy as np
import pytest

import oracle
from paper_1405_2255_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [3, 4, 5, 7, 8, 9, 15, 16, 17, 20])
def test_jerk_of_every_layout_matches_oracle(gpu_lib, p):
    import torch
    n, eps = 2500, 1e-4 if p < 8 else 1e-8
    pos, vel = W.plummer(n, 40 + p, with_velocities=True)
    m = np.random.default_rng(p).random(n) / n
    P, V, M = (torch.as_tensor(np.ascontiguousarray(a), device="cuda") for a in (pos, vel, m))
    ctx = gpu_lib.Context(leaf_size=8, p2p_factor=0.01)
    pot, acc, jerk = ctx.forces_jerk(P, V, M, p=p, target_err=eps)
    ref = oracle.fmm(pos, m, p=p, eps=eps, leaf_size=8, p2p_pairs=0.01 * (p + 1) ** 3, vel=vel)
    assert ctx.stats()["n_m2l"] == ref["stats"]["n_m2l"] > 0
    j = jerk.cpu().numpy()
    err = np.linalg.norm(j - ref["jerk"], axis=1) / np.linalg.norm(ref["jerk"], axis=1)
    assert err.max() < 1e-9
