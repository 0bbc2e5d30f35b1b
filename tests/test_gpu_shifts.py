"""Upward and downward shifts at the orders where a lane's number of coefficients
changes (64 per round) and for cells that lie along one axis or in one plane,
where a part of the shift vanishes; against the oracle, as the parity tests."""
import numpy as np
import pytest

import oracle
from paper_1405_2255_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,kind", [(3, "ball"), (9, "ball"), (10, "ball"), (14, "ball"),
                                    (15, "ball"), (18, "ball"), (19, "ball"), (20, "ball"),
                                    (10, "line"), (15, "line"), (10, "plane"), (15, "plane")])
def test_shifts_match_oracle(gpu_lib, p, kind):
    import torch
    pos, m = W.cluster("plummer", 3000, 11, masses="salpeter")
    if kind == "line":
        pos[:, :2] = 0.0
    elif kind == "plane":
        pos[:, 2] = 0.0
    eps = 1e-4 if p < 9 else 1e-8
    ctx = gpu_lib.Context(leaf_size=8, p2p_factor=0.01)
    pot, acc = ctx.forces(torch.as_tensor(pos, device="cuda"), torch.as_tensor(m, device="cuda"),
                          p=p, target_err=eps)
    ref = oracle.fmm(pos, m, p=p, eps=eps, leaf_size=8, p2p_pairs=0.01 * (p + 1) ** 3)
    assert ctx.stats()["n_m2l"] == ref["stats"]["n_m2l"] > 0
    acc, pot = acc.cpu().numpy(), pot.cpu().numpy()
    err = np.linalg.norm(acc - ref["acc"], axis=1) / np.linalg.norm(ref["acc"], axis=1)
    assert err.max() < 1e-10
    assert np.max(np.abs(pot - ref["pot"]) / np.abs(ref["pot"])) < 1e-10
