"""M2L kernels at every compiled order, against the oracle's FMM with the same
parameters: lists of one to many entries per sink (chunks of 16, blocks of 64
chunks), and pairs whose separation lies on the z axis, where the azimuth is
arbitrary.

Tolerance: as in the parity tests, expansions are sums of terms up to ~1/eps
larger than the result, each correct to ~1e-16: 1e-10 relative; in mixed
precision the FP32 terms and direct sums: 64 FP32 units of sum mu / r^2.
"""
import numpy as np
import pytest

import oracle
from paper_1405_2255_amd import workloads

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _points(kind, n, seed):
    if kind == "axis":        # every separation along z, either way
        rng = np.random.default_rng(seed)
        pos = np.zeros((n, 3))
        pos[:, 2] = rng.uniform(-1.0, 1.0, n)
        return pos, np.full(n, 1.0 / n)
    return workloads.cluster(kind, n, seed, masses="salpeter")


@pytest.mark.parametrize("kind", ["plummer", "axis"])
@pytest.mark.parametrize("p", list(range(3, 17)))
def test_orders_match_oracle(gpu_lib, p, kind):
    n, leaf, eps = 1500, 8, 10.0 ** (-0.5 * p)
    pos, m = _points(kind, n, 40 + p)
    ctx = gpu_lib.Context(leaf_size=leaf, p2p_factor=0.05)
    pot, acc = ctx.forces(_dev(pos), _dev(m), 1.0, p=p, target_err=eps)
    ref = oracle.fmm(pos, m, p=p, eps=eps, leaf_size=leaf, p2p_pairs=0.05 * (p + 1) ** 3)
    assert ctx.stats()["n_m2l"] == ref["stats"]["n_m2l"] > 0
    f0 = oracle.direct(pos, m)[2]
    assert np.max(np.linalg.norm(acc.cpu().numpy() - ref["acc"], axis=1) / f0) < 1e-10
    assert np.max(np.abs(pot.cpu().numpy() - ref["pot"]) / np.abs(ref["pot"])) < 1e-10
    mixed = gpu_lib.Context(leaf_size=leaf, p2p_factor=0.05, precision="mixed")
    _, a32 = mixed.forces(_dev(pos), _dev(m), 1.0, p=p, target_err=eps)
    d = np.linalg.norm(a32.cpu().numpy() - ref["acc"], axis=1)
    assert np.max(d / f0) < 64 * 2.0 ** -24
