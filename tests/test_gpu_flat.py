"""Bodies on a lattice in the plane x = 0 but for offsets whose squares are
denormal: many cells lie beside each other along z with nothing but such an
offset between their axes.  Against the oracle's method with the same parameters
(the bound of the other comparisons with it)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0.0, 2e-162, 1e-158, 1e-150])
def test_plane_with_tiny_offsets(gpu_lib, offset):
    import torch
    rng = np.random.default_rng(23)
    y, z = np.meshgrid(np.arange(48.0), np.arange(48.0), indexing="ij")
    pos = np.stack([offset * rng.standard_normal(y.size), y.ravel(), z.ravel()], axis=1)
    m = rng.random(len(pos)) / len(pos)
    p, eps, leaf = 8, 1e-6, 4
    ctx = gpu_lib.Context(leaf_size=leaf, p2p_factor=0.05, centre="midpoint")
    pot, acc = ctx.forces(*(torch.from_numpy(a).to("cuda:0") for a in (pos, m)), 1.0, p, eps)
    ref = oracle.fmm(pos, m, p=p, eps=eps, leaf_size=leaf, p2p_pairs=0.05 * (p + 1) ** 3,
                     centre=oracle.CENTRE_MIDPOINT)
    assert ctx.stats()["n_m2l"] == ref["stats"]["n_m2l"] > 0
    f0 = oracle.direct(pos, m)[2]
    assert np.max(np.linalg.norm(acc.cpu().numpy() - ref["acc"], axis=1) / f0) < 1e-10
    assert np.max(np.abs(pot.cpu().numpy() - ref["pot"]) / np.abs(ref["pot"])) < 1e-10
