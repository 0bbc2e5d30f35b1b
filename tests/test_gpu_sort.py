"""Sorted particles and lists at the sizes where the radix sort changes its way:
one block up to 8192 keys, one tile more or less, a last tile of one key, and
lists long enough for the wide tiles (over 2^21 entries)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (particles, leaf size)
SIZES = [(2, 8), (63, 8), (2047, 8), (8191, 16), (8192, 16), (8193, 16), (10240, 16),
         (10241, 16), (16385, 32), (150001, 48)]


@pytest.mark.parametrize("n,leaf", SIZES)
def test_particles_and_lists_are_in_order(gpu_lib, n, leaf):
    import torch
    rng = np.random.default_rng(n)
    # a tight clump beside a wide one: upper digits shared by whole wavefronts
    pos = rng.standard_normal((n, 3))
    pos[: n // 2] = pos[: n // 2] * 1e-3 + 0.3
    m = rng.random(n) / n + 1e-3 / n
    P, M = torch.as_tensor(pos, device="cuda"), torch.as_tensor(m, device="cuda")
    ctx = gpu_lib.Context(leaf_size=leaf)
    pot, acc = ctx.forces(P, M, p=8, target_err=1e-6)
    st = ctx.stats()
    # every body sits in the leaf that the order says, or its force is off by
    # far more than the expansions' error (a few 1e-5 at the worst body)
    sinks = torch.as_tensor(rng.integers(0, n, min(n, 512)), device="cuda")
    p0, a0 = ctx.direct_sinks(P, M, sinks)
    err = (acc[sinks] - a0).norm(dim=1) / a0.norm(dim=1)
    assert err.max().item() < 1e-3
    assert ((pot[sinks] - p0) / p0).abs().max().item() < 1e-3
    # lists by sink cell (and first source particle), nothing lost
    m2l = ctx.export_m2l()
    assert m2l.shape[0] == st["n_m2l"] and np.all(np.diff(m2l[:, 1]) >= 0)
    p2p = ctx.export_p2p()
    end_of = dict(map(tuple, ctx.export_cells()))
    sink, beg, end = p2p[:, 0], p2p[:, 1], p2p[:, 2]
    same = np.diff(sink) == 0
    assert p2p.shape[0] == st["n_p2p_lists"] and np.all(np.diff(sink) >= 0)
    assert np.all(np.diff(beg)[same] > 0)
    size = np.array([end_of[s] - (s & ((1 << 40) - 1)) for s in sink])
    own = np.minimum(end, (sink & ((1 << 40) - 1)) + size) - np.maximum(beg, sink & ((1 << 40) - 1))
    pairs = (size * (end - beg)).sum() - np.maximum(own, 0).sum()
    assert pairs == st["n_p2p_pairs"]
    if n > 100000:
        assert st["n_p2p_lists"] > 1 << 21
