"""The radix sort where its tiles change their width (2^17 keys): particles in the
order of their keys, on one context that sorts the longer array first, so that
the shorter one finds its scratch made."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def test_particles_around_the_change_of_width(gpu_lib):
    import torch
    rng = np.random.default_rng(31)
    pos = rng.standard_normal((135169, 3))
    pos[::2] = pos[::2] * 1e-3 + 0.3        # upper digits that whole wavefronts share
    m = rng.random(len(pos)) / len(pos)
    ctx = gpu_lib.Context(leaf_size=32)
    # 131072 is the last length of 64 narrow tiles; 131073 has 33 wide ones, the
    # last with one key; 135168 = 33 full wide tiles
    for n in (135169, 135168, 131073, 131072, 131071, 129025):
        P, M = torch.from_numpy(pos[:n]).to("cuda:0"), torch.from_numpy(m[:n]).to("cuda:0")
        pot, acc = ctx.forces(P, M, p=6, target_err=1e-5)
        fresh = gpu_lib.Context(leaf_size=32)
        want = fresh.forces(P, M, p=6, target_err=1e-5)
        assert torch.equal(pot, want[0]) and torch.equal(acc, want[1])
        # every cell holds the particles that its place in the key order says
        cells = ctx.export_cells()
        level, beg, end = cells[:, 0] >> 40, cells[:, 0] & ((1 << 40) - 1), cells[:, 1]
        lo = pos[:n].min(0)
        q = (pos[:n] - lo) * (2.0 ** 21 / (pos[:n].max(0) - lo).max())
        q = np.minimum(np.floor(q), 2 ** 21 - 1).astype(np.int64)
        key = np.zeros(n, dtype=np.int64)
        for b in range(21):
            for d in range(3):
                key |= ((q[:, d] >> b) & 1) << (3 * b + d)
        key = np.sort(key)
        for s in (2, 5, 8):
            k = key >> (3 * (21 - s))
            on = level == s
            assert np.all(k[beg[on]] == k[end[on] - 1])
        sinks = rng.integers(0, n, 256)
        _, a0, f0 = oracle.direct(pos[:n], m[:n], sinks=sinks)
        err = np.linalg.norm(acc.cpu().numpy()[sinks] - a0, axis=1) / f0
        assert err.max() < 1e-3             # a body in the wrong leaf is off by far more
