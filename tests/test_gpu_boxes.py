"""Boxes and keys of batched clusters whose boundaries fall anywhere in the pieces
that a wavefront takes: many tiny clusters, one of thousands, close bodies
(long runs of one key) at a cluster's ends.  Each cluster must come out as in a
call of its own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[2, 3, 61, 64, 65, 63, 1, 130, 7] * 5,
                                   [5, 9000, 3, 4097, 64, 2],
                                   [70] * 200 + [20001]])
def test_clusters_equal_calls_of_their_own(gpu_lib, sizes):
    import torch
    rng = np.random.default_rng(len(sizes))
    off = np.concatenate([[0], np.cumsum(sizes)])
    pos = rng.standard_normal((off[-1], 3))
    for c, n in enumerate(sizes):
        pos[off[c]:off[c + 1]] = pos[off[c]:off[c + 1]] * 10.0 ** rng.integers(-3, 4) + c
        k = n // 8        # bodies close together: one key of the first word
        pos[off[c]:off[c] + k] = pos[off[c]] * (1.0 + 1e-7 * rng.random((k, 1)))
    m = rng.random(off[-1]) + 0.5
    P, M = torch.as_tensor(pos, device="cuda"), torch.as_tensor(m, device="cuda")
    pot, acc = gpu_lib.Context(leaf_size=16).forces_batched(off, P, M, p=6, target_err=1e-5)
    one = gpu_lib.Context(leaf_size=16)
    for c in list(range(0, len(sizes), max(1, len(sizes) // 12))) + [len(sizes) - 1]:
        a, b = off[c], off[c + 1]
        p1, a1 = one.forces(P[a:b].contiguous(), M[a:b].contiguous(), p=6, target_err=1e-5)
        assert torch.equal(p1, pot[a:b]) and torch.equal(a1, acc[a:b])
