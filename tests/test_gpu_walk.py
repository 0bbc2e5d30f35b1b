"""A context plans a walk's launches from the frontiers of its last walk (one
block, tiles, full sweeps).  Whatever the last call was, the lists and results
must be those of a fresh context, whose walk does not know the sizes."""
import numpy as np
import pytest

from paper_1405_2255_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1500, 1500), (12000, 12000), (60000, 60000),
                                   (1500, 90000, 1500), (90000, 12000, 90000)])
def test_walk_does_not_depend_on_the_last_one(gpu_lib, sizes):
    import torch

    def call(ctx, n):
        pos, m = W.cluster("dehnen1.5" if n % 60000 else "plummer", n, n, masses="salpeter")
        pot, acc = ctx.forces(torch.as_tensor(pos, device="cuda"),
                              torch.as_tensor(m, device="cuda"), p=8, target_err=1e-6)
        st = ctx.stats()
        return (ctx.export_m2l(), ctx.export_p2p(), pot.cpu().numpy(), acc.cpu().numpy(),
                [st[k] for k in ("n_m2l", "n_p2p_lists", "n_p2p_pairs", "n_est_m2l",
                                 "n_est_p2p_pairs", "walk_iterations", "walk_pairs")])

    ctx = gpu_lib.Context(leaf_size=16)
    for n in sizes:
        got, want = call(ctx, n), call(gpu_lib.Context(leaf_size=16), n)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
