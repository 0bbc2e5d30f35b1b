"""FP64 direct sums at the edges of their tiles, against the oracle's direct
sum: sinks per wavefront (8; 6 with the jerk), 64 sources per step, 4096
sources per slice, 64 list entries held at a time.

Tolerance: every pair's term has a relative error of a few 1e-16 and the terms
of one sink are added in lanes and slices of at most a few thousand, so the sum
is within 1e-12 of sum |terms| (the bound of the direct-sum tests); the sums
of these samples cancel by less than the margin left.
"""
import numpy as np
import pytest

import oracle
from paper_1405_2255_amd import workloads

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _check(gpu_lib, pos, m, leaf, **kw):
    ctx = gpu_lib.Context(leaf_size=leaf)
    vel = np.random.default_rng(7).standard_normal(pos.shape)
    pot, acc = ctx.forces(_dev(pos), _dev(m), 1.0, **kw)
    p0, a0, f0 = oracle.direct(pos, m)
    assert np.max(np.abs(pot.cpu().numpy() - p0) / np.abs(p0)) < 1e-12
    assert np.max(np.linalg.norm(acc.cpu().numpy() - a0, axis=1) / f0) < 1e-12
    pj, aj, jerk = ctx.forces_jerk(_dev(pos), _dev(vel), _dev(m), 1.0, **kw)
    assert np.array_equal(pj.cpu().numpy(), pot.cpu().numpy())
    assert np.array_equal(aj.cpu().numpy(), acc.cpu().numpy())
    j0 = oracle.direct_jerk(pos, vel, m)
    assert np.max(np.linalg.norm(jerk.cpu().numpy() - j0, axis=1) /
                  np.linalg.norm(j0, axis=1)) < 1e-10


@pytest.mark.parametrize("n", [2, 3, 6, 7, 8, 9, 13, 16, 17, 63, 64, 65, 127, 128, 129, 191, 1025,
                               4095, 4096])
def test_one_leaf(gpu_lib, n):
    pos, m = workloads.cluster("uniform", n, 100 + n, masses="salpeter")
    _check(gpu_lib, pos, m, 4096, p=4, target_err=1e-6)


@pytest.mark.parametrize("n,leaf", [(4097, 512), (8192, 100), (8193, 64), (12300, 200)])
def test_lists_of_several_slices(gpu_lib, n, leaf):
    # an accuracy that no cell pair meets: every pair is summed directly, in
    # lists of n sources
    pos, m = workloads.cluster("uniform", n, 200 + n, masses="salpeter")
    _check(gpu_lib, pos, m, leaf, p=3, target_err=1e-300)


@pytest.mark.parametrize("n,leaf", [(700, 1), (3000, 1), (3000, 2)])
def test_lists_of_many_short_ranges(gpu_lib, n, leaf):
    # tiny leaves and a loose accuracy: lists of hundreds of ranges of one or a
    # few particles, against the oracle's method with the same parameters
    pos, m = workloads.cluster("plummer", n, 300 + n, masses="salpeter")
    ctx = gpu_lib.Context(leaf_size=leaf, p2p_factor=0.1)
    pot, acc = ctx.forces(_dev(pos), _dev(m), 1.0, p=4, target_err=1e-3)
    ref = oracle.fmm(pos, m, p=4, eps=1e-3, leaf_size=leaf, p2p_pairs=0.1 * 125)
    st = ctx.stats()
    assert st["n_m2l"] == ref["stats"]["n_m2l"] and st["n_p2p_pairs"] == ref["stats"]["n_p2p_pairs"]
    assert np.max(np.linalg.norm(acc.cpu().numpy() - ref["acc"], axis=1) /
                  np.linalg.norm(ref["acc"], axis=1)) < 1e-10
    assert np.max(np.abs(pot.cpu().numpy() - ref["pot"]) / np.abs(ref["pot"])) < 1e-10


@pytest.mark.parametrize("n", [2, 7, 8, 9, 63, 64, 65, 513, 1023, 1024, 1025, 2049, 5000])
def test_exact_sums(gpu_lib, n):
    # 8 sinks per wavefront, 64 sources per step, chunks of at least 512 sources;
    # the list unsorted and with repeats, its ends at the ends of chunks
    pos, m = workloads.cluster("uniform", n, 400 + n, masses="salpeter")
    vel = np.random.default_rng(n).standard_normal(pos.shape)
    P, V, M = _dev(pos), _dev(vel), _dev(m)
    ctx = gpu_lib.Context()
    p0, a0, f0 = oracle.direct(pos, m)
    pot, acc = ctx.direct(P, M, 1.0)
    assert np.max(np.abs(pot.cpu().numpy() - p0) / np.abs(p0)) < 1e-12
    assert np.max(np.linalg.norm(acc.cpu().numpy() - a0, axis=1) / f0) < 1e-12
    rng = np.random.default_rng(n + 1)
    for k in (1, 5, 11):
        s = np.concatenate([rng.integers(0, n, k), [n - 1, 0, n // 2, n - 1]]).astype(np.int64)
        pot, acc = ctx.direct_sinks(P, M, _dev(s), 1.0)
        assert np.max(np.abs(pot.cpu().numpy() - p0[s]) / np.abs(p0[s])) < 1e-12
        assert np.max(np.linalg.norm(acc.cpu().numpy() - a0[s], axis=1) / f0[s]) < 1e-12
        jerk = ctx.direct_jerk_sinks(P, V, M, _dev(s), 1.0).cpu().numpy()
        j0 = oracle.direct_jerk(pos, vel, m, sinks=s)
        assert np.max(np.linalg.norm(jerk - j0, axis=1) / np.linalg.norm(j0, axis=1)) < 1e-10
