"""A context on torch's default stream uses a call's tensors only after the work
that is queued there: inputs that are still being made when the call comes give
the results of the finished ones."""
import numpy as np
import pytest

from paper_1405_2255_amd import workloads

pytestmark = pytest.mark.gpu


def test_inputs_still_being_made(gpu_lib):
    import torch
    n = 20000
    pos, m = workloads.cluster("plummer", n, 8)
    vel = np.random.default_rng(9).standard_normal(pos.shape)
    P, V, M = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (pos, vel, m))
    S = torch.arange(0, n, 7, device="cuda:0")
    eps = torch.full((n,), 1e-6, dtype=torch.float64, device="cuda:0")
    ctx = gpu_lib.Context()
    assert ctx.stream.cuda_stream == 0
    w = torch.randn(4096, 4096, device="cuda:0")

    def late(t):
        """A copy of t that the device makes some milliseconds from now (until
        then another valid input: t in reverse order)."""
        out = t.flip(0).contiguous()
        torch.cuda.synchronize()
        x = w
        for _ in range(40):
            x = (x @ w) * 1e-2
        out.copy_(t)
        return out

    calls = [lambda f: ctx.forces(f(P), M, 1.0, 6, 1e-5),
             lambda f: ctx.forces_batched([0, n // 2, n], f(P), M, 1.0, 6, 1e-5),
             lambda f: ctx.forces_active(P, M, f(S), 1.0, 6, 1e-5),
             lambda f: ctx.forces_eps(f(P), M, eps, 1.0, 6),
             lambda f: ctx.forces_jerk(P, f(V), M, 1.0, 6, 1e-5),
             lambda f: ctx.forces_jerk_active(P, V, M, f(S), 1.0, 6, 1e-5),
             lambda f: ctx.direct(f(P), M),
             lambda f: ctx.direct_sinks(P, M, f(S)),
             lambda f: ctx.direct_jerk_sinks(P, V, M, f(S))]
    for call in calls:
        want = call(lambda t: t)
        torch.cuda.synchronize()
        got = call(late)
        for a, b in zip(want, got):
            assert torch.equal(a, b)
