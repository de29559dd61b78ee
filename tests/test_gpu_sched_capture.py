"""A scheduler build of up to 16384 bodies depends on nothing that an earlier call
left behind: captured on a fresh context, replayed after the context's scratch
has grown."""
import numpy as np
import pytest
import torch

import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

K = 20


def _want(lev):
    order = np.lexsort((np.arange(lev.size), -lev)).astype(np.int32)
    return order, np.array([(lev >= L).sum() for L in range(K + 2)], np.int32)


@pytest.mark.parametrize("scratch_first", [False, True])
@pytest.mark.parametrize("n", [8193, 10240, 10241, 16384])
def test_captured_build_outlives_the_scratch(n, scratch_first):
    say(f"captured build n={n} scratch={scratch_first}")
    rng = np.random.default_rng(n)
    level = dev(rng.integers(0, K + 1, n).astype(np.int32))
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    le = torch.empty(K + 2, dtype=torch.int32, device="cuda")
    s = W.small_state(3, 6000, k_nn=20)
    ib = np.arange(6000, dtype=np.int32)
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(s["rs2"]), 16, "fp64")
    ctx = nb.Context(0)
    try:
        if scratch_first:
            nb.sched_build(dev(np.zeros(70000, np.int32)), K, ctx=ctx)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            nb.sched_build(level, K, order=order, level_end=le, ctx=ctx)
        for k in range(3):
            lev = rng.integers(0, K + 1, n).astype(np.int32)
            level.copy_(torch.from_numpy(lev))
            g.replay()
            torch.cuda.synchronize()
            want, ends = _want(lev)
            assert np.array_equal(host(order), want) and np.array_equal(host(le), ends)
            # grows the scratch, and allocates where it was
            nb.regular_force(*args, ctx=ctx)
            torch.cuda.synchronize()
            eager, ends2 = nb.sched_build(level, K, ctx=ctx)
            assert np.array_equal(host(eager), want) and np.array_equal(host(ends2), ends)
    finally:
        ctx.close()
