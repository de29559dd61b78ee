"""Automatic plans without room for their split scratch take fewer splits: under a
scratch limit, and while a stream is being captured on a context without any."""
import numpy as np
import pytest
import torch

import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import TOL_FP64, TOL_MIXED, compare_force, dev, host, say

pytestmark = pytest.mark.gpu

TOL = {"fp64": TOL_FP64, "mixed": TOL_MIXED}


def _case(n, n_i, cap):
    s = W.small_state(70 + n_i, n, k_nn=20)
    ib = np.random.default_rng(n).permutation(n)[:n_i].astype(np.int32)
    return s, ib, s["rs2"][ib]


def _defined(out, cap):
    cnt, lst = host(out[2]), host(out[3])
    used = np.arange(cap)[None, :] < np.minimum(cnt, cap)[:, None]
    return cnt, np.where(used, lst, -1)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_i,limit,least", [(8192, 8192, 64 << 20, 16), (1024, 1024, 1 << 20, 2),
                                               (2000, 300, 3 << 20, 16), (512, 200, 4096, 1),
                                               (70000, 1200, 80 << 20, 137)])
def test_fewer_splits_under_a_limit(n, n_i, limit, least, prec):
    say(f"scratch limit {limit} n={n} n_i={n_i} {prec}")
    cap = 24
    s, ib, rs2 = _case(n, n_i, cap)
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2), cap, prec)
    free, tight = nb.Context(0), nb.Context(0)
    try:
        tight.set_scratch_limit(limit)
        a = nb.regular_force(*args, ctx=free)
        b = nb.regular_force(*args, ctx=tight)
        k0, k1 = (int(c.last_plan().split("splits=")[1].split()[0]) for c in (free, tight))
        say(f"  {k0} splits, {k1} in {limit} bytes")
        assert least <= k1 < k0
        for x, y in zip(_defined(a, cap), _defined(b, cap)):
            assert np.array_equal(x, y)
        rows = np.random.default_rng(1).choice(n_i, min(n_i, 64), replace=False)
        compare_force(b, s["x"], s["v"], s["m"], ib, rs2, cap, TOL[prec], rows=rows)
        tight.set_scratch_limit(1024)
        if k1 > 1:      # not even the least splits fit
            tight2 = nb.Context(0)
            tight2.set_scratch_limit(1024)
            with pytest.raises(nb.NbError) as err:
                nb.regular_force(*args, ctx=tight2)
            assert err.value.code == -3
            tight2.close()
    finally:
        free.close()
        tight.close()


def test_small_block_captured_on_a_fresh_context():
    """A small FP64 block needs no scratch, so its first call may be a captured one."""
    n, n_i, cap = 500, 200, 24
    say("captured first call")
    s, ib, rs2 = _case(n, n_i, cap)
    x, v, m = dev(s["x"]), dev(s["v"]), dev(s["m"])
    out = (torch.empty((3, n_i), dtype=torch.float64, device="cuda"),
           torch.empty((3, n_i), dtype=torch.float64, device="cuda"),
           torch.empty(n_i, dtype=torch.int32, device="cuda"),
           torch.empty((n_i, cap), dtype=torch.int32, device="cuda"),
           torch.empty(1, dtype=torch.int32, device="cuda"))
    dib, drs2 = dev(ib), dev(rs2)
    ctx = nb.Context(0)
    try:
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            nb.regular_force(x, v, m, dib, drs2, cap, "fp64", out=out, ctx=ctx)
        for k in range(3):
            x.copy_(torch.from_numpy(np.ascontiguousarray(s["x"] * (1.0 + 0.25 * k))))
            g.replay()
            torch.cuda.synchronize()
            compare_force(out, s["x"] * (1.0 + 0.25 * k), s["v"], s["m"], ib, rs2, cap, TOL_FP64)
            eager = nb.regular_force(x, v, m, dib, drs2, cap, "fp64", ctx=ctx)
            torch.cuda.synchronize()
            for p, q in zip(_defined(out, cap), _defined(eager, cap)):
                assert np.array_equal(p, q)
    finally:
        ctx.close()
