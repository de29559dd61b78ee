"""The mixed packed pass at 2^18 bodies and more, whose near pairs wait in queues,
against the LDS pass, which adds them at once: equal lists, sums within twice the
mixed tolerance of each other (each is within one of the exact ones)."""
import numpy as np
import pytest

import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import TOL_MIXED, compare_force, dev, host, row_rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_i", [(1 << 18, 1030), ((1 << 18) + 31, 600), (300001, 2049)])
def test_packed_near_pairs_against_lds(n, n_i):
    say(f"packed near pairs n={n} n_i={n_i}")
    cap = 40
    s = W.small_state(n_i, n, k_nn=20)
    rng = np.random.default_rng(n)
    ib = rng.choice(n, n_i, replace=False).astype(np.int32)
    rs2 = s["rs2"][ib].copy()
    rs2[::7] *= 4.0
    rs2[1::11] = 0.0
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2), cap, "mixed")
    ctx = nb.Context(0)
    try:
        ctx.set_plan(1, 1, 5)
        a = [host(t) for t in nb.regular_force(*args, ctx=ctx)]
        assert "bodies=packed" in ctx.last_plan(), ctx.last_plan()
        ctx.set_plan(1, 2, 5)     # two rows per lane: the LDS pass
        b = [host(t) for t in nb.regular_force(*args, ctx=ctx)]
        assert "packed" not in ctx.last_plan()
        ctx.set_plan(1, 1, 5)
        res = nb.regular_force(*args, ctx=ctx)
    finally:
        ctx.close()
    used = np.arange(cap)[None, :] < np.minimum(a[2], cap)[:, None]
    assert np.array_equal(a[2], b[2])
    assert np.array_equal(np.where(used, a[3], -1), np.where(used, b[3], -1))
    for k in (0, 1):
        assert row_rel_err(a[k], b[k]).max() <= 2 * TOL_MIXED
    compare_force(res, s["x"], s["v"], s["m"], ib, rs2, cap, TOL_MIXED,
                  rows=rng.choice(n_i, 48, replace=False))
