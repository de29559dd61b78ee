"""The scheduler's one-work-group and two-launch sorts at the sizes where either
may run."""
import numpy as np
import pytest

import paper_1504_03687_amd as nb
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k_max", [(8193, 63), (16384, 20), (16384, 0), (65536 + 4095, 63)])
def test_both_paths_give_one_list(n, k_max):
    """Builds and updates of up to 16384 bodies run in one work-group while the
    context has no scratch and in two launches once it has: same offsets and,
    for the stable build, the same list; every level up to 63 and a single one."""
    say(f"sched paths n={n} k_max={k_max}")
    rng = np.random.default_rng(n + k_max)
    lev = rng.integers(0, k_max + 1, n).astype(np.int32)
    want = np.lexsort((np.arange(n), -lev)).astype(np.int32)
    ends = np.array([(lev >= L).sum() for L in range(k_max + 2)], np.int32)
    L = k_max // 2
    new = np.where(lev >= L, rng.integers(L, k_max + 1, n), lev).astype(np.int32)
    c = nb.Context(0)
    try:
        for with_scratch in (False, True):
            if with_scratch:      # a build above 16384 bodies leaves scratch behind
                nb.sched_build(dev(np.zeros(70000, np.int32)), 20, ctx=c)
            order, le = nb.sched_build(dev(lev), k_max, ctx=c)
            assert np.array_equal(host(order), want) and np.array_equal(host(le), ends)
            nb.sched_update(order, le, int(ends[L]), L, dev(new), k_max, ctx=c)
            got, e2 = host(order), host(le)
            assert np.array_equal(e2[L:], [(new >= q).sum() for q in range(L, k_max + 2)])
            assert np.array_equal(np.sort(got), np.arange(n))
            assert (np.diff(new[got[: ends[L]]]) <= 0).all()
    finally:
        c.close()
