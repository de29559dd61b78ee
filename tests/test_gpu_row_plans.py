"""Row-per-lane plans.  The scalar-operand pass over the packed j-set (large
blocks): lists and sums bit-identical to the LDS row pass with the same splits,
at ragged sizes, and the LDS pass where the packed bodies find no room.  Short
splits of small blocks: against the oracle and the unsplit launch."""
import numpy as np
import pytest
import torch

import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import TOL_FP64, TOL_MIXED, compare_force, dev, host, say

pytestmark = pytest.mark.gpu

TOL = {"fp64": TOL_FP64, "mixed": TOL_MIXED}


def _defined(out, cap):
    acc, jerk, cnt, lst, ovf = (host(t) for t in out)
    used = np.arange(cap)[None, :] < np.minimum(cnt, cap)[:, None]
    return acc, jerk, cnt, np.where(used, lst, -1), ovf


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_i,splits", [(65537, 2049, 7), (65567, 4096, 1), (140001, 1000, 0),
                                          (30011, 4600, 3), (65535, 2100, 1),
                                          (16390, 4300, 5)])
def test_packed_equals_lds_pass(n, n_i, splits, prec):
    """n and n_i one past and one short of the runs and tiles; several splits,
    one (direct stores), and the automatic count; duplicate rows, a bad index
    and rows without neighbours."""
    say(f"packed n={n} n_i={n_i} splits={splits} {prec}")
    rng = np.random.default_rng(n)
    s = W.small_state(300 + n_i, n, k_nn=24)
    ib = rng.choice(n, n_i, replace=False).astype(np.int32)
    ib[5] = ib[6]
    rs2 = s["rs2"][ib].copy()
    rs2[::101] = 0.0
    ib[n_i - 1] = n          # out of range: a zero row and a status bit
    cap = 20
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2), cap, prec)
    ctx = nb.Context(0)
    try:
        st = [torch.zeros(1, dtype=torch.int32, device="cuda") for _ in range(3)]
        ctx.set_plan(1, 1, splits)
        packed = nb.regular_force(*args, status=st[0], ctx=ctx)
        assert "bodies=packed" in ctx.last_plan(), ctx.last_plan()
        k = int(ctx.last_plan().split("splits=")[1].split()[0])
        ctx.set_plan(1, 2, k)    # two rows per lane: the LDS kernel
        lds = nb.regular_force(*args, status=st[1], ctx=ctx)
        assert "packed" not in ctx.last_plan()
        ctx.set_plan(1, 1, k)
        # room for the split slots and the refinement, but not for the bodies
        ctx2 = nb.Context(0)
        try:
            ctx2.set_plan(1, 1, k)
            ctx2.set_scratch_limit(64 * n - 1 if k == 1 else
                                   k * n_i * 452 + n_i * 12 + (n // 8192 + 1) * n_i * 48 + 65536)
            small = nb.regular_force(*args, status=st[2], ctx=ctx2)
            plan = ctx2.last_plan()
        finally:
            ctx2.close()
        torch.cuda.synchronize()
        a, b, c = (_defined(o, cap) for o in (packed, lds, small))
        for x, y, z in zip(a, b, c):
            assert np.array_equal(x, y) and np.array_equal(x, z)
        assert "packed" not in plan, plan
        assert len({int(t.item()) for t in st}) == 1 and int(st[0].item()) & nb.STATUS_BAD_INDEX
        assert not host(packed[0])[:, n_i - 1].any() and a[2][n_i - 1] == 0
        rows = rng.choice(n_i - 1, 96, replace=False)
        compare_force(packed, s["x"], s["v"], s["m"], ib, rs2, cap, TOL[prec], rows=rows)
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_i,mapping,step", [
    (33, 33, 2, 0), (65, 64, 3, 32), (1000, 250, 1, 32), (1024, 1024, 1, 32), (4033, 300, 3, 32),
    (4096, 1000, 1, 32), (4097, 1000, 1, 64), (9000, 700, 1, 64)])
def test_short_splits(n, n_i, mapping, step, prec):
    """Automatic plans of small blocks cut the j-set into splits of 32 bodies
    up to one wave per SIMD (in splits of 64), and of 64 above: a part of a
    256-body tile in mapping 1, a ragged last split."""
    say(f"short splits n={n} n_i={n_i} {prec}")
    rng = np.random.default_rng(n + 1)
    s = W.small_state(400 + n_i, n, k_nn=20)
    ib = rng.choice(n, n_i, replace=False).astype(np.int32)
    rs2 = s["rs2"][ib]
    cap = 24
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2), cap, prec)
    ctx = nb.Context(0)
    try:
        auto = nb.regular_force(*args, ctx=ctx)
        plan = ctx.last_plan()
        assert f"mapping={mapping}" in plan, plan
        if step:
            assert f"split_len={step}" in plan and f"splits={-(-n // step)}" in plan, plan
        ctx.set_plan(1, 1, 1)
        one = nb.regular_force(*args, ctx=ctx)
        torch.cuda.synchronize()
        for x, y in zip(_defined(auto, cap)[2:], _defined(one, cap)[2:]):
            assert np.array_equal(x, y)
        compare_force(auto, s["x"], s["v"], s["m"], ib, rs2, cap, TOL[prec])
    finally:
        ctx.close()


def test_near_queue_rows_do_not_depend_on_their_wave():
    """Mixed packed pass at n >= 2^18, where near pairs wait in queues: rows
    with no, few and far more near pairs than a queue holds, against the
    oracle, and the same bits for a row whatever rows share its wave."""
    n, n_i, cap = (1 << 18) + 77, 640, 16
    say(f"near queue n={n}")
    rng = np.random.default_rng(18)
    x = rng.uniform(-1, 1, (3, n))
    v = rng.standard_normal((3, n))
    m = rng.uniform(0.5, 1.5, n) / n
    ib = rng.choice(n, n_i, replace=False).astype(np.int32)
    r = 2.0 * (8.0 / n) ** (1 / 3) * np.ones(n_i)     # about 4 neighbours, 30 near pairs
    r[::7] = 0.2                                      # about 1000 near pairs
    r[::31] = 1.0                                     # most of the bodies
    r[::13] = 0.0
    rs2 = (0.25 * r) ** 2 * np.where(r == 1.0, 16, 1)
    X, V, M = dev(x), dev(v), dev(m)
    ctx = nb.Context(0)
    try:
        ctx.set_plan(1, 1, 3)
        one = nb.regular_force(X, V, M, dev(ib), dev(rs2), cap, "mixed", ctx=ctx)
        assert "bodies=packed" in ctx.last_plan(), ctx.last_plan()
        p = rng.permutation(n_i)
        two = nb.regular_force(X, V, M, dev(ib[p]), dev(rs2[p]), cap, "mixed", ctx=ctx)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    a, b = _defined(one, cap), _defined(two, cap)
    for k in (0, 1):
        assert np.array_equal(a[k][:, p], b[k])
    for k in (2, 3):
        assert np.array_equal(a[k][p], b[k])
    rows = np.concatenate([np.arange(0, 64), rng.choice(n_i, 32, replace=False)])
    compare_force(one, x, v, m, ib, rs2, cap, TOL_MIXED, rows=rows)


@pytest.mark.parametrize("n,rows", [(300, 300), (2048, 41), (2048, 2048), (2049, 200)])
def test_refined_rows_of_one_chunk(n, rows):
    """Refinement of every row: a row of one chunk (2048 bodies) goes straight
    to the outputs, longer ones through chunk partials; single and batched
    calls give the same bits, at FP64 accuracy, call after call."""
    say(f"refinement n={n} rows={rows}")
    rng = np.random.default_rng(n + rows)
    s = W.small_state(800 + rows, n, k_nn=20)
    ib = rng.choice(n, rows, replace=False).astype(np.int32)
    rs2 = s["rs2"][ib]
    cap = 24
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2))
    ctx = nb.Context(0)
    try:
        ctx.set_plan(1, 1, 0)    # the mixed kernel at every block size
        ctx.set_mixed_tolerance(1e-30, 32.0)
        runs = []
        for _ in range(2):
            res = nb.regular_force(*args, cap, "mixed", ctx=ctx)
            assert ctx.last_refined_rows() == rows
            runs.append([host(t) for t in res])
        compare_force(res, s["x"], s["v"], s["m"], ib, rs2, cap, TOL_FP64)
        bat = nb.regular_force_batched([0, n], [0, rows], *args, cap, "mixed", ctx=ctx)
        assert ctx.last_refined_rows() == rows
        for k in (0, 1):
            assert np.array_equal(runs[0][k], runs[1][k])
            assert np.array_equal(host(bat[k]), runs[0][k])
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_i,mapping", [(1030, 70, 3), (1030, 1030, 1), (40961, 3300, 1)])
def test_rare_pairs_by_runs(n, n_i, mapping, prec):
    """Passes over less than 65536 bodies settle neighbours once per 32 bodies:
    the same lists and bits as the passes that do it at once (two rows per
    lane), with rows whose radius takes in everything (also the padding), a
    few, or nothing, and two bodies so close that their squared distance is
    below the smallest normal float (a near pair of a row without radius)."""
    say(f"rare pairs by runs n={n} n_i={n_i} {prec}")
    rng = np.random.default_rng(n + n_i)
    s = W.small_state(900 + n_i, n, k_nn=20)
    x = s["x"].copy()
    ib = rng.permutation(n)[:n_i].astype(np.int32)
    x[:, ib[0]] = 0.0
    x[:, ib[1]] = [3e-20, 0.0, 0.0]
    rs2 = s["rs2"][ib].copy()
    rs2[:2] = 0.0
    rs2[2::17] = np.inf
    rs2[3::17] = (2.0 * np.abs(x).max()) ** 2
    rs2[4::17] = 0.0
    cap = 40
    args = (dev(x), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2), cap, prec)
    ctx = nb.Context(0)
    try:
        ctx.set_mixed_tolerance(0.0)   # no refinement: the sums of the pass itself
        runs = nb.regular_force(*args, ctx=ctx)
        plan = ctx.last_plan()
        assert f"mapping={mapping}" in plan and "rows_per_lane=1" in plan, plan
        assert ("packed" in plan) == (n * n_i > 1 << 27), plan
        k = 3
        ctx.set_plan(mapping, 1, k)
        runs_k = nb.regular_force(*args, ctx=ctx)
        ctx.set_plan(1, 2, k)
        once = nb.regular_force(*args, ctx=ctx)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    a, b, c = (_defined(o, cap) for o in (runs, runs_k, once))
    for i in (2, 3, 4):
        assert np.array_equal(a[i], c[i]) and np.array_equal(b[i], c[i])
    if mapping == 1:     # the same splits: the same bits
        assert np.array_equal(b[0], c[0], equal_nan=True)
        assert np.array_equal(b[1], c[1], equal_nan=True)
    assert (a[2][2::17] == n - 1).all() and (a[2][4::17] == 0).all()
    fin = np.setdiff1d(np.arange(n_i), [0, 1])   # rows 0 and 1: a pair at 3e-20
    compare_force(runs, x, s["v"], s["m"], ib, rs2, cap, TOL[prec],
                  rows=rng.choice(fin, min(48, fin.size), replace=False))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_even_splits_of_packed_launches(prec):
    """Automatic plans of mid-size blocks take a split length that fills the CUs
    evenly (a multiple of 64 bodies, 512 to 1024): lists as with other splits,
    sums against the oracle."""
    n, n_i, cap = 131075, 4100, 24
    say(f"even splits n={n} n_i={n_i} {prec}")
    rng = np.random.default_rng(n)
    s = W.small_state(950, n, k_nn=20)
    ib = rng.choice(n, n_i, replace=False).astype(np.int32)
    rs2 = s["rs2"][ib]
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2), cap, prec)
    ctx = nb.Context(0)
    try:
        auto = nb.regular_force(*args, ctx=ctx)
        plan = ctx.last_plan()
        length = int(plan.split("split_len=")[1].split()[0])
        assert "bodies=packed" in plan and length % 64 == 0 and 512 < length <= 1024, plan
        ctx.set_plan(1, 1, 5)
        five = nb.regular_force(*args, ctx=ctx)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    for x, y in zip(_defined(auto, cap)[2:], _defined(five, cap)[2:]):
        assert np.array_equal(x, y)
    compare_force(auto, s["x"], s["v"], s["m"], ib, rs2, cap, TOL[prec],
                  rows=rng.choice(n_i, 64, replace=False))


@pytest.mark.parametrize("splits", [256, 257, 512, 513, 1024, 1025, 2048, 2049])
def test_merge_batches(splits):
    """The work-group merge at the edges of its batches: short, long and
    overflowed segments, a full list, rows without neighbours."""
    n, n_i, cap = 64 * (2048 + splits % 2) - 5, 66, 700
    say(f"merge of {splits} splits")
    rng = np.random.default_rng(splits)
    s = W.small_state(960, n, k_nn=40)
    ib = rng.choice(n, n_i, replace=False).astype(np.int32)
    rs2 = s["rs2"][ib].copy()
    rs2[::5] *= 9.0
    rs2[1::11] = 0.0
    rs2[2::13] = (4.0 * np.abs(s["x"]).max()) ** 2
    args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(rs2), cap, "fp64")
    ctx = nb.Context(0)
    try:
        ctx.set_plan(3, 1, splits)
        got = nb.regular_force(*args, ctx=ctx)
        k = int(ctx.last_plan().split("splits=")[1].split()[0])
        assert k == splits, ctx.last_plan()
        ctx.set_plan(3, 1, 1)
        one = nb.regular_force(*args, ctx=ctx)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    for x, y in zip(_defined(got, cap)[2:], _defined(one, cap)[2:]):
        assert np.array_equal(x, y)
    some = np.setdiff1d(np.arange(n_i), np.arange(2, n_i, 13))   # rows with a regular force
    compare_force(got, s["x"], s["v"], s["m"], ib, rs2, cap, TOL_FP64, rows=some[:32])
