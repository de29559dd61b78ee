"""Split lengths of the batched ensemble: small ensembles cut their clusters
into splits of 64 to 1024 bodies, with items past the grid handed out by the
queue; clusters around the length that stays whole; the coarse splits where a
scratch limit has no room for the slots of the fine ones."""
import numpy as np
import pytest
import torch

import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import TOL_FP64, TOL_MIXED, check_lists, dev, host, row_rel_err, say

import oracle

pytestmark = pytest.mark.gpu
TOL = {"fp64": TOL_FP64, "mixed": TOL_MIXED}


def _ensemble(sizes, share, seed):
    rng = np.random.default_rng(seed)
    parts = [W.small_state(700 + c, n, k_nn=min(20, max(n - 1, 1))) for c, n in enumerate(sizes)]
    j_off = np.concatenate([[0], np.cumsum(sizes)])
    blocks = [rng.choice(n, max(1, int(n * share)), replace=False) for n in sizes]
    i_off = np.concatenate([[0], np.cumsum([len(b) for b in blocks])])
    return dict(x=np.concatenate([p["x"] for p in parts], 1),
                v=np.concatenate([p["v"] for p in parts], 1),
                m=np.concatenate([p["m"] for p in parts]), j_off=j_off, i_off=i_off,
                ib=np.concatenate([b + j for b, j in zip(blocks, j_off)]).astype(np.int32),
                rs2=np.concatenate([p["rs2"][b] for p, b in zip(parts, blocks)]))


def _args(E):
    return (E["j_off"], E["i_off"], dev(E["x"]), dev(E["v"]), dev(E["m"]), dev(E["ib"]),
            dev(E["rs2"]))


def _defined(out, cap):
    acc, jerk, cnt, lst, ovf = (host(t) for t in out)
    used = np.arange(cap)[None, :] < np.minimum(cnt, cap)[:, None]
    return acc, jerk, cnt, np.where(used, lst, -1), ovf


def _check(E, out, cap, tol, per_cluster=64):
    acc, jerk, cnt, lst, _ = (host(t) for t in out)
    for c in range(len(E["j_off"]) - 1):
        j0, j1 = E["j_off"][c], E["j_off"][c + 1]
        rows = np.arange(E["i_off"][c], E["i_off"][c + 1])
        if rows.size > per_cluster:
            rows = np.random.default_rng(c).choice(rows, per_cluster, replace=False)
        r = oracle.regular(E["x"][:, j0:j1], E["v"][:, j0:j1], E["m"][j0:j1], E["ib"][rows] - j0,
                           E["rs2"][rows], cap)
        check_lists(cnt[rows], lst[rows], r[2], np.where(r[3] >= 0, r[3] + j0, r[3]), cap)
        assert max(row_rel_err(acc[:, rows], r[0]).max(),
                   row_rel_err(jerk[:, rows], r[1]).max()) <= tol


def _splits(nc, length):
    """Splits of a cluster of nc bodies at the ensemble's split length."""
    if 4 * nc < 7 * length:
        return 1
    s = -(-nc // length)
    unit = min(length, 256)
    per = -(-(-(-nc // unit)) // s)
    return -(-nc // (per * unit))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes,share,length", [
    ((1000,), 1.0, 64), ((1, 63, 111, 112, 113, 129, 700), 1.0, 64), ((2048,) * 8, 1.0, 128),
    ((4000, 447, 448, 449) * 8, 0.35, 256), ((4100, 3000) * 4, 1.0, 512),
    ((9001,) * 4, 0.5, 512), ((4000, 300) * 20, 1.0, 1024)])
def test_split_lengths(sizes, share, length, prec):
    """Against the oracle, and lists equal to those of unsplit clusters; replays
    give the same bits."""
    say(f"split length {length} of {len(sizes)} clusters {prec}")
    E = _ensemble(sizes, share, len(sizes))
    cap = 24
    ctx = nb.Context(0)
    try:
        args = _args(E)
        out = nb.regular_force_batched(*args, cap, prec, ctx=ctx)
        plan = ctx.last_plan()
        rows = np.diff(E["i_off"])
        S = [_splits(n, length) for n in sizes]
        packed = "bodies=packed" in plan
        per = 64 if packed else 256
        assert f"items={sum(-(-r // per) * s for r, s in zip(rows, S))} " in plan, plan
        assert f"merge_rows={sum(int(r) for r, s in zip(rows, S) if s > 1)} " in plan, plan
        first = _defined(out, cap)
        again = nb.regular_force_batched(*args, cap, prec, out=out, ctx=ctx)
        for a, b in zip(first, _defined(again, cap)):
            assert np.array_equal(a, b)
        _check(E, out, cap, TOL[prec])
        ctx.set_plan(0, 0, 1)
        one = _defined(nb.regular_force_batched(*args, cap, prec, ctx=ctx), cap)
        for k in (2, 3, 4):
            assert np.array_equal(first[k], one[k])
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_fine_splits_without_room(prec):
    """A scratch limit with room for the whole clusters but not for the slots
    of fine splits: the call is accepted and runs whole clusters."""
    say(f"batched scratch limit {prec}")
    sizes, cap = (1500,) * 3, 24
    E = _ensemble(sizes, 1.0, 3)
    ctx = nb.Context(0)
    try:
        args = _args(E)
        fine = nb.regular_force_batched(*args, cap, prec, ctx=ctx)
        assert f"merge_rows={sum(sizes)} " in ctx.last_plan()
        ctx.set_plan(0, 0, 1)
        one = nb.regular_force_batched(*args, cap, prec, ctx=ctx)
        a = _defined(fine, cap)
        b = _defined(one, cap)
        ctx2 = nb.Context(0)
        try:
            ctx2.set_scratch_limit(2 << 20)
            small = _defined(nb.regular_force_batched(*args, cap, prec, ctx=ctx2), cap)
            assert "merge_rows=0 " in ctx2.last_plan(), ctx2.last_plan()
        finally:
            ctx2.close()
        for x, y in zip(small, b):
            assert np.array_equal(x, y)
        for k in (2, 3, 4):
            assert np.array_equal(a[k], b[k])
    finally:
        ctx.close()
