"""Ensembles of many small clusters stay whole once a few waves per CU are there,
and are split below that."""
import numpy as np
import pytest

import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("bodies,clusters,whole", [(250, 700, True), (300, 500, True),
                                                   (400, 300, True), (250, 60, False),
                                                   (600, 60, False)])
def test_small_clusters(bodies, clusters, whole, prec):
    """Lists are those of whole clusters, and so are the sums where the automatic
    plan leaves them whole."""
    say(f"{clusters} clusters of {bodies} {prec}")
    parts = [W.small_state(40 + k % 7, bodies, k_nn=20) for k in range(7)]
    parts = [parts[k % 7] for k in range(clusters)]
    off = bodies * np.arange(clusters + 1)
    ib = np.concatenate([np.arange(bodies) + o for o in off[:-1]]).astype(np.int32)
    args = (off, off, dev(np.concatenate([p["x"] for p in parts], 1)),
            dev(np.concatenate([p["v"] for p in parts], 1)),
            dev(np.concatenate([p["m"] for p in parts])), dev(ib),
            dev(np.concatenate([p["rs2"] for p in parts])))
    cap = 32
    ctx = nb.Context(0)
    try:
        got = [host(t) for t in nb.regular_force_batched(*args, cap, prec, ctx=ctx)]
        assert ("merge_rows=0 " in ctx.last_plan()) == whole, ctx.last_plan()
        ctx.set_plan(0, 0, 1)
        one = [host(t) for t in nb.regular_force_batched(*args, cap, prec, ctx=ctx)]
    finally:
        ctx.close()
    assert np.array_equal(got[2], one[2])
    used = np.arange(cap)[None, :] < np.minimum(one[2], cap)[:, None]
    assert np.array_equal(np.where(used, got[3], -1), np.where(used, one[3], -1))
    tol = 0.0 if whole else (1e-12 if prec == "fp64" else 1e-5)
    for k in (0, 1):
        d = np.linalg.norm(got[k] - one[k], axis=0)
        assert (d <= tol * np.linalg.norm(one[k], axis=0)).all()
