"""The one-pass adjoint at the edges of its row blocks, tiles and panels, with
duplicate rows, against the oracle; small panels under a scratch limit give the
same gradient; replays are bitwise equal."""
import numpy as np
import pytest
import torch

import oracle
import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

TOL = 1e-10   # per body, norm-wise, of the gradient's own scale (as the oracle tests)


def _err(got, ref):
    d = np.linalg.norm(np.atleast_2d(got - ref), axis=0)
    r = np.linalg.norm(np.atleast_2d(ref), axis=0)
    return (d / np.maximum(r, 1e-3 * r.max())).max()


def _case(n, n_i, seed, dup):
    s = W.small_state(500 + seed, n, k_nn=min(20, n - 1))
    rng = np.random.default_rng(seed)
    ib = rng.permutation(n)[:n_i].astype(np.int32) if not dup else \
        rng.integers(0, n, n_i).astype(np.int32)
    if dup:
        ib[: n_i // 3] = ib[0]          # one body with many rows
    return (s["x"], s["v"], s["m"], ib, s["rs2"][ib], rng.standard_normal((3, n_i)),
            rng.standard_normal((3, n_i)))


def _run(args, limit=0):
    ctx = nb.Context(0)
    try:
        if limit:
            ctx.set_scratch_limit(limit)
        d = [dev(t) for t in args]
        one = [host(t) for t in nb.regular_force_adjoint(*d, ctx=ctx)]
        two = [host(t) for t in nb.regular_force_adjoint(*d, ctx=ctx)]
    finally:
        ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(one, two))
    return one


@pytest.mark.parametrize("n,n_i,dup", [(63, 1, False), (64, 64, False), (65, 130, True),
                                       (257, 256, False), (1000, 257, True), (8192, 300, False),
                                       (8193, 255, False), (8300, 2049, True),
                                       (9000, 70, True), (9500, 1700, False)])
def test_adjoint_block_edges(n, n_i, dup):
    say(f"adjoint blocks n={n} n_i={n_i}")
    args = _case(n, n_i, n + n_i, dup)
    got = _run(args)
    ref = oracle.adjoint(*args)
    errs = [_err(g, r) for g, r in zip(got, ref)]
    say(f"  err {max(errs):.2e}")
    assert max(errs) <= TOL


@pytest.mark.parametrize("n,n_i,limit", [(3000, 2000, 600_000), (3000, 2000, 370_000),
                                         (9000, 5000, 1_300_000)])
def test_adjoint_under_scratch_limit(n, n_i, limit):
    """Room for a few row blocks, then for one with long body blocks (and, at
    the tightest, the bodies' row index in the mass gradient)."""
    say(f"adjoint limit n={n} n_i={n_i} {limit}")
    args = _case(n, n_i, 7, True)
    free, tight = _run(args), _run(args, limit)
    ref = oracle.adjoint(*args)
    for f, t, r in zip(free, tight, ref):
        assert _err(t, r) <= TOL and _err(f, r) <= TOL
