"""The pair-wise potential (each pair evaluated once) against the oracle at the
edges of its blocks and shapes, in panels under a scratch limit, and the plain
kernel where not even one block of entries fits; a coincident pair; replays."""
import numpy as np
import pytest
import torch

import oracle
import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

TOL = 1e-12   # the potential's terms share one sign


def _check(x, m, limit=0, rows=None):
    ctx = nb.Context(0)
    try:
        if limit:
            ctx.set_scratch_limit(limit)
        X, M = dev(x), dev(m)
        phi, U = nb.potential(X, M, ctx=ctx)
        again, U2 = nb.potential(X, M, ctx=ctx)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    p = host(phi)
    assert np.array_equal(p, host(again)) and host(U)[0] == host(U2)[0]
    if rows is None:
        oU, ophi = oracle.potential(x, m)
        assert abs(host(U)[0] - oU) <= TOL * abs(oU)
    else:
        ophi = oracle.potential_rows(x, m, rows)
        p = p[rows]
        full = host(phi)
        U0 = 0.5 * float(np.sum(m * full))
        assert abs(host(U)[0] - U0) <= TOL * abs(U0)
    assert (np.abs(p - ophi) <= TOL * np.abs(ophi)).all()


# one row per lane up to 8191 bodies, two above (four, and more waves: below)
@pytest.mark.parametrize("n", [2, 63, 64, 65, 128, 129, 1000, 4095, 4096, 4225, 8191, 8193,
                               16385])
def test_potential_block_edges(n):
    say(f"potential n={n}")
    x, _, m = W.plummer(np.random.default_rng(n), n, "kroupa")
    _check(x, m)


@pytest.mark.parametrize("n", [28671, 28672, 33025, 65536, 66561, 131073])
def test_potential_large_blocks(n):
    say(f"potential n={n}")
    x, _, m = W.plummer(np.random.default_rng(n), n, "kroupa")
    _check(x, m, rows=np.sort(np.random.default_rng(1).choice(n, 200, replace=False)).astype(np.int32))


@pytest.mark.parametrize("n,limit", [(2000, 20_000), (2000, 40_000), (5000, 400_000),
                                     (17000, 1_500_000)])
def test_potential_under_scratch_limit(n, limit):
    """20000 bytes hold no block of entries (the plain kernel); the others hold
    a few blocks per panel."""
    say(f"potential n={n} limit={limit}")
    x, _, m = W.plummer(np.random.default_rng(n + 7), n, "kroupa")
    _check(x, m, limit=limit)


def test_potential_coincident_pair():
    """Two bodies in one place: their potentials and the energy are not finite,
    every other body's is."""
    n = 300
    x, _, m = W.plummer(np.random.default_rng(5), n, "kroupa")
    x[:, 250] = x[:, 7]
    phi, U = nb.potential(dev(x), dev(m))
    p = host(phi)
    bad = ~np.isfinite(p)
    assert bad[7] and bad[250] and bad.sum() == 2 and not np.isfinite(host(U)[0])
