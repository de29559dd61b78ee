"""Rows that name one body several times: their row sums reach the body in a fixed
order, through the work-group's look at all rows of the call."""
import numpy as np
import pytest

import oracle
import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

TOL = 1e-10   # as the adjoint's other tests


def _err(got, ref):
    d = np.linalg.norm(np.atleast_2d(got - ref), axis=0)
    r = np.linalg.norm(np.atleast_2d(ref), axis=0)
    return (d / np.maximum(r, 1e-3 * r.max())).max()


def _rows(kind, n, n_i, rng):
    if kind == "one":        # a single body, the last one
        return np.full(n_i, n - 1)
    if kind == "twice":      # every body of the block twice
        return rng.permutation(np.arange(n_i) // 2) % n
    if kind == "ends":       # the first and the last row name one body, the others are single
        ib = np.arange(n_i) % n
        ib[-1] = ib[0]
        return ib
    return rng.integers(-1, n + 1, n_i)   # anything, with indices out of range


# 64 bodies a work-group, 16 shares of whole runs of 64 rows, 8 runs at a time
@pytest.mark.parametrize("kind", ["one", "twice", "ends", "any"])
@pytest.mark.parametrize("n,n_i", [(63, 2), (64, 65), (65, 1024), (130, 1025), (1000, 8193),
                                   (300, 17000), (9000, 2500)])
def test_duplicate_rows(n, n_i, kind):
    say(f"duplicate rows n={n} n_i={n_i} {kind}")
    rng = np.random.default_rng(n + n_i)
    s = W.small_state(n, n, k_nn=min(20, n - 1))
    ib = _rows(kind, n, n_i, rng).astype(np.int32)
    ok = (ib >= 0) & (ib < n)
    rs2 = s["rs2"][np.where(ok, ib, 0)]
    args = (s["x"], s["v"], s["m"], ib, rs2, rng.standard_normal((3, n_i)),
            rng.standard_normal((3, n_i)))
    d = [dev(t) for t in args]
    one = [host(t) for t in nb.regular_force_adjoint(*d)]
    two = [host(t) for t in nb.regular_force_adjoint(*d)]
    assert all(np.array_equal(a, b) for a, b in zip(one, two))
    ref = oracle.adjoint(args[0], args[1], args[2], ib[ok], rs2[ok],
                         np.ascontiguousarray(args[5][:, ok]),
                         np.ascontiguousarray(args[6][:, ok]))
    assert all(_err(a, b) <= TOL for a, b in zip(one, ref))
