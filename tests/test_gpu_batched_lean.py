"""A mixed ensemble runs where its memory holds the refinement's row lists but no
chunk partial."""
import numpy as np
import pytest

import oracle
import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import TOL_FP64, dev, host, row_rel_err, say

pytestmark = pytest.mark.gpu


def test_refinement_without_chunk_partials():
    """Few rows of 2^20 bodies: 247552 bytes hold the work list, the slots of 512
    splits a row and 128 partials, but not the 512 that a row's chunks are; every
    row is refined, to the bits of a call with room."""
    n, rows, cap = 1 << 20, 1, 8
    say("batched lean")
    rng = np.random.default_rng(20)
    x = rng.uniform(-1, 1, (3, n))
    v = rng.standard_normal((3, n))
    m = rng.uniform(0.5, 1.5, n) / n
    ib = np.array([12345], np.int32)
    rs2 = np.array([1e-4])
    args = ([0, n], [0, rows], dev(x), dev(v), dev(m), dev(ib), dev(rs2), cap, "mixed")
    free, tight = nb.Context(0), nb.Context(0)
    try:
        for c in (free, tight):
            c.set_mixed_tolerance(1e-30, 32.0)
        tight.set_scratch_limit(247552)
        a = nb.regular_force_batched(*args, ctx=free)
        b = nb.regular_force_batched(*args, ctx=tight)
        assert free.last_refined_rows() == rows and tight.last_refined_rows() == rows
        for k in (0, 1, 2, 4):
            assert np.array_equal(host(a[k]), host(b[k]))
        used = int(host(a[2])[0])
        assert used <= cap and np.array_equal(host(a[3])[:, :used], host(b[3])[:, :used])
    finally:
        free.close()
        tight.close()
    ref = oracle.regular(x, v, m, ib, rs2, cap)
    assert row_rel_err(host(b[0]), ref[0]).max() <= TOL_FP64
    assert row_rel_err(host(b[1]), ref[1]).max() <= TOL_FP64
