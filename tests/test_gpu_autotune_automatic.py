"""Tuned tables may say that the automatic plan was the fastest: such an entry is
kept in the file and leaves every block its own automatic plan."""
import numpy as np
import pytest

import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import dev, say

pytestmark = pytest.mark.gpu


def _plans(ctx, s, n, blocks):
    out = []
    for n_i in blocks:
        ib = np.random.default_rng(n_i).choice(n, n_i, replace=False).astype(np.int32)
        args = (dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(s["rs2"][ib]), 32)
        for prec in ("fp64", "mixed"):
            nb.regular_force(*args, prec, ctx=ctx)
            out.append(ctx.last_plan())
    return out


def test_automatic_entries(tmp_path):
    n, blocks = 16384, (20, 300, 9000, 16384)
    say("automatic entries of a tuned table")
    s = W.small_state(31, n, k_nn=20)
    path = tmp_path / "tune.txt"
    table = "nbreg-tune 2\n" + "".join(f"{p} 14 {b} 0 0 0 0\n" for p in (0, 1) for b in range(15))
    path.write_text(table)
    auto, tuned, again = nb.Context(0), nb.Context(0), nb.Context(0)
    try:
        want = _plans(auto, s, n, blocks)
        nb.autotune(n, str(path), ctx=tuned)
        assert path.read_text() == table      # loaded, not timed again
        assert _plans(tuned, s, n, blocks) == want
        # and a table that the tuner wrote is read back to the same plans
        nb.autotune(n, str(path), force=True, ctx=tuned)
        rows = [line.split() for line in path.read_text().splitlines()[1:]]
        assert {(r[0], r[2]) for r in rows} == {(str(p), str(b)) for p in (0, 1) for b in range(15)}
        say(f"  automatic: {sum(r[3] == '0' for r in rows)} of {len(rows)} buckets")
        nb.autotune(n, str(path), ctx=again)
        assert _plans(again, s, n, blocks) == _plans(tuned, s, n, blocks)
    finally:
        for c in (auto, tuned, again):
            c.close()
