"""The adjoint where its entries cannot be allocated (here: while the stream is
being captured): smaller panels and longer body blocks in the scratch that is
there, down to 7 n + 12 n_i values."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("n,n_i,have", [(9000, 3000, 2100), (9500, 9500, 4000), (20000, 300, 4000)])
def test_adjoint_in_the_scratch_there_is(n, n_i, have):
    """A potential of 'have' bodies sets the scratch: 1 or 2 MiB, against 24, 45 and
    7 MB that the gradients would take (at the least 0.8, 1.4 and 1.1)."""
    say(f"captured adjoint n={n} n_i={n_i}")
    s = W.small_state(500 + n_i, n, k_nn=20)
    rng = np.random.default_rng(n)
    ib = rng.permutation(n)[:n_i].astype(np.int32)
    ib[: n_i // 50] = ib[0]
    wa, wj = rng.standard_normal((3, n_i)), rng.standard_normal((3, n_i))
    x, v, m, dib, rs2 = dev(s["x"]), dev(s["v"]), dev(s["m"]), dev(ib), dev(s["rs2"][ib])
    dwa, dwj = dev(wa), dev(wj)
    ctx, other = nb.Context(0), nb.Context(0)
    try:
        nb.potential(dev(s["x"][:, :have]), dev(s["m"][:have]), ctx=ctx)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            out = nb.regular_force_adjoint(x, v, m, dib, rs2, dwa, dwj, ctx=ctx)
        for k in range(3):
            dwa.copy_(torch.from_numpy(wa * (1.0 + k)))
            dwj.copy_(torch.from_numpy(wj * (1.0 + k)))
            g.replay()
            torch.cuda.synchronize()
            got = [host(t) for t in out]
            free = [host(t) for t in
                    nb.regular_force_adjoint(x, v, m, dib, rs2, dwa, dwj, ctx=other)]
            assert all(_err(a, b) <= 2 * TOL for a, b in zip(got, free))
        ref = oracle.adjoint(s["x"], s["v"], s["m"], ib, s["rs2"][ib], 3.0 * wa, 3.0 * wj)
        assert all(_err(a, b) <= TOL for a, b in zip(got, ref))
    finally:
        ctx.close()
        other.close()
