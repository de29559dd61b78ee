"""The potential where its entries cannot be allocated (here: while the stream is
being captured): smaller panels, or the plain kernel, in the scratch that is
there."""
import numpy as np
import pytest
import torch

import oracle
import paper_1504_03687_amd as nb
import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

TOL = 1e-12   # as the potential's other tests


@pytest.mark.parametrize("n,have", [(16385, 8192), (16385, 4000), (3000, 1200)])
def test_potential_in_the_scratch_there_is(n, have):
    """An earlier potential of 'have' bodies sets the scratch (4.3 MB for 8192,
    2.1 MB for 4000, 1 MB for 1200: the bodies below need 17 and 1.2 MB in one
    panel)."""
    say(f"captured potential n={n} scratch of {have}")
    x, _, m = W.plummer(np.random.default_rng(n), n, "kroupa")
    X, M = dev(x), dev(m)
    ctx = nb.Context(0)
    other = nb.Context(0)
    try:
        nb.potential(dev(x[:, :have]), dev(m[:have]), ctx=ctx)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            phi, U = nb.potential(X, M, ctx=ctx)
        for k in range(3):
            M.copy_(torch.from_numpy(m * (1.0 + k)))
            g.replay()
            torch.cuda.synchronize()
            oU, ophi = oracle.potential(x, m * (1.0 + k))
            assert (np.abs(host(phi) - ophi) <= TOL * np.abs(ophi)).all()
            assert abs(host(U)[0] - oU) <= TOL * abs(oU)
            p2, U2 = nb.potential(X, M, ctx=other)
            assert (np.abs(host(p2) - ophi) <= TOL * np.abs(ophi)).all()
    finally:
        ctx.close()
        other.close()
