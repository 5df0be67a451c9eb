"""x_lo updated once per pair of iterations against once per iteration.

With the fused finish phase B adds two iterations' alpha q to x_lo in the
launches of odd parity; the three-launch iteration (WD_CG_UNFUSED=1) adds each
at once.  The sums are the same ones in the same order, so solutions and
reports agree bit for bit, with even-odd preconditioning too (whose fused
finish takes four launches per iteration instead of six).  Reliable updates every 7 iterations freeze fields
after launches of either parity and in the middle of chunks (the pending update
is applied by the reliable update, and the field resumes from either q buffer);
odd chunks end on a launch of parity 0; chunk 1 never pairs.  max_iter stops a
field half way through a pair."""
import os

import numpy as np
import pytest

import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


def _solve(g, m0, eta, p, unfused):
    if unfused:
        os.environ["WD_CG_UNFUSED"] = "1"
    try:
        x, reps, rc = wd.cg_solve_batch(g, m0, dev(eta), params=p, raise_on_error=False)
    finally:
        os.environ.pop("WD_CG_UNFUSED", None)
    return host(x), reps, rc


# plane blocks (64- and 70-site planes), site blocks; even-odd on half-plane
# blocks (64-site half planes) and on site blocks
@pytest.mark.parametrize("dims,eo", [((8, 8, 4, 6), 0), ((10, 7, 4, 4), 0), ((5, 6, 4, 5), 0),
                                     ((16, 8, 4, 4), 1), ((6, 4, 4, 6), 1)], ids=str)
@pytest.mark.parametrize("inner", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
def test_paired_x_update_is_bitwise_the_single_one(dims, eo, inner):
    m0 = 0.1
    U = wdgen.gauge_field(dims, 0.5, 1700 + sum(dims))
    eta = wdgen.mixed_sources(dims, 3, 2, 1800 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, recon12=True)
    for every, chunk, max_iter in ((7, 10, 20000), (7, 7, 20000), (20, 1, 20000), (0, 9, 15)):
        p = wd.cg_default_params(inner=inner, reliable_every=every, chunk=chunk, max_iter=max_iter, precondition=eo)
        say("paired x update", dims, eo, inner, every, chunk, max_iter)
        xa, ra, rca = _solve(g, m0, eta, p, unfused=False)
        xb, rb, rcb = _solve(g, m0, eta, p, unfused=True)
        assert rca == rcb == (wd.WD_OK if max_iter > 15 else wd.WD_ENOTCONV)
        assert np.array_equal(xa.view(np.uint64), xb.view(np.uint64))
        for a, b in zip(ra, rb):
            assert all(a[k] == b[k] for k in ("status", "iters", "reliable_updates", "true_rel_res", "iter_rel_res"))
    g.close()
