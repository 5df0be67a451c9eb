"""Direction-split phases A and B (four threads per site, for launches of at most
one plane block per compute unit) against site blocks with one hop at a time.

Planes at the edges of a group's wavefronts (64, 65, 128, 129 sites), of the
64 KB of LDS (225 sites fit in FP32, 228 do not; FP64 112 and 114) and of the
block count (256, 257 blocks; 512 and 513 of 64 sites).  Every solution passes
the oracle's residual at the solver's tolerance and agrees with the site blocks'
within kappa(D) (2 tol); in FP64 without reliable updates the iteration counts
agree to rounding."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, rel, say

pytestmark = pytest.mark.gpu
TOL = 1e-10

CASES = [((8, 8, 2, 3), 2), ((13, 5, 3, 2), 3), ((16, 8, 2, 2), 1), ((43, 3, 2, 2), 2), ((15, 15, 2, 2), 1),
         ((19, 12, 2, 2), 1), ((16, 7, 3, 2), 2), ((19, 6, 3, 2), 2), ((14, 5, 8, 16), 2), ((14, 5, 1, 257), 1),
         ((8, 8, 8, 16), 4), ((8, 8, 1, 171), 3)]


@pytest.mark.parametrize("dims,nrhs", CASES, ids=str)
@pytest.mark.parametrize("inner", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
def test_split_phases(dims, nrhs, inner):
    m0 = 0.2
    U = wdgen.gauge_field(dims, 0.4, 2400 + sum(dims))
    eta = wdgen.gaussian_source(dims, nrhs, 2450 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, recon12=inner == wd.F32)
    p = wd.cg_default_params(inner=inner, reliable_every=0 if inner == wd.F64 else 50)
    sols, iters = {}, {}
    for xy in (1, 0):
        for fam, dag in ((wd.FAMILY_CG_A, True), (wd.FAMILY_CG_B, False)):
            wd.shape_set(g, inner, nrhs, dag, fam, 256, 1, 1, 5 if xy else 1, 1, 0, 0, xy)
        say("split phases", dims, nrhs, inner, "planes" if xy else "sites")
        x, reps, rc = wd.cg_solve_batch(g, m0, dev(eta), params=p)
        assert rc == wd.WD_OK, reps
        sols[xy], iters[xy] = host(x), [r["iters"] for r in reps]
        assert np.all(oracle.true_residual(U, eta, sols[xy], dims, m0, -1) <= TOL * 1.0000001)
    for i in range(nrhs):
        assert rel(sols[1][i], sols[0][i]) <= (8.0 + m0) / m0 * 2 * TOL
        if inner == wd.F64:
            assert abs(iters[1][i] - iters[0][i]) <= 2, (iters, i)
    g.close()
