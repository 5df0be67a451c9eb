"""Cache policies of phases A and B's streams at the size where they change: the
fields of an iteration (r, q twice, x_lo) just below and just above 256 MB
(and FP64 below 128 MB).

Planes of 240 sites (the last wavefront partly idle), with and without the
reconstruct-12 links.  The first and the last solution pass the oracle's residual
at the solver's tolerance, and all agree with site blocks, one hop at a time,
within kappa(D) (2 tol)."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, rel, say

pytestmark = pytest.mark.gpu
TOL = 1e-10
DIMS = (16, 15, 12, 12)
M0 = 0.5


@pytest.mark.parametrize("inner,r12,nrhs", [(wd.F64, False, 4), (wd.F64, False, 10), (wd.F64, False, 11), (wd.F32, True, 20),
                                            (wd.F32, False, 20), (wd.F32, True, 21), (wd.F32, False, 21),
                                            (wd.F16N, False, 30), (wd.F16N, False, 31)],
                         ids=["f64-4", "f64-10", "f64-11", "f32r12-20", "f32-20", "f32r12-21", "f32-21", "f16n-30", "f16n-31"])
def test_stream_policies(inner, r12, nrhs):
    bytes_per_site = {wd.F64: 4 * 192, wd.F32: 4 * 96, wd.F16N: 3 * 52 + 96}[inner]
    below = bytes_per_site * int(np.prod(DIMS)) * nrhs <= 256 << 20
    assert below == (nrhs in (4, 10, 20, 30))
    U = wdgen.gauge_field(DIMS, 0.4, 2600)
    eta = wdgen.gaussian_source(DIMS, nrhs, 2650)
    g = wd.Gauge(dev(U), DIMS, -1, recon12=r12)
    p = wd.cg_default_params(inner=inner, reliable_every=0 if inner == wd.F64 else 50)
    sols = []
    for xy in (1, 0):
        for fam, dag in ((wd.FAMILY_CG_A, True), (wd.FAMILY_CG_B, False)):
            wd.shape_set(g, inner, nrhs, dag, fam, 256, 1, 1, 5 if xy else 1, 1, 0, 0, xy)
        say("stream policy", DIMS, nrhs, inner, r12, "planes" if xy else "sites")
        x, reps, rc = wd.cg_solve_batch(g, M0, dev(eta), params=p)
        assert rc == wd.WD_OK, reps
        sols.append(host(x))
    ends = [0, nrhs - 1]
    assert np.all(oracle.true_residual(U, eta[ends], sols[0][ends], DIMS, M0, -1) <= TOL * 1.0000001)
    for i in range(nrhs):
        assert rel(sols[0][i], sols[1][i]) <= (8.0 + M0) / M0 * 2 * TOL
    g.close()
