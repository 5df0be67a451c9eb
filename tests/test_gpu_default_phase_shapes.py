"""Default launch shapes of CG phases A and B by plane size, and solves with them.

FP16N takes plane blocks for one field, or where a plane fills 7/8 of its
wavefronts and there are enough planes, else site blocks; FP32 and FP16N take
two planes per block for 256-site planes whose blocks come in whole rounds of
the compute units.  Each solution must pass the oracle's residual at the
solver's tolerance 1e-10."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


# dims, fields, precision, plane-blocked, planes per block
CASES = [((16, 16, 16, 32), 1, wd.F16N, 1, 2), ((16, 16, 16, 32), 1, wd.F32, 1, 2),   # 256 blocks: one round
         ((16, 16, 16, 16), 1, wd.F16N, 1, 1),                                          # half a round
         ((16, 16, 7, 8), 2, wd.F16N, 0, 1), ((16, 16, 7, 8), 2, wd.F32, 1, 1),         # odd Lz, few planes
         ((14, 16, 8, 24), 4, wd.F16N, 1, 1), ((14, 14, 8, 24), 4, wd.F16N, 0, 1),      # 7/8 of the lanes, and less
         ((8, 8, 24, 32), 1, wd.F16N, 1, 1), ((8, 8, 8, 32), 3, wd.F16N, 0, 1)]         # 64-site planes


@pytest.mark.parametrize("dims,nrhs,prec,xy,planes", CASES, ids=str)
def test_default_phase_shapes(dims, nrhs, prec, xy, planes):
    m0 = 0.2
    U = wdgen.gauge_field(dims, 0.5, 1900 + sum(dims))
    eta = wdgen.gaussian_source(dims, nrhs, 1950 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, precs=(wd.F64, prec))
    for fam in (wd.FAMILY_CG_A, wd.FAMILY_CG_B):
        sh = wd.shape_get(g, prec, nrhs, fam == wd.FAMILY_CG_A, fam)
        assert (sh["xy_lds"], sh["xy_planes"]) == (xy, planes), sh
    say("default phase shapes", dims, nrhs, prec)
    x, reps, rc = wd.cg_solve_batch(g, m0, dev(eta), params=wd.cg_default_params(inner=prec))
    assert rc == wd.WD_OK, reps
    assert np.all(oracle.true_residual(U, eta, host(x), dims, m0, -1) <= 1e-10 * 1.0000001)
    g.close()
