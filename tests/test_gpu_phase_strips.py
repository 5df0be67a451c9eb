"""The width of the z-strips in which CG phases A and B walk planes of 256 sites with
two planes per block: 8 for one or two fields, and for three or four where Lt is
at least 2 Lz, else 4; solves in either order pass the oracle's residual."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

CASES = [((16, 16, 16, 16), 4, 4), ((16, 16, 16, 16), 2, 8), ((16, 16, 16, 32), 4, 8), ((16, 16, 10, 32), 8, 4),
         ((16, 16, 16, 32), 3, 8)]


@pytest.mark.parametrize("dims,nrhs,strip", CASES, ids=str)
@pytest.mark.parametrize("prec", [wd.F32, wd.F16N], ids=["f32", "f16n"])
def test_strips(dims, nrhs, strip, prec):
    m0 = 0.2
    U = wdgen.gauge_field(dims, 0.5, 6200 + sum(dims))
    eta = wdgen.gaussian_source(dims, nrhs, 6250 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, precs=(wd.F64, prec))
    for fam in (wd.FAMILY_CG_A, wd.FAMILY_CG_B):
        sh = wd.shape_get(g, prec, nrhs, fam == wd.FAMILY_CG_A, fam)
        assert (sh["xy_planes"], sh["strip"]) == (2, strip), sh
    say("phase strips", dims, nrhs, prec)
    x, reps, rc = wd.cg_solve_batch(g, m0, dev(eta), params=wd.cg_default_params(inner=prec))
    assert rc == wd.WD_OK, reps
    assert np.all(oracle.true_residual(U, eta, host(x), dims, m0, -1) <= 1e-10 * 1.0000001)
    g.close()
