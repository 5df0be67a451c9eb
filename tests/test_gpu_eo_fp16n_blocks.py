"""Even-odd FP16N phases at the edges of the window in which they leave half-plane
blocks for site blocks (more than 256 and at most 512 half-planes): the kernels a
solve launches, by name, and the oracle's residual of its solutions."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, say
from test_gpu_operator_routes import kernels

pytestmark = pytest.mark.gpu
M0 = 0.2


@pytest.mark.parametrize("dims,nrhs,half", [((16, 16, 16, 16), 1, True), ((16, 16, 2, 130), 1, False),
                                            ((16, 16, 16, 16), 2, False), ((16, 16, 2, 258), 1, True)], ids=str)
def test_window(dims, nrhs, half):
    U = wdgen.gauge_field(dims, 0.5, 6500 + sum(dims))
    eta = wdgen.gaussian_source(dims, nrhs, 6550 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, precs=(wd.F64, wd.F16N))
    assert wd.shape_get(g, wd.F16N, nrhs, False, wd.FAMILY_CG_B)["xy_lds"] == 1
    p = wd.cg_default_params(inner=wd.F16N, precondition=wd.PRECOND_EO)
    out = []
    names = kernels(lambda: out.append(wd.cg_solve_batch(g, M0, dev(eta), params=p)))
    g.close()
    hops = {n for n in names if "k_eo_hop1<2" in n}
    say("even-odd FP16N", dims, nrhs, hops)
    assert hops and all(("false, true>" in n) == half for n in hops), hops   # the last argument: half-plane blocks
    x, reps, rc = out[0]
    assert rc == wd.WD_OK, reps
    assert np.all(oracle.true_residual(U, eta, host(x), dims, M0, -1) <= 1e-10 * 1.0000001)
