"""FP16N: the operator's default shapes and the blocks of the even-odd phases.

The operator takes the memory hops first and z-strips on planes of 224 sites or
more, and two planes per block from 8 fields on; every site agrees with the oracle
on the links and fields the GPU holds.  CG takes plane blocks on planes of more
than 192 sites from 128 of them on.  Even-odd phases change between half-plane and
site blocks at 256 and 1024 half-planes; every solution passes the oracle's
residual at the solver's tolerance 1e-10."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import sitecheck
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
M0 = 0.2


@pytest.mark.parametrize("dims,nrhs,hop,strip,planes",
                         [((16, 14, 4, 3), 8, 5, 4, 2), ((16, 14, 5, 3), 7, 5, 4, 1), ((223, 1, 6, 2), 8, 3, 0, 2),
                          ((16, 16, 3, 2), 8, 5, 4, 2), ((9, 7, 2, 3), 8, 3, 0, 2)], ids=str)
@pytest.mark.parametrize("dag", [False, True], ids=["D", "Ddag"])
def test_operator(dims, nrhs, hop, strip, planes, dag):
    U = wdgen.gauge_field(dims, 0.5, 2700 + sum(dims))
    psi = wdgen.gaussian_source(dims, nrhs, 2750 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, precs=(wd.F64, wd.F16N))
    sh = wd.shape_get(g, wd.F16N, nrhs, dag, 0)
    assert (sh["hop_order"], sh["strip"], sh["xy_planes"]) == (hop, strip, planes), sh
    say("fp16n operator", dims, nrhs, dag)
    got = host(wd.dslash(g, M0, dev(psi), prec=wd.F16N, dagger=dag))
    c, n = oracle.fp16n_encode(psi.reshape(nrhs, -1, 4, 3).astype(np.complex64))
    pin = oracle.fp16n_decode(c, n).astype(np.complex128).reshape(psi.shape)
    want = oracle.dirac(sitecheck.links_f16(U), pin, dims, M0, -1, dagger=dag)
    sitecheck.assert_sites(got, want, pin, M0, sitecheck.F16N_BOUND, "%s %d" % (dims, nrhs))
    g.close()


@pytest.mark.parametrize("dims,nrhs,eo", [((16, 16, 8, 16), 2, 1), ((16, 16, 2, 86), 3, 1), ((16, 8, 32, 16), 2, 1),
                                          ((16, 8, 2, 102), 5, 1), ((16, 14, 8, 8), 2, 0), ((16, 14, 7, 9), 2, 0)],
                         ids=str)
def test_solves(dims, nrhs, eo):
    U = wdgen.gauge_field(dims, 0.5, 2800 + sum(dims))
    eta = wdgen.gaussian_source(dims, nrhs, 2850 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, precs=(wd.F64, wd.F16N))
    if eo:   # plane blocks wherever the rule allows them
        for fam in (wd.FAMILY_CG_A, wd.FAMILY_CG_B):
            wd.shape_set(g, wd.F16N, nrhs, fam == wd.FAMILY_CG_A, fam, 256, 1, 1, 5, 1, 4, 0, 1)
    else:
        assert wd.shape_get(g, wd.F16N, nrhs, False, wd.FAMILY_CG_B)["xy_lds"] == (dims[2] * dims[3] * nrhs >= 128)
    p = wd.cg_default_params(inner=wd.F16N, precondition=wd.PRECOND_EO if eo else 0)
    say("fp16n solve", dims, nrhs, "even-odd" if eo else "")
    x, reps, rc = wd.cg_solve_batch(g, M0, dev(eta), params=p)
    assert rc == wd.WD_OK, reps
    assert np.all(oracle.true_residual(U, eta, host(x), dims, M0, -1) <= 1e-10 * 1.0000001)
    g.close()
