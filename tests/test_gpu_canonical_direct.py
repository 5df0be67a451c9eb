"""The operator on canonical fields without packed copies against pack, packed
operator, unpack: the same arithmetic per site, so bitwise the same fields.
Odd extents, a single-site and a full 256-site plane, extents of 1 and 2
(coinciding neighbours), more planes than an XCD round, both time boundaries,
and a plane of 272 sites, which keeps the packed path.  One case per precision
is also checked against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, rel, say

pytestmark = pytest.mark.gpu

CASES = [((13, 11, 3, 5), 3, -1), ((16, 16, 2, 2), 2, -1), ((1, 1, 3, 4), 2, 1), ((2, 1, 2, 2), 1, -1),
         ((5, 7, 6, 9), 7, 1), ((17, 16, 2, 3), 2, -1)]


@pytest.mark.parametrize("dims,nrhs,t_sign", CASES, ids=str)
@pytest.mark.parametrize("prec,recon12", [(wd.F64, False), (wd.F32, False), (wd.F32, True)],
                         ids=["f64", "f32", "f32r12"])
def test_canonical_operator_is_pack_operator_unpack(dims, nrhs, t_sign, prec, recon12):
    m0 = 0.07
    U = wdgen.gauge_field(dims, 0.5, 2100 + sum(dims))
    psi = wdgen.gaussian_source(dims, nrhs, 2150 + sum(dims))
    g = wd.Gauge(dev(U), dims, t_sign, recon12=recon12)
    x = dev(psi)
    for dagger in (False, True):
        say("canonical operator", dims, nrhs, prec, recon12, dagger)
        got = host(wd.dslash(g, m0, x, prec, dagger=dagger))
        packed = wd.dslash(g, m0, wd.pack_spinor(g, x, prec), prec, dagger=dagger, packed=True, nrhs=nrhs)
        ref = host(wd.unpack_spinor(g, packed, prec, nrhs))
        assert np.array_equal(got.view(np.uint64), ref.reshape(got.shape).view(np.uint64))
        want = oracle.dirac(U, psi, dims, m0, t_sign, dagger=dagger)
        assert rel(got, want) <= (1e-13 if prec == wd.F64 else 1e-5)
    g.close()
