"""Where site-blocked CG phases update x_lo in pairs of iterations: FP32 while r, the
two q buffers and x_lo fit 24 MB (65536 sites times fields), FP64 beyond 256 MB
(349525), FP16N beyond 327680 sites times fields.
Paired or single, fused finish or separate launches, the arithmetic is the same:
the solutions and reports equal those of WD_CG_UNFUSED=1 bit for bit, on both sides
of each limit and with shapes set for one phase only (which run the separate
launches where the phases would pair differently).  Chunks of 7 iterations and
reliable updates after 9 cut pairs in half."""
import os

import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
M0, TOL = 0.2, 1e-10


def _check(U, eta, dims, inner, **kw):
    g = wd.Gauge(dev(U), dims, -1, recon12=inner == wd.F32)
    out = {}
    for unfused in (False, True):
        if unfused:
            os.environ["WD_CG_UNFUSED"] = "1"
        try:
            say("site pairing", dims, eta.shape[0], inner, kw, "unfused" if unfused else "")
            x, reps, rc = wd.cg_solve_batch(g, M0, dev(eta), params=wd.cg_default_params(inner=inner, **kw))
        finally:
            os.environ.pop("WD_CG_UNFUSED", None)
        assert rc == wd.WD_OK, reps
        out[unfused] = (host(x), [(r["iters"], r["true_rel_res"], r["reliable_updates"]) for r in reps])
    g.close()
    assert out[False][1] == out[True][1]
    assert np.array_equal(out[False][0].view(np.uint64), out[True][0].view(np.uint64))
    assert np.all(oracle.true_residual(U, eta, out[False][0], dims, M0, -1) <= TOL * 1.0000001)


@pytest.mark.parametrize("inner", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
@pytest.mark.parametrize("nrhs", [6, 7, 34, 35, 37, 38])   # 9408 sites: 56448, 65856; 319872, 329280; 348096, 357504
def test_both_sides_of_the_limits(nrhs, inner):
    dims = (4, 14, 12, 14)
    U = wdgen.gauge_field(dims, 0.4, 6000)
    eta = wdgen.gaussian_source(dims, nrhs, 6001)
    _check(U, eta, dims, inner, reliable_every=0 if inner == wd.F64 else 50)
    _check(U, eta, dims, inner, reliable_every=9, chunk=7)


@pytest.mark.parametrize("inner", [wd.F64, wd.F32], ids=["f64", "f32"])
@pytest.mark.parametrize("fam,dag", [(wd.FAMILY_CG_A, True), (wd.FAMILY_CG_B, False)], ids=["A", "B"])
@pytest.mark.parametrize("shape", [dict(hop_order=3), dict(hop_order=3, rhs_per_thread=2), dict(hop_order=1)], ids=str)
def test_a_shape_for_one_phase(shape, fam, dag, inner):
    dims = (8, 9, 4, 3)     # the other phase on plane blocks
    nrhs = 3 + shape.get("rhs_per_thread", 1) + 2 * shape["hop_order"] + 8 * (fam == wd.FAMILY_CG_A)
    U = wdgen.gauge_field(dims, 0.4, 6100)
    eta = wdgen.gaussian_source(dims, nrhs, 6101)
    g = wd.Gauge(dev(U), dims, -1)
    wd.shape_set(g, inner, nrhs, dag, fam, 256, **shape)
    g.close()
    _check(U, eta, dims, inner, reliable_every=9, chunk=7)
