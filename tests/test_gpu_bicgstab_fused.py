"""The fused BiCGSTAB iteration (four launches, reductions completed by the
launch that needs them, rho of the new residual formed before it) against the
five-stage one with finish launches (WD_CG_UNFUSED=1, or a workspace without the
fused iteration's pieces).  Both must pass the oracle's residual at the solver's
tolerance; their solutions agree within kappa(D) (2 tol), and in FP64 without
reliable updates both iterate the same recurrence to rounding.  Point sources
meet the near breakdown after one iteration; a zero source and a field that
max_iter stops keep their reports; chunks of 1 and 7 iterations cross the
trailing finish in every state."""
import os

import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, rel, say

pytestmark = pytest.mark.gpu
TOL = 1e-10


def _solve(g, m0, eta, p, unfused=False, ws=None):
    if unfused:
        os.environ["WD_CG_UNFUSED"] = "1"
    try:
        x, reps, rc = wd.cg_solve_batch(g, m0, dev(eta), params=p, ws=ws, raise_on_error=False)
    finally:
        os.environ.pop("WD_CG_UNFUSED", None)
    return host(x), reps, rc


@pytest.mark.parametrize("inner", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
@pytest.mark.parametrize("dims", [(8, 8, 4, 6), (13, 5, 4, 3), (4, 4, 4, 4), (3, 2, 2, 2)], ids=str)
def test_fused_iteration(dims, inner):
    m0 = 0.1
    U = wdgen.gauge_field(dims, 0.5, 2200 + sum(dims))
    eta = wdgen.mixed_sources(dims, 3, 3, 2250 + sum(dims))
    eta[4] = 0
    g = wd.Gauge(dev(U), dims, -1, recon12=inner == wd.F32)
    kappa = (8.0 + m0) / m0
    for every, chunk in ((0 if inner == wd.F64 else 50, 0), (9, 7), (0 if inner == wd.F64 else 20, 1)):
        p = wd.cg_default_params(inner=inner, reliable_every=every, chunk=chunk, method=wd.METHOD_BICGSTAB)
        say("fused bicgstab", dims, inner, every, chunk)
        xa, ra, rca = _solve(g, m0, eta, p)
        xb, rb, rcb = _solve(g, m0, eta, p, unfused=True)
        assert rca == rcb == wd.WD_OK, (ra, rb)
        live = [i for i in range(eta.shape[0]) if i != 4]
        assert np.all(oracle.true_residual(U, eta[live], xa[live], dims, m0, -1) <= TOL * 1.0000001)
        assert not np.any(xa[4]) and ra[4]["iters"] == 0
        for i in live:
            assert rel(xa[i], xb[i]) <= kappa * 2 * TOL
            if inner == wd.F64 and every == 0:
                assert abs(ra[i]["iters"] - rb[i]["iters"]) <= max(2, rb[i]["iters"] // 20), (i, ra[i], rb[i])
    p = wd.cg_default_params(inner=inner, reliable_every=0, max_iter=3, method=wd.METHOD_BICGSTAB)
    _, r3, rc3 = _solve(g, m0, eta[5:6], p)
    assert rc3 == wd.WD_ENOTCONV and r3[0]["iters"] == 3
    g.close()


def test_workspace_without_the_fused_pieces():
    """A workspace of the five-stage iteration's size is still accepted and runs it."""
    import ctypes

    import torch
    dims, m0 = (8, 8, 4, 4), 0.1
    U = wdgen.gauge_field(dims, 0.5, 2301)
    eta = wdgen.gaussian_source(dims, 2, 2302)
    g = wd.Gauge(dev(U), dims)
    p = wd.cg_default_params(inner=wd.F32, method=wd.METHOD_BICGSTAB)
    full = wd.cg_workspace_bytes(g, 2, p)
    V = 8 * 8 * 4 * 4
    least = full - (-(-(V // 64 * 2 * 7 * 8) // 256) * 256) - (-(-(3 * 112 * 2) // 256) * 256)
    src, sol = dev(eta), torch.zeros_like(dev(eta))
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    reps = (wd.CGReport * 2)()

    def call(nbytes):
        return wd.lib().wd_cg_solve_batch(g.handle, m0, ctypes.c_void_p(src.data_ptr()),
                                          ctypes.c_void_p(sol.data_ptr()), 2, ctypes.byref(p),
                                          ctypes.c_void_p(ws.data_ptr()), nbytes, reps, None)
    say("bicgstab least workspace", least, full)
    assert call(least) == wd.WD_OK
    assert np.all(oracle.true_residual(U, eta, host(sol), dims, m0, -1) <= TOL * 1.0000001)
    assert call(least - 256) == wd.WD_ENOMEM
