"""PRECOND_EO on lattices with an odd Ly, Lz or Lt, where the wrap-around joins sites
of one parity and no even-odd splitting exists: the solve runs without
preconditioning, bit for bit, alone and in the server, and passes the oracle's
residual (of the full system, not of a Schur complement)."""
import time

import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
M0, TOL = 0.1, 1e-10
DIMS = [(6, 5, 4, 4), (8, 8, 5, 4), (4, 6, 4, 7), (16, 9, 3, 3), (2, 1, 4, 4)]


@pytest.mark.parametrize("inner", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
@pytest.mark.parametrize("dims", DIMS, ids=str)
def test_solve(dims, inner):
    U = wdgen.gauge_field(dims, 0.5, 6300 + sum(dims))
    eta = wdgen.mixed_sources(dims, 2, 1, 6350 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1)
    out = []
    for eo in (wd.PRECOND_EO, wd.PRECOND_NONE):
        p = wd.cg_default_params(inner=inner, reliable_every=0 if inner == wd.F64 else 50, precondition=eo)
        say("even-odd, odd extents", dims, inner, eo)
        x, reps, rc = wd.cg_solve_batch(g, M0, dev(eta), params=p)
        assert rc == wd.WD_OK, reps
        out.append((host(x), [r["iters"] for r in reps]))
    g.close()
    assert np.all(oracle.true_residual(U, eta, out[0][0], dims, M0, -1) <= TOL * 1.0000001)
    assert out[0][1] == out[1][1]
    assert np.array_equal(out[0][0].view(np.uint64), out[1][0].view(np.uint64))


def test_server():
    import torch
    srv = wd.Server(torch.empty(1 << 28, dtype=torch.uint8, device="cuda"))
    jobs = []
    for dims in DIMS[:3] + [(4, 4, 4, 4)]:
        U = wdgen.gauge_field(dims, 0.5, 6400 + sum(dims))
        eta = wdgen.gaussian_source(dims, 2, 6450 + sum(dims))
        dU, src = dev(U), dev(eta)
        sol = torch.zeros_like(src)
        say("even-odd server request", dims)
        req = wd.Server.request(dims, 2, M0, dU, src, sol, wd.cg_default_params(inner=wd.F32, precondition=wd.PRECOND_EO))
        jobs.append((dims, U, eta, sol, srv.submit(req), dU, src))
    for dims, U, eta, sol, ticket, _, _ in jobs:
        rep = srv.poll(ticket)
        while rep is None:
            time.sleep(1e-3)
            rep = srv.poll(ticket)
        assert all(r["status"] == 0 for r in rep), rep
        assert np.all(oracle.true_residual(U, eta, host(sol), dims, M0, -1) <= TOL * 1.0000001)
    srv.close()
