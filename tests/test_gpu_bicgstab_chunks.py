"""BiCGSTAB's results do not depend on where its chunks end: the solutions and
reports with the library's chunk lengths and with fixed chunks of 1, 7 and 50
iterations are bitwise the same.

A restart at a near breakdown, |<r_hat, r>| <= 1e-6 |r_hat| |r|, falls on a
chunk's end in some of these and inside a chunk in others.  The sources: a point
source and a Gaussian one on lattices of site and of plane blocks (the point
source meets the near breakdown after one iteration, with a direction that is r to
rounding), and one chosen to meet it after two iterations with a small
<r_hat, r> before it, where the direction formed from beta is not near r."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
TOL = 1e-10

# a point source plus 0.01 times these combinations of four Gaussian fields
LATE = {(8, 8, 4, 4): (4024, [1.8349609 + 4.2823195j, 1.9137412 - 1.9538463j, 0.1343238 - 1.5874085j,
                              -1.1193721 + 1.2736770j]),
        (4, 4, 4, 4): (4016, [1.1676564 + 1.4150532j, 1.0994421 + 1.5163641j, -0.1216655 - 1.4241275j,
                              -3.1859553 + 1.4300610j])}
M0 = 0.1


def late_source(dims):
    seed, coef = LATE[dims]
    U = wdgen.gauge_field(dims, 0.5, seed)
    g = wdgen.gaussian_source(dims, 4, seed + 1)
    eta = wdgen.point_sources(dims, range(1)).copy()
    for k in range(4):
        eta += 0.01 * coef[k] * g[k:k + 1] / np.linalg.norm(g[k])
    return U, eta


def two_iterations(U, eta, dims):
    """<r_hat, r> / |r_hat| |r| after the first two iterations, and |p - r| / |r|
    of the direction the second one forms."""
    D = lambda v: oracle.dirac(U, v, dims, M0, -1)
    r, ratio = eta, []
    p, rho = r, np.vdot(eta, eta)
    for _ in range(2):
        v = D(p)
        alpha = rho / np.vdot(eta, v)
        s = r - alpha * v
        t = D(s)
        omega = np.vdot(t, s) / np.vdot(t, t)
        r = s - omega * t
        rho, old = np.vdot(eta, r), rho
        p = r + rho / old * alpha / omega * (p - omega * v)
        ratio.append(abs(rho) / np.linalg.norm(eta) / np.linalg.norm(r))
    return ratio, np.linalg.norm(p - r) / np.linalg.norm(r)


def _solve(g, eta, inner, chunk):
    import torch
    p = wd.cg_default_params(inner=inner, reliable_every=0 if inner == wd.F64 else 50, chunk=chunk,
                             method=wd.METHOD_BICGSTAB)
    ws = torch.empty(wd.cg_workspace_bytes(g, eta.shape[0], p), dtype=torch.uint8, device="cuda")
    say("bicgstab chunk length", chunk, inner, eta.shape)
    x, reps, rc = wd.cg_solve_batch(g, M0, dev(eta), params=p, ws=ws)
    assert rc == wd.WD_OK, reps
    return host(x), [(r["iters"], r["true_rel_res"], r["iter_rel_res"], r["reliable_updates"]) for r in reps]


def _neutral(U, eta, dims, inner):
    g = wd.Gauge(dev(U), dims, -1, recon12=inner == wd.F32)
    out = {chunk: _solve(g, eta, inner, chunk) for chunk in (0, 1, 7, 50)}
    g.close()
    for chunk in (1, 7, 50):
        assert out[0][1] == out[chunk][1], chunk
        assert np.array_equal(out[0][0].view(np.uint64), out[chunk][0].view(np.uint64)), chunk
    assert np.all(oracle.true_residual(U, eta, out[0][0], dims, M0, -1) <= TOL * 1.0000001)


@pytest.mark.parametrize("inner", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
@pytest.mark.parametrize("dims", [(8, 8, 4, 6), (4, 4, 4, 4), (13, 5, 4, 3)], ids=str)
def test_point_and_gaussian_sources(dims, inner):
    U = wdgen.gauge_field(dims, 0.5, 4100 + sum(dims))
    _neutral(U, wdgen.mixed_sources(dims, 2, 1, 4150 + sum(dims)), dims, inner)


@pytest.mark.parametrize("inner", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
@pytest.mark.parametrize("dims", sorted(LATE), ids=str)
def test_near_breakdown_after_a_small_rho(dims, inner):
    U, eta = late_source(dims)
    ratio, off = two_iterations(U, eta, dims)
    assert 1e-6 < ratio[0] < 1e-4 and 5e-7 < ratio[1] < 9e-7 and off > 1e-4, (ratio, off)
    _neutral(U, np.concatenate([eta, wdgen.gaussian_source(dims, 1, 4060)]), dims, inner)
