"""Which kernels an operator call launches, by the kernels' names in a trace of the
call, and the packed operator in its default shapes.

Canonical complex128 fields go through k_dslash_cn in the default shape; a shape
set to another kernel (several planes per block among them) is packed, run on that
kernel and unpacked.  The default packed FP32 shape has two planes per block from 8
fields on (one where Lz is odd, or two planes exceed 512 sites), with complete and
with two-row links; every site is compared with the oracle on the links and
fields the GPU holds."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import sitecheck
import wdgen
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
M0 = 0.07


def kernels(call):
    """names of the kernels `call` launches"""
    import torch
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.name for e in prof.events()]


def _inputs(dims, nrhs, seed):
    return wdgen.gauge_field(dims, 0.5, seed + sum(dims)), wdgen.gaussian_source(dims, nrhs, seed + 50 + sum(dims))


def test_a_set_shape_keeps_its_kernel():
    dims, nrhs = (6, 9, 4, 5), 8
    U, psi = _inputs(dims, nrhs, 5000)
    g = wd.Gauge(dev(U), dims, -1)
    x = dev(psi)
    want = oracle.dirac(sitecheck.links_f32(U), sitecheck.links_f32(psi), dims, M0, -1)

    def run(direct):
        got = []
        names = kernels(lambda: got.append(wd.dslash(g, M0, x, wd.F32)))
        say("operator route", names)
        assert any("k_dslash_cn" in n for n in names) == direct, names
        assert any("k_dslash_xy" in n for n in names) == (not direct), names
        sitecheck.assert_sites(host(got[0]), want, psi, M0, sitecheck.F32_BOUND, "direct %s" % direct)

    assert wd.shape_get(g, wd.F32, nrhs, False, wd.FAMILY_DSLASH)["xy_planes"] == 2
    run(True)                     # the default shape
    for planes, direct in ((2, False), (4, False), (3, True), (1, True)):   # 3 planes: Lz = 4, one plane
        wd.shape_set(g, wd.F32, nrhs, False, wd.FAMILY_DSLASH, 54 * planes, hop_order=5, xy_lds=1, xy_planes=planes)
        run(direct)
    wd.shape_set(g, wd.F32, nrhs, False, wd.FAMILY_DSLASH, 54, hop_order=3, xy_lds=1)
    run(False)
    g.close()


DEFAULTS = [((14, 14, 12, 14), 16, 2), ((16, 14, 4, 3), 9, 2), ((16, 16, 2, 3), 8, 2), ((9, 7, 5, 3), 8, 2),
            ((5, 13, 6, 2), 7, 1)]


@pytest.mark.parametrize("recon12", [False, True], ids=["complete", "two-row"])
@pytest.mark.parametrize("dims,nrhs,planes", DEFAULTS, ids=str)
def test_default_packed_fp32(dims, nrhs, planes, recon12):
    U, psi = _inputs(dims, nrhs, 5100)
    g = wd.Gauge(dev(U), dims, -1, recon12=recon12)
    x = wd.pack_spinor(g, dev(psi), wd.F32)
    for dag in (False, True):
        assert wd.shape_get(g, wd.F32, nrhs, dag, wd.FAMILY_DSLASH)["xy_planes"] == planes
        say("packed operator", dims, nrhs, recon12, dag)
        out = wd.dslash(g, M0, x, wd.F32, dagger=dag, packed=True, nrhs=nrhs)
        got = host(wd.unpack_spinor(g, out, wd.F32, nrhs)).reshape(psi.shape)
        want = oracle.dirac(sitecheck.links_f32(U), sitecheck.links_f32(psi), dims, M0, -1, dagger=dag)
        sitecheck.assert_sites(got, want, psi, M0, sitecheck.F32_BOUND, "%s %d" % (dims, nrhs))
    g.close()


@pytest.mark.parametrize("prec", [wd.F64, wd.F32], ids=["f64", "f32"])
def test_overlapping_canonical_fields(prec):
    """An output shifted by one field against the input takes the packed copies,
    which read the whole input first; the fields are those of a call without overlap."""
    import torch
    dims, nrhs = (6, 9, 4, 7), 3
    U, psi = _inputs(dims, nrhs, 5200)
    g = wd.Gauge(dev(U), dims, -1)
    x = dev(psi)
    want = host(wd.dslash(g, M0, x, prec))
    for shift in (1, -1):
        buf = torch.zeros((nrhs + 1,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda")
        src, dst = (buf[:nrhs], buf[1:]) if shift > 0 else (buf[1:], buf[:nrhs])
        for call in (wd.dslash, wd.dslash_noalloc):
            src.copy_(x)
            say("overlapping canonical fields", prec, shift)
            call(g, M0, src, prec, out=dst)
            assert np.array_equal(host(dst).view(np.uint64), want.view(np.uint64))
    g.close()
