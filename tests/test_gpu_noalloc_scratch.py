"""wd_dslash_noalloc where it uses its static scratch: shapes that keep the packed
copies (hop order 3, or planes of more than 256 sites), with calls that nearly fill
the 64 MiB array followed by smaller ones, and FP16N, whose codes and norms are
separate parts of a packed field.  Compared with the FP64 oracle field by field and,
bit for bit, with wd_dslash, whose temporaries are allocated."""
import numpy as np
import pytest

import oracle
import paper_2111_14958_amd as wd
import wdgen
from gpu_util import dev, host, rel, say
from test_gpu_operator_routes import kernels

pytestmark = pytest.mark.gpu
M0 = 0.05
TOL = {wd.F64: 1e-13, wd.F32: 1e-6, wd.F16N: 2e-3}
BYTES = {wd.F64: 192, wd.F32: 96, wd.F16N: 52}


@pytest.mark.parametrize("prec", [wd.F64, wd.F32, wd.F16N], ids=["f64", "f32", "f16n"])
@pytest.mark.parametrize("dims,hop3", [((12, 12, 11, 12), True), ((17, 16, 8, 9), False)], ids=str)
def test_scratch_calls(dims, hop3, prec):
    V = int(np.prod(dims))
    most = wd.NOALLOC_SCRATCH_BYTES // (2 * V * BYTES[prec])
    U = wdgen.gauge_field(dims, 0.5, 5300 + sum(dims))
    g = wd.Gauge(dev(U), dims, -1, precs=(wd.F64, wd.F32, wd.F16N))
    psi = wdgen.gaussian_source(dims, most, 5350 + sum(dims))
    for nrhs, dag in ((most, False), (2, True), (1, False)):
        assert 2 * nrhs * V * BYTES[prec] > wd.NOALLOC_SCRATCH_BYTES * 7 // 8 or nrhs <= 2
        if hop3:
            wd.shape_set(g, prec, nrhs, dag, wd.FAMILY_DSLASH, dims[0] * dims[1], hop_order=3, strip=2, xy_lds=1)
        say("noalloc scratch", dims, prec, nrhs, dag)
        x = dev(psi[:nrhs])
        got = []
        names = kernels(lambda: got.append(wd.dslash_noalloc(g, M0, x, prec, dagger=dag)))
        assert any("pack_spinor" in n for n in names) and not any("k_dslash_cn" in n for n in names), names
        got, ref = host(got[0]), host(wd.dslash(g, M0, x, prec, dagger=dag))
        assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))
        for i in {0, nrhs - 1}:
            assert rel(got[i:i + 1], oracle.dirac(U, psi[i:i + 1], dims, M0, -1, dagger=dag)) <= TOL[prec], i
    g.close()
