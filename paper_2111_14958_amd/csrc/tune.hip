// Launch-shape table and autotuner.
//
// The paper tunes the SYCL workgroup size of its CG kernels per device
// (Sec. 3.1, Fig. 1).  Here the equivalent knobs of the operator kernel are the
// block size, the number of right-hand sides each thread carries (link reuse
// against register pressure) and the XCD-contiguous tile order.  Candidates are
// timed on scratch fields with HIP events; a candidate must reproduce the
// reference shape's output to rounding (shapes that sum the eight hops in
// another order round differently) or it is rejected.  Tuned shapes are kept
// in a table per (lattice, precision, rhs count, dagger, kernel family) and,
// when WD_TUNE_CACHE names a file, appended to it (format: tune_cache.h).
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "wd_device.h"
#include "tune_cache.h"
#include "wd_host.h"

namespace wd {

bool ShapeKey::operator<(const ShapeKey &o) const {
    for (int d = 0; d < 4; ++d)
        if (L[d] != o.L[d]) return L[d] < o.L[d];
    if (prec != o.prec) return prec < o.prec;
    if (nrhs != o.nrhs) return nrhs < o.nrhs;
    if (dag != o.dag) return dag < o.dag;
    return fam < o.fam;
}

static std::mutex g_mu;
static std::map<ShapeKey, std::pair<Shape, double>> g_table;
static bool g_loaded = false;

// Untuned shapes (the measured best on gfx950 for 14^4 x 16 rhs): XCD-
// contiguous tiles, z-strips of 4 planes, pipelined hops (plane blocks: the
// hops that read memory first), 256-thread blocks.
// The plane-blocked LDS variants are used where an xy-plane has at most 256
// sites (else the site-blocked kernels).  One rhs per thread everywhere.
// Operator kernel: plane-blocked, two z-adjacent planes per block in FP32 and
// FP16 storage with 8 or more rhs.
// CG phase kernels: plane-blocked in FP32 and FP64, one plane per block or two
// (cg_two_planes); in FP16N by fp16_planes.  The reliable-update kernel:
// plane-blocked.
// wd_tune_result.site_order: strip | planes per block << 12 (0: one) |
// group-major << 16 | plane-blocked << 17 | blocks-per-CU cap << 18 |
// z-marching << 24 (z-marching: xylds 2) | rhs passes << 25
int encode_order(const Shape &s) {
    return s.strip | ((s.planes > 1 ? s.planes : 0) << 12) | (s.gmajor << 16) | ((s.xylds ? 1 : 0) << 17) |
           (s.occ << 18) | ((s.xylds == 2) << 24) | (s.fpass << 25);
}

// FP16N phases A and B on plane blocks rather than site blocks.  The decoding
// and coding of FP16N make the phases bound by issue as much as by memory, so
// lanes left idle by a plane that does not fill its wavefronts cost more than
// the x and y neighbours from LDS save: 7/8 of the lanes in use, and planes of
// more than 192 sites with blocks for half the compute units, or of more than 128
// with three blocks or more per compute unit.  Whole solves, site against plane blocks: 16 x 16 planes (16^3 x 32, 12
// fields) 33.4 -> 30.8, (16^4, 2 fields) 4.42 -> 4.13, (16 x 16 x 8 x 8, 2 fields)
// 2.89 -> 2.81 ms, 15 x 15 (15 x 15 x 8 x 8, 4 fields) 3.24 -> 3.05 ms, 13 x 14 (16 x
// 24 of them, 4 fields) 7.9 -> 6.8 ms; but 14 x 14 (196 of 256 lanes; 14^4, 4
// fields) 5.1 -> 5.2 ms, 16 x 12 (192 planes, 3 fields) 4.15 -> 4.42 ms.  One field is bound by latency, where planes win at every
// size (8^4 2.6 -> 2.5 ms, 12^4 2.9 -> 2.6 ms, 14^4 3.0 -> 2.9 ms).
static bool fp16_planes(const int L[4], int nrhs) {
    const int np = L[0] * L[1], lanes = (np + 63) / 64 * 64;
    const int64_t blocks = (int64_t)L[2] * L[3] * nrhs;
    return nrhs == 1 || (8 * np >= 7 * lanes && ((np > 192 && blocks >= 128) || (np > 128 && blocks >= 768)));
}

// Planes per block of phases A and B (FP32, FP16N): two where a plane has 256
// sites, so that 512-thread blocks have no idle lane and three of them fill a
// compute unit's wavefronts, if the blocks come in whole rounds of the 256
// compute units or there are four rounds or more.  Whole solves, one plane
// against two: 16^3 x 32 FP16N 1 / 2 / 12 fields 5.0 -> 4.5, 6.8 -> 6.2, 30.8
// -> 30.0 ms, FP32 1 / 4 / 8 fields 5.3 -> 4.8, 14.7 -> 13.9, 29.8 -> 28.7 ms;
// but 16^4 with 1 and 3 fields (a half and one and a half rounds) FP32 3.5 ->
// 3.7, 5.6 -> 6.1 ms, and planes of 240 or 224 sites gain nothing.
static bool cg_two_planes(const int L[4], int nrhs) {
    const int64_t blocks = (int64_t)L[2] * L[3] * nrhs / 2;
    return L[0] * L[1] == 256 && L[2] % 2 == 0 && (blocks % 256 == 0 || blocks >= 1024);
}

Shape default_shape(const ShapeKey &k) {
    const int prec = k.prec, nrhs = k.nrhs, fam = k.fam;
    Shape s;
    s.block = 256;
    s.remap = 1;
    s.ordered = 3;
    s.rloop = 1;
    s.strip = 4;
    if (fam == FAM_DSLASH) {
        // one rhs per thread: at 14^4 x 16 rhs it beat two with FP16 storage
        // (33 vs 38 us, lexicographic plane order) and in FP32 on the
        // reconstruct-12 links (45 vs 48.5 us; 50 vs 49 us on complete links)
        s.nr = 1;
        s.xylds = 1;
        // memory hops (z, t) first: 47.6 -> 45.0 us FP32, 99 -> 97 us FP64
        // (fabric reads 242 -> 196 MB).  FP16 storage with z-strips: planes of 224
        // sites or more (16 x 16, 32 x 12 of them 75 -> 69 us, x 16 fields 91 ->
        // 84; 15 x 15 as 16 x 16); smaller ones gain nothing by it (16 x 12, 12
        // fields 28.5 -> 29.3 us) and keep the lexicographic order
        if (prec == WD_F16N && k.L[0] * k.L[1] < 224) s.strip = 0;
        else s.ordered = 5;
        // FP32 with 8 or more rhs: two z-adjacent planes per block (a 14 x 14
        // plane fills 196 of 256 lanes, two fill 392 of 448): 14^4 x 16 rhs
        // 45.1-45.9 -> 42.7-44.5 us.  With one field the halved block count
        // costs more than it saves (14^4: 7.1 -> 7.7 us, 12^4: 6.5 -> 6.9 us).
        // FP16 storage alike: 12^4 x 12 17.1 -> 15.8, 13 x 14 planes 17.5 -> 16.2,
        // 14^4 x 16 32.3 -> 31.9, 16^3 x 32 x 12 69 -> 65 us (both rules: 78.5 ->
        // 76.6 us over rotating buffers), 8 x 8 planes the same
        if (prec != WD_F64 && nrhs >= 8) s.planes = 2;
    } else if (fam == FAM_CG_R) {
        s.nr = 1;
        s.xylds = 1;
    } else {
        s.nr = 1;
        s.xylds = prec != WD_F16N || fp16_planes(k.L, nrhs);
        // FP64: strips of 2 z-planes measured faster than 4 at 14^4, 16 rhs
        // (phase B 6 %; the whole solve 3 % more with phase A's too)
        if (prec == WD_F64) s.strip = 2;
        // plane blocks with the memory hops first: FP32 phase A 57.0 -> 53.4 us,
        // phase B 71.7 -> 69.5 us; FP64 phase A 112.8 -> 109.7 us
        if (s.xylds) s.ordered = 5;
        if (s.xylds && prec != WD_F64 && cg_two_planes(k.L, nrhs)) {
            s.planes = 2;
            // wider strips with few fields, and with three or four where t is
            // long against z.  Whole solves, strips of 4 against 8: 16^3 x 32 FP32
            // 1 / 2 / 3 / 4 / 6 / 12 fields 5.68 -> 5.59, 9.18 -> 8.77, 12.71 -> 12.52,
            // 16.02 -> 15.94, 21.8 -> 22.0, 48.8 -> 49.4 ms (FP16N -2.5, -1.1, -0.6,
            // -0.6, 0, +0.6 %), 16 x 16 x 8 x 32 x 4 9.29 -> 9.03; but 16^4 x 4 8.00 ->
            // 8.47, 16^3 x 24 x 4 11.76 -> 11.88 ms
            s.strip = nrhs <= 2 || (nrhs <= 4 && k.L[3] >= 2 * k.L[2]) ? 8 : 4;
        }
    }
    return s;
}

// arch and runtime version of the current device, the key of cache lines
static bool cache_identity(std::string *arch, int *ver) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess ||
        hipRuntimeGetVersion(ver) != hipSuccess)
        return false;
    *arch = prop.gcnArchName;
    return true;
}

static void load_cache_locked() {
    if (g_loaded) return;
    g_loaded = true;
    const char *path = getenv("WD_TUNE_CACHE");
    if (!path || !*path) return;
    std::string arch;
    int ver = 0;
    if (!cache_identity(&arch, &ver)) return;
    FILE *f = fopen(path, "r");
    if (!f) return;
    char line[512];
    while (fgets(line, sizeof line, f)) {
        line[strcspn(line, "\n")] = 0;
        CacheKey ck;
        CacheShape cs;
        double us = 0;
        if (!cache_parse(line, arch.c_str(), ver, &ck, &cs, &us)) continue;
        ShapeKey k{{ck.L[0], ck.L[1], ck.L[2], ck.L[3]}, ck.prec, ck.nrhs, ck.dag, ck.fam};
        Shape s;
        s.block = cs.block;
        s.nr = cs.nr;
        s.remap = cs.remap;
        s.ordered = cs.ordered;
        s.rloop = cs.rloop;
        s.strip = cs.strip;
        s.gmajor = cs.gmajor;
        s.xylds = cs.xylds;
        s.occ = cs.occ;
        s.fpass = cs.fpass;
        s.planes = cs.planes;
        g_table[k] = {s, us};
    }
    fclose(f);
}

Shape shape_lookup(const ShapeKey &k, bool *stored) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_cache_locked();
    auto it = g_table.find(k);
    if (stored) *stored = it != g_table.end();
    if (it != g_table.end()) return it->second.first;
    return default_shape(k);
}

void shape_store(const ShapeKey &k, const Shape &s) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_cache_locked();
    g_table[k] = {s, 0.0};
}

void shape_store_persist(const ShapeKey &k, const Shape &s, double us) {
    shape_store(k, s);
    const char *path = getenv("WD_TUNE_CACHE");
    if (!path || !*path) return;
    std::string arch;
    int ver = 0;
    if (!cache_identity(&arch, &ver)) return;
    const CacheKey ck{k.fam, {k.L[0], k.L[1], k.L[2], k.L[3]}, k.prec, k.nrhs, k.dag};
    const CacheShape cs{s.block, s.nr, s.remap, s.ordered, s.rloop, s.strip, s.gmajor, s.xylds, s.occ, s.fpass,
                        s.planes};
    const std::string line = cache_line(arch.c_str(), ver, ck, cs, us);
    std::lock_guard<std::mutex> lk(g_mu);
    FILE *f = fopen(path, "a");
    if (!f) return;
    fputs(line.c_str(), f);
    fclose(f);
}

// Deterministic scratch data: a counter hash mapped to [-1, 1).
__device__ __forceinline__ float hash_unit(uint32_t i) {
    i ^= i >> 16; i *= 0x7feb352du; i ^= i >> 15; i *= 0x846ca68bu; i ^= i >> 16;
    return (float)(i >> 8) * (2.0f / 16777216.0f) - 1.0f;
}

// Fill a packed spinor buffer with valid data of precision P.
template <int P>
__global__ void k_fill(void *buf, int V, int nrhs, uint32_t seed) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    if (s >= V) return;
    typedef typename real_of<P>::type R;
    cx<R> v[12];
    for (int k = 0; k < 12; ++k) {
        const uint32_t base = seed + 24u * ((uint32_t)r * (uint32_t)V + (uint32_t)s) + 2u * k;
        v[k] = {(R)hash_unit(base), (R)hash_unit(base + 1)};
    }
    FieldPtr f{buf, V, nrhs};
    Spinor<P>::store(f, r, s, v);
}

static int fill_spinor(int prec, void *buf, int V, int nrhs, hipStream_t st) {
    dim3 grid((V + 255) / 256, nrhs);
    if (prec == WD_F64) hipLaunchKernelGGL(k_fill<P64>, grid, dim3(256), 0, st, buf, V, nrhs, 12345u);
    if (prec == WD_F32) hipLaunchKernelGGL(k_fill<P32>, grid, dim3(256), 0, st, buf, V, nrhs, 12345u);
    if (prec == WD_F16N) hipLaunchKernelGGL(k_fill<P16>, grid, dim3(256), 0, st, buf, V, nrhs, 12345u);
    WD_HIP(hipGetLastError());
    return WD_OK;
}

static double algorithmic_bytes(int prec, int64_t V, int nrhs) {
    return (double)link_bytes(prec, V) + 2.0 * (double)spinor_bytes(prec, V, nrhs);
}

// Time `reps` launches of one shape; returns the median in microseconds.
static int time_shape(const wd_gauge *g, int prec, bool dag, const void *in, void *out, int nrhs,
                      const Shape &sh, hipStream_t st, int reps, double *median_us) {
    hipEvent_t e0, e1;
    WD_HIP(hipEventCreate(&e0));
    WD_HIP(hipEventCreate(&e1));
    std::vector<double> t;
    int rc = WD_OK;
    for (int w = 0; w < 2 && !rc; ++w) rc = launch_dslash(g, 0.1, prec, dag, in, out, nrhs, sh, st);
    for (int i = 0; i < reps && !rc; ++i) {
        hipEventRecord(e0, st);
        rc = launch_dslash(g, 0.1, prec, dag, in, out, nrhs, sh, st);
        hipEventRecord(e1, st);
        if (hipEventSynchronize(e1) != hipSuccess) rc = fail(WD_EHIP, "event sync failed");
        float ms = 0;
        hipEventElapsedTime(&ms, e0, e1);
        t.push_back(ms * 1000.0);
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (rc) return rc;
    std::sort(t.begin(), t.end());
    *median_us = t[t.size() / 2];
    return WD_OK;
}

}  // namespace wd

using namespace wd;

extern "C" {

int wd_tune_lookup(const wd_gauge *g, int32_t prec, int32_t nrhs, int32_t dagger, wd_tune_result *cfg) {
    clear_error();
    WD_CHECK(g && cfg, WD_EINVAL, "null argument");
    ShapeKey k{{g->dims[0], g->dims[1], g->dims[2], g->dims[3]}, prec, nrhs, dagger ? 1 : 0};
    Shape s = shape_lookup(k);
    memset(cfg, 0, sizeof(*cfg));
    cfg->block = s.block;
    cfg->rhs_per_thread = s.nr;
    cfg->xcd_remap = s.remap;
    cfg->hop_order = s.ordered;
    cfg->rhs_loop = s.rloop;
    cfg->site_order = encode_order(s);
    return WD_OK;
}

int wd_shape_get(const wd_gauge *g, int32_t prec, int32_t nrhs, int32_t dagger, int32_t family,
                 wd_tune_result *cfg) {
    clear_error();
    WD_CHECK(g && cfg, WD_EINVAL, "null argument");
    WD_CHECK(family >= FAM_DSLASH && family <= FAM_CG_R, WD_EINVAL, "unknown kernel family %d", family);
    ShapeKey k{{g->dims[0], g->dims[1], g->dims[2], g->dims[3]}, prec, nrhs, dagger ? 1 : 0, family};
    const Shape s = shape_lookup(k);
    memset(cfg, 0, sizeof(*cfg));
    cfg->block = s.block;
    cfg->rhs_per_thread = s.nr;
    cfg->xcd_remap = s.remap;
    cfg->hop_order = s.ordered;
    cfg->rhs_loop = s.rloop;
    cfg->site_order = encode_order(s);
    return WD_OK;
}

int wd_shape_set(const wd_gauge *g, int32_t prec, int32_t nrhs, int32_t dagger, int32_t family,
                 const wd_tune_result *sh) {
    clear_error();
    WD_CHECK(g && sh, WD_EINVAL, "null argument");
    WD_CHECK(prec >= 0 && prec <= 2, WD_EINVAL, "unknown precision %d", prec);
    WD_CHECK(nrhs >= 1 && nrhs <= MAX_RHS, WD_EINVAL, "nrhs %d out of range", nrhs);
    WD_CHECK(family >= FAM_DSLASH && family <= FAM_CG_R, WD_EINVAL, "unknown kernel family %d", family);
    WD_CHECK(sh->block == 64 || sh->block == 128 || sh->block == 256 || ((sh->site_order >> 17) & 1), WD_EINVAL,
             "block %d", sh->block);   // the plane-blocked variant takes the plane size
    WD_CHECK(sh->rhs_per_thread == 1 || sh->rhs_per_thread == 2 || sh->rhs_per_thread == 4, WD_EINVAL,
             "rhs_per_thread %d", sh->rhs_per_thread);
    WD_CHECK(sh->hop_order >= 0 && sh->hop_order <= 5 && sh->rhs_loop >= 1, WD_EINVAL, "bad hop order / rhs loop");
    WD_CHECK(sh->hop_order != 5 || (family != FAM_CG_R && ((sh->site_order >> 17) & 1)), WD_EINVAL,
             "hop order 5 (memory hops first): plane-blocked operator and CG phase A/B kernels only");
    WD_CHECK(family == FAM_DSLASH || ((sh->hop_order == 1 || sh->hop_order == 3 || sh->hop_order == 5) &&
                                      sh->rhs_loop == 1),
             WD_EINVAL, "CG kernels take hop order 1, 3 or 5 and one rhs group per block");
    WD_CHECK(!(family == FAM_CG_R && sh->rhs_per_thread > 2), WD_EINVAL, "reliable-update kernel takes <= 2 rhs");
    WD_CHECK(!(prec == WD_F64 && family != FAM_DSLASH && sh->rhs_per_thread > 2), WD_EINVAL,
             "FP64 CG kernels take <= 2 rhs per thread");
    const int zm = (sh->site_order >> 24) & 1;
    const int strip = sh->site_order & 0xfff, planes = std::max(1, (sh->site_order >> 12) & 7),
              gmajor = (sh->site_order >> 16) & 1,
              xylds = (sh->site_order >> 17) & 1 ? 1 + zm : 0, occ = (sh->site_order >> 18) & 0x3f;
    const int fpass = (sh->site_order >> 25) & 0x3f;
    WD_CHECK(sh->site_order >= 0 && (sh->site_order >> 31) == 0 && ((sh->site_order >> 15) & 1) == 0 && occ <= 8,
             WD_EINVAL, "site_order 0x%x", sh->site_order);
    WD_CHECK(planes == 1 || (((sh->site_order >> 17) & 1) && !zm && sh->rhs_per_thread == 1 && planes <= 4 &&
                             family != FAM_CG_R && (sh->hop_order == 5 || (sh->hop_order == 3 && family == FAM_DSLASH))),
             WD_EINVAL, "several planes per block: plane-blocked operator (hop order 3 or 5) and CG phase A/B "
             "kernels (hop order 5), one rhs per thread, at most 4 planes");
    WD_CHECK(fpass == 0 || ((family == FAM_CG_A || family == FAM_CG_B) && !gmajor && !zm), WD_EINVAL,
             "passes of rhs groups: CG phase A/B kernels in site-block-major order only");
    WD_CHECK(!zm || ((sh->site_order >> 17) & 1), WD_EINVAL, "z-marching needs the plane-blocked bit");
    WD_CHECK(!xylds || g->dims[0] * g->dims[1] <= 256, WD_EINVAL, "plane-blocked LDS variant: Lx*Ly <= 256");
    WD_CHECK(!(xylds && family == FAM_CG_R && sh->rhs_per_thread != 1), WD_EINVAL,
             "plane-blocked reliable update: one rhs per thread");
    WD_CHECK(!zm || family != FAM_CG_R, WD_EINVAL,
             "z-marching: operator and CG phase A/B kernels only (FP64 falls back to plane blocks)");
    ShapeKey k{{g->dims[0], g->dims[1], g->dims[2], g->dims[3]}, prec, nrhs, dagger ? 1 : 0, family};
    Shape s;
    s.block = sh->block;
    s.nr = sh->rhs_per_thread;
    s.remap = sh->xcd_remap ? 1 : 0;
    s.ordered = sh->hop_order;
    s.rloop = sh->rhs_loop;
    s.strip = strip;
    s.gmajor = gmajor;
    s.xylds = xylds;
    s.occ = occ;
    s.fpass = fpass;
    s.planes = planes;
    shape_store(k, s);
    return WD_OK;
}

// Does a candidate's packed output b agree with the reference a to rounding?
// Shapes that sum the eight hops in another order (hop order 5) round
// differently; a wrong shape (a lost hop, a wrong neighbour) is off by O(1).
// Bound per component: FP64 1e-12, FP32 2e-5 of the largest reference
// component; FP16N (decoded) two half ulps of the site's norm plus 2e-5.
static bool within_rounding(int prec, const unsigned char *a, const unsigned char *b, int V, int nrhs) {
    if (prec == WD_F16N) {
        const size_t ncode = (size_t)nrhs * 3 * V * 8;   // halves
        const _Float16 *ca = (const _Float16 *)a, *cb = (const _Float16 *)b;
        const float *na = (const float *)(a + ncode * 2), *nb = (const float *)(b + ncode * 2);
        double amax = 0;
        for (size_t i = 0; i < (size_t)nrhs * V; ++i) amax = std::max(amax, (double)na[i]);
        for (int r = 0; r < nrhs; ++r)
            for (int j = 0; j < 3; ++j)
                for (int s = 0; s < V; ++s)
                    for (int k = 0; k < 8; ++k) {
                        const size_t ci = (((size_t)r * 3 + j) * V + s) * 8 + k, ni = (size_t)r * V + s;
                        const double va = (double)na[ni] * (double)ca[ci], vb = (double)nb[ni] * (double)cb[ci];
                        const double tol = std::ldexp(std::max((double)na[ni], (double)nb[ni]), -10) + 2e-5 * amax;
                        if (!(std::fabs(va - vb) <= tol)) return false;
                    }
        return true;
    }
    const size_t n = spinor_bytes(prec, V, nrhs) / (prec == WD_F64 ? 8 : 4);
    double amax = 0;
    for (size_t i = 0; i < n; ++i)
        amax = std::max(amax, std::fabs(prec == WD_F64 ? ((const double *)a)[i] : (double)((const float *)a)[i]));
    const double tol = (prec == WD_F64 ? 1e-12 : 2e-5) * amax;
    for (size_t i = 0; i < n; ++i) {
        const double va = prec == WD_F64 ? ((const double *)a)[i] : (double)((const float *)a)[i];
        const double vb = prec == WD_F64 ? ((const double *)b)[i] : (double)((const float *)b)[i];
        if (!(std::fabs(va - vb) <= tol)) return false;
    }
    return true;
}

int wd_tune_dslash(const wd_gauge *g, int32_t prec, int32_t nrhs, int32_t dagger, wd_tune_result *best,
                   void *stream) {
    clear_error();
    WD_CHECK(g, WD_EINVAL, "null gauge");
    WD_CHECK(prec >= 0 && prec <= 2 && g->U[prec], WD_EINVAL, "gauge holds no links in precision %d", prec);
    WD_CHECK(nrhs >= 1 && nrhs <= MAX_RHS, WD_EINVAL, "nrhs %d out of range", nrhs);
    int rc = require_gfx950();
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int V = (int)g->V;
    const size_t nb = spinor_bytes(prec, V, nrhs);
    void *in = nullptr, *ref = nullptr, *out = nullptr;
    WD_HIP(hipMalloc(&in, nb));
    if (hipMalloc(&ref, nb) != hipSuccess || hipMalloc(&out, nb) != hipSuccess) {
        hipFree(in);
        if (ref) hipFree(ref);
        return fail(WD_ENOMEM, "autotuner scratch allocation failed");
    }
    std::vector<unsigned char> h_ref(nb), h_out(nb);
    const bool dag = dagger != 0;
    Shape refshape;
    refshape.block = 256;
    refshape.nr = 1;
    refshape.remap = 0;
    refshape.ordered = 1;
    refshape.rloop = 1;
    Shape bestshape = refshape;
    double best_us = 1e30;
    rc = fill_spinor(prec, in, V, nrhs, st);
    if (!rc) rc = launch_dslash(g, 0.1, prec, dag, in, ref, nrhs, refshape, st);
    if (!rc && hipMemcpyAsync(h_ref.data(), ref, nb, hipMemcpyDeviceToHost, st) != hipSuccess)
        rc = fail(WD_EHIP, "copy of reference output failed");
    if (!rc && hipStreamSynchronize(st) != hipSuccess) rc = fail(WD_EHIP, "stream sync failed");
    const int blocks[3] = {64, 128, 256};
    const int nrs[3] = {1, 2, 4};
    const bool verbose = getenv("WD_TUNE_VERBOSE") != nullptr;
    const int rloops[3] = {1, 2, 4};
    // processing orders: lexicographic, z-strips of 2, 4 and about half the z extent
    const int Lz = g->dims[2];
    const int strips[4] = {0, Lz > 2 ? 2 : 0, Lz > 4 ? 4 : 0, Lz > 4 ? (Lz + 1) / 2 : 0};
    // run one candidate: reject it unless its output agrees with the reference
    // to rounding (within_rounding), else time it and keep the fastest
    auto try_shape = [&](const Shape &s) {
        hipMemsetAsync(out, 0, nb, st);
        rc = launch_dslash(g, 0.1, prec, dag, in, out, nrhs, s, st);
        if (rc) return;
        if (hipMemcpyAsync(h_out.data(), out, nb, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            rc = fail(WD_EHIP, "copy of candidate output failed");
            return;
        }
        if (!within_rounding(prec, h_ref.data(), h_out.data(), V, nrhs)) {   // rejected
            if (verbose) fprintf(stderr, "[wd tune] block %d nr %d remap %d ordered %d rloop %d strip %d gmajor %d "
                                 "xylds %d occ %d planes %d: output differs, rejected\n", s.block, s.nr, s.remap,
                                 s.ordered, s.rloop, s.strip, s.gmajor, s.xylds, s.occ, s.planes);
            return;
        }
        double us = 0;
        rc = time_shape(g, prec, dag, in, out, nrhs, s, st, 10, &us);
        if (verbose && !rc)
            fprintf(stderr, "[wd tune] block %d nr %d remap %d ordered %d rloop %d strip %d gmajor %d xylds %d occ %d "
                    "planes %d: %.2f us, %.0f GB/s\n", s.block, s.nr, s.remap, s.ordered, s.rloop, s.strip, s.gmajor,
                    s.xylds, s.occ, s.planes, us, algorithmic_bytes(prec, V, nrhs) / (us * 1e-6) / 1e9);
        if (!rc && us < best_us) { best_us = us; bestshape = s; }
    };
    for (int bi = 0; bi < 3 && !rc; ++bi)
        for (int ni = 0; ni < 3 && !rc; ++ni)
            for (int cand = 0; cand < 30 * 8 && !rc; ++cand) {
                Shape s;
                const int c = cand % 30, o = cand / 30;
                s.block = blocks[bi];
                s.nr = nrs[ni];
                s.remap = c & 1;
                s.ordered = (c >> 1) % 5;         // 0 free, 1 per hop, 2 per direction, 3 pipelined,
                                                  // 4 pipelined with the own spinor first
                s.rloop = rloops[c / 10];
                s.strip = strips[o & 3];
                s.gmajor = o >> 2;
                if (o > 0 && strips[o & 3] == 0 && (o & 3) != 0) continue;   // order unavailable
                if (s.gmajor && s.rloop > 1) continue;
                if (s.ordered == 4 && s.nr != 1) continue;
                const int ngroups = (nrhs + s.nr - 1) / s.nr;
                if (s.gmajor && ngroups == 1) continue;
                if (s.rloop > 1 && s.rloop > ngroups) continue;
                if (s.nr > 1 && s.nr > nrhs) continue;
                if (prec == WD_F64 && s.nr > 2) continue;
                try_shape(s);
            }
    // plane-blocked variant: one xy-plane per block, x/y neighbours from LDS
    const int np = g->dims[0] * g->dims[1];
    const Geom geo = make_geom(g);
    if (np <= 256)
        for (int cand2 = 0; cand2 < 2 * 2 * 3 * 8 * 4 * 2 && !rc; ++cand2) {
            Shape s;
            const int occs[4] = {0, 3, 4, 6}, ords[3] = {1, 3, 5};
            const int cand = cand2 % 384;
            s.planes = cand2 < 384 ? 1 : 2;   // two z-adjacent planes per block
            s.occ = occs[cand / 96];
            const int o = (cand / 12) & 7;
            s.block = np;
            s.nr = (cand & 1) ? 2 : 1;
            s.remap = (cand >> 1) & 1;
            s.ordered = ords[(cand >> 2) % 3];
            if (s.ordered == 5 && s.nr != 1) continue;   // memory hops first: one rhs per thread
            s.rloop = 1;
            s.strip = strips[o & 3];
            s.gmajor = o >> 2;
            s.xylds = 1;
            if (o > 0 && strips[o & 3] == 0 && (o & 3) != 0) continue;
            if (s.nr > 1 && (prec == WD_F64 || nrhs < 2)) continue;
            if (s.gmajor && (nrhs + s.nr - 1) / s.nr == 1) continue;
            if (s.planes > 1 && (s.ordered == 1 || xy_planes(s, geo, prec, s.nr) != s.planes)) continue;
            try_shape(s);
        }
    hipFree(in);
    hipFree(ref);
    hipFree(out);
    if (rc) return rc;
    ShapeKey k{{g->dims[0], g->dims[1], g->dims[2], g->dims[3]}, prec, nrhs, dagger ? 1 : 0};
    shape_store_persist(k, bestshape, best_us);
    if (best) {
        memset(best, 0, sizeof(*best));
        best->block = bestshape.block;
        best->rhs_per_thread = bestshape.nr;
        best->xcd_remap = bestshape.remap;
        best->hop_order = bestshape.ordered;
        best->rhs_loop = bestshape.rloop;
        best->site_order = encode_order(bestshape);
        best->us = best_us;
        best->gbps = algorithmic_bytes(prec, V, nrhs) / (best_us * 1e-6) / 1e9;
    }
    return WD_OK;
}

}  // extern "C"
