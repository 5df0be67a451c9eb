// Conjugate gradient on the normal equations (arXiv 2111.14958, Sec. 2):
// kernels of the phases, the hipGraph that replays a chunk of iterations, and
// the solve driver behind wd_cg_solve / wd_cg_solve_batch.
//
// A solve runs
//   init   eta64 <- src, x64 <- x0 or 0, x_lo <- 0, scalars <- host record,
//          N (|eta|^2), R2 (r = eta - D x64, true-residual test)
//          (and C, p = r, with a z-marching phase A)
//   chunk  K x [A, B], then R1 (x64 += x_lo), R2, summary   (one graph; with a
//          z-marching phase A, which reads p: K x [A, B, C], then R1, R2, C)
// and replays the chunk graph until no right-hand side is active, reading back
// the summary (active count, abort flag, estimated iterations left) after each
// replay; with the library's chunk length a replay is cut to that estimate.
// BiCGSTAB (bicgstab_core.h) uses the same driver with the chunk S1, K x [F2,
// S3, F4, F5], trailing finish (without room for the fused iteration's records:
// K x [S1, S2, S3, S4, S5] with their finishes), then R1, R2, summary.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include <hip/hip_ext.h>

#include "bicgstab_core.h"
#include "cg_host.h"
#include "eo_core.h"

namespace wd {

// ------------------------------------------------------------------ kernels
// `remap`: XCD-contiguous tile order.  Kernels that reduce leave their
// per-block partial sums in the workspace; k_finish, launched after them,
// completes the reduction.
#define WD_KERNEL_PROLOGUE(K)                                                  \
    const int b_ = remap ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x; \
    const Prob &pr = probs[find_prob(probs, nprob, K, b_)];                    \
    const int t_ = b_ - pr.t0[K];

// R12: links from the reconstruct-12 copy (FP32 storage).  POL: cache policy of
// the streaming accesses (stream_policy).  k_phaseB completes
// phase A's reduction in its blocks (phaseB_tile with FA), so phase A has no
// finish launch of its own.  k_phaseA forms the direction as q = D^dagger r +
// beta q (phaseA_tile with QR): solves that launch it (LaunchSet::qrec) have
// no phase C; so do the even-odd phase-A kernels.
// par >= 0: the fused finish (LaunchSet::fused): iteration parity par of the
// chunk, first = 1 (phase A) for the chunk's first iteration, last = 1 (phase
// B) for its last (see phaseA_tile, phaseB_tile); -1: the three-launch
// iteration with k_finish after phase B.
// MP: plane blocks of several z-adjacent planes (up to 512 threads).
// Waves per SIMD asked of the register allocator: 3 for the FP64 kernels with
// one rhs per thread (<= 168 VGPRs; left to the compiler some take more, which
// allows 2).
// FP64 site blocks with two hops in flight (order 3): held to two waves, so that
// the second hop has its registers.  Left to itself the compiler gives up the
// second hop for waves, which these launches, short of blocks, do not have: whole
// solves 8 x 4 x 16 x 16 x 6 4.95 -> 4.62 ms, 6 x 8 x 8 x 8 x 3 3.34 -> 3.17, 4^4 2.14
// -> 2.07, 16 x 3 x 32 x 24 x 4 12.8 -> 12.7 ms.
template <int P, int NR, int ORD, bool XY>
constexpr int phase_waves(bool most) {
    if (P == P64 && NR == 1 && ORD == 3 && !XY) return 2;
    return most ? 8 : P == P64 && NR == 1 ? 3 : 1;
}
#define WD_PHASE_WAVES \
    __attribute__((amdgpu_waves_per_eu(phase_waves<P, NR, ORD, XY>(false), phase_waves<P, NR, ORD, XY>(true))))

template <int P, int NR, int ORD, bool XY, bool R12 = false, int POL = 0, bool MP = false, bool PAIR = XY>
__global__ __launch_bounds__(MP ? 512 : 256) WD_PHASE_WAVES void k_phaseA(
    const Prob *__restrict__ probs, int nprob, int remap, int par, int first) {
    WD_KERNEL_PROLOGUE(KA)
    phaseA_tile<P, NR, ORD, XY, R12, POL, true, MP, PAIR>(pr, t_, par, first);
}

template <int P, int NR, int ORD, bool XY, bool R12 = false, int POL = 0, bool MP = false, bool PAIR = XY>
__global__ __launch_bounds__(MP ? 512 : 256) WD_PHASE_WAVES void k_phaseB(
    const Prob *__restrict__ probs, int nprob, int remap, int par, int last) {
    WD_KERNEL_PROLOGUE(KB)
    phaseB_tile<P, NR, ORD, XY, R12, POL, true, MP, PAIR>(pr, t_, par, last);
}

// direction-split phases A and B (phaseA_split_tile), four threads per site
template <int P, bool R12, bool B>
__global__ __launch_bounds__(P == P64 ? 512 : 1024) void k_phase_split(const Prob *__restrict__ probs, int nprob, int remap, int par,
                                                      int edge) {
    extern __shared__ uint4 split_lds_raw[];
    WD_KERNEL_PROLOGUE(B ? KB : KA)
    if constexpr (B) phaseB_split_tile<P, R12>(pr, t_, par, edge, split_lds_raw);
    else phaseA_split_tile<P, R12>(pr, t_, par, edge, split_lds_raw);
}

// z-marching phases A and B (zm_tile); dynamic LDS of two plane buffers
template <int P, int ORD>
__global__ __launch_bounds__(256) void k_phaseA_zm(const Prob *__restrict__ probs, int nprob, int remap) {
    extern __shared__ uint4 zm_lds[];
    WD_KERNEL_PROLOGUE(KA)
    zm_tile<P, ORD, false>(pr, t_, (typename LdsSpinor<P>::word *)zm_lds);
}

template <int P, int ORD>
__global__ __launch_bounds__(256) void k_phaseB_zm(const Prob *__restrict__ probs, int nprob, int remap) {
    extern __shared__ uint4 zm_lds[];
    WD_KERNEL_PROLOGUE(KB)
    zm_tile<P, ORD, true>(pr, t_, (typename LdsSpinor<P>::word *)zm_lds);
}

template <int P>
__global__ __launch_bounds__(256) void k_phaseC(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KC)
    phaseC_tile<P>(pr, t_);
}

template <int P>
__global__ __launch_bounds__(256) void k_ru1(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KR1)
    ru1_tile<P>(pr, t_);
}

template <int P, int NR, bool XY = false, bool ZX = false>
__global__ __launch_bounds__(256) void k_ru2(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KR2)
    ru2_tile<P, NR, XY, ZX>(pr, t_);
}

__global__ __launch_bounds__(256) void k_norm(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KN)
    norm_tile(pr, t_);
}

// Even-odd preconditioning (eo_core.h)
// XY: half-plane blocks (see eo_tile), hop order 5, one rhs per thread
template <int P, int NR, bool DAG, bool R12 = false, bool XY = false>
__global__ __launch_bounds__(256) void k_eo_hop1(const Prob *__restrict__ probs, int nprob, int remap, int par, int /*edge*/) {
    WD_KERNEL_PROLOGUE(DAG ? KEA1 : KEB1)
    eo_hop1_tile<P, NR, DAG, true, R12, XY>(pr, t_, par);
}
template <int P, int NR, bool R12 = false, bool XY = false>
__global__ __launch_bounds__(256) void k_eo_phaseA(const Prob *__restrict__ probs, int nprob, int remap, int par, int edge) {
    WD_KERNEL_PROLOGUE(KA)
    eo_phaseA_tile<P, NR, true, R12, XY>(pr, t_, par, edge);
}
// Waves per SIMD asked of the register allocator for the half-plane variant in
// FP16N, which left to itself takes 103 VGPRs (4 waves; FP32 76-81, FP64 127)
template <int P, int NR, bool XY> constexpr int eo_phaseB_waves() { return XY && NR == 1 && P == P16 ? 5 : 1; }
template <int P, int NR, bool R12 = false, bool XY = false>
__global__ __launch_bounds__(256, (eo_phaseB_waves<P, NR, XY>())) void k_eo_phaseB(const Prob *__restrict__ probs, int nprob, int remap, int par, int edge) {
    WD_KERNEL_PROLOGUE(KB)
    eo_phaseB_tile<P, NR, R12, XY>(pr, t_, par, edge);
}
template <int NR>
__global__ __launch_bounds__(256) void k_eo_ru2a(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KER2A)
    eo_ru2a_tile<NR>(pr, t_);
}
template <int P, int NR, bool ZX = false>
__global__ __launch_bounds__(256) void k_eo_ru2b(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KR2)
    eo_ru2b_tile<P, NR, ZX>(pr, t_);
}
__global__ __launch_bounds__(256) void k_eo_source(const Prob *__restrict__ probs) {
    eo_source_tile(probs[0], (int)blockIdx.x);
}

// canonical complex128 [rhs][V][12] -> FP64 half-lattice fields of the even and
// odd sites (packed layout, V/2 sites each)
__global__ __launch_bounds__(256) void k_eo_split(const Prob *__restrict__ probs, const double2 *__restrict__ in, void *even, void *odd) {
    const Prob &pr = probs[0];
    const int k = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
    if (k >= pr.vf) return;
    FieldPtr fe{even, pr.vf, pr.nrhs}, fo{odd, pr.vf, pr.nrhs};
    for (int par = 0; par < 2; ++par) {
        const int s = eo_site(pr.g, k, par);
        const double2 *src = in + ((size_t)r * pr.g.V + s) * 12;
        cx<double> v[12];
#pragma unroll
        for (int m = 0; m < 12; ++m) v[m] = {src[m].x, src[m].y};
        Spinor<P64>::store(par ? fo : fe, r, k, v);
    }
}

// x_o = (eta_o + H_oe x_e / 2) / A and the canonical complex128 solution
__global__ __launch_bounds__(256) void k_eo_merge(const Prob *__restrict__ probs, double2 *__restrict__ out) {
    const Prob &pr = probs[0];
    const int k = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
    if (k >= pr.vf) return;
    const Geom g = pr.g;
    FieldPtr fx{pr.x64, pr.vf, pr.nrhs}, fo{pr.eta_o, pr.vf, pr.nrhs};
    cx<double> v[12], acc[1][12];
    Spinor<P64>::load(fx, r, k, v);
    double2 *dst = out + ((size_t)r * g.V + eo_site(g, k, 0)) * 12;
#pragma unroll
    for (int m = 0; m < 12; ++m) dst[m] = make_double2(v[m].re, v[m].im);
    const int so = eo_site(g, k, 1);
    hopping<P64, false, 1, 1, false, true>(g, so, pr.U64, fx, r, 1u, acc);
    Spinor<P64>::load(fo, r, k, v);
    dst = out + ((size_t)r * g.V + so) * 12;
#pragma unroll
    for (int m = 0; m < 12; ++m)
        dst[m] = make_double2(fma(0.5, acc[0][m].re, v[m].re) / pr.diag, fma(0.5, acc[0][m].im, v[m].im) / pr.diag);
}

void launch_eo_split(const Prob *d, int64_t vf, int nrhs, const void *src, void *even, void *odd, hipStream_t st) {
    hipLaunchKernelGGL(k_eo_split, dim3((unsigned)((vf + 255) / 256), (unsigned)nrhs), dim3(256), 0, st, d,
                       (const double2 *)src, even, odd);
}
void launch_eo_source(const Prob *d, int64_t vf, int nrhs, hipStream_t st) {
    hipLaunchKernelGGL(k_eo_source, dim3((unsigned)(((vf + 255) / 256) * nrhs)), dim3(256), 0, st, d);
}
void launch_eo_merge(const Prob *d, int64_t vf, int nrhs, void *sol, hipStream_t st) {
    hipLaunchKernelGGL(k_eo_merge, dim3((unsigned)((vf + 255) / 256), (unsigned)nrhs), dim3(256), 0, st, d,
                       (double2 *)sol);
}

// The reduction of a phase as a launch of its own (one block): the kernel
// boundary makes every block's partial sums visible.  (Finishing it in the
// last block of the phase instead, found with an atomic ticket, needs a
// device-scope release fence in every block, which on a multi-XCD GPU writes
// back the XCD's L2 each time: the whole CG ran 1.4x slower that way.)
// kind | FIN_AB: phase B's finish after k_phaseB, which also completes phase A's.
// kind | FIN_TRAIL | parity << 12: the finish of the last iteration of a chunk
// run with the fused finish (K iterations, parity K & 1): the records that
// iteration's phase A wrote (pr.sc2 for an odd K, else pr.sc) and its phase A
// partials (slot 0 for an odd K, else slot 2) give the final records in pr.sc.
// KS5 | FIN_TRAIL_BI: the trailing finish of a chunk of fused BiCGSTAB iterations.
// FIN_SINGLE: x_lo is not updated in pairs (q stays in pr.q).
constexpr int FIN_AB = 0x100, FIN_TRAIL = 0x200, FIN_TRAIL_BI = 0x400, FIN_SINGLE = 0x800;
__global__ __launch_bounds__(1024) void k_finish(const Prob *__restrict__ probs, int nprob, int kind) {
    for (int j = 0; j < nprob; ++j) {
        const Prob &pr = probs[j];
        if (kind & FIN_TRAIL) {
            const int pk = (kind >> 12) & 1;
            phaseAB_finish(pr, pk ? pr.sc2 : pr.sc, pr.sc, pk ? 0 : 2, (kind & FIN_SINGLE) || pk ? 0 : 1);
            continue;
        }
        switch (kind) {
        case KA: phaseA_finish(pr); break;
        case KB: phaseB_finish(pr); break;
        case KB | FIN_AB: phaseAB_finish(pr); break;
        case KR2: ru2_finish(pr); break;
        case KN: norm_finish(pr); break;
        case KS2: bi2_finish(pr); break;
        case KS4: bi4_finish(pr); break;
        case KS5: bi5_finish(pr); break;
        case KS5 | FIN_TRAIL_BI: bi_trail_finish(pr); break;
        default: break;
        }
    }
}

// out[0] = right-hand sides still active or frozen over all problems,
// out[1] = the persistent kernel's abort flag (0 when there is none),
// out[2] = for one problem, an estimate of the iterations its active fields
// still need: |r|^2 of each is extrapolated at its rate of decrease since the
// previous summary (log-linear) down to the stopping value; -1 when unknown
// (several problems, a field without such a history).  The
// previous summary's |r|^2 and iteration count of each field sit 256 bytes
// after out (SumHist; the summary area has room for MAX_RHS of them) and are
// replaced.  One block of MAX_RHS threads.
struct SumHist {
    double rho;
    int iters, pad;
};
__global__ void k_summary(const Prob *__restrict__ probs, int nprob, int *out, const int *abort_flag) {
    __shared__ int unknown, need;
    const int i = threadIdx.x;
    if (i == 0) {
        int live = 0;
        for (int j = 0; j < nprob; ++j)
            for (int f = 0; f < probs[j].nrhs; ++f) {
                const int st = probs[j].sc[f].state;
                live += (st == ST_ACTIVE || st == ST_FROZEN);
            }
        out[0] = live;
        out[1] = abort_flag ? *abort_flag : 0;
        unknown = nprob != 1;
        need = 0;
    }
    __syncthreads();
    if (nprob == 1 && i < probs[0].nrhs) {
        const Scal &c = probs[0].sc[i];
        SumHist *h = (SumHist *)((char *)out + 256) + i;
        const SumHist prev = *h;
        if (c.state == ST_ACTIVE) {
            if (!(c.rho > c.stop2)) {
                atomicMax(&need, 1);
            } else if (c.stop2 > 0.0 && c.iters > prev.iters && prev.rho > c.rho) {
                const double rate = log(prev.rho / c.rho) / (double)(c.iters - prev.iters);
                const double n = log(c.rho / c.stop2) / rate;
                atomicMax(&need, n < 1e6 ? (int)ceil(n) : 1000000);
            } else {
                atomicOr(&unknown, 1);
            }
        }
        *h = SumHist{c.rho, c.iters, 0};
    }
    __syncthreads();
    if (i == 0) out[2] = unknown ? -1 : need;
}

// BiCGSTAB stages (bicgstab_core.h)
template <int P>
__global__ __launch_bounds__(256) void k_bi1(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KS1)
    bi1_tile<P>(pr, t_);
}

// F: the kernels of the fused iteration (F2, S3, F4, F5)
template <int P, int NR, bool S4, int ORD = 1, bool XY = false, bool R12 = false, bool F = false>
__global__ __launch_bounds__(256) void k_bi_stencil(const Prob *__restrict__ probs, int nprob, int remap, int first) {
    constexpr int K = S4 ? KS4 : KS2;
    WD_KERNEL_PROLOGUE(K)
    bi_stencil_tile<P, NR, S4, ORD, XY, R12, F>(pr, t_, first);
}

template <int P, bool F = false>
__global__ __launch_bounds__(256) void k_bi3(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KS3)
    bi3_tile<P, F>(pr, t_);
}

template <int P>
__global__ __launch_bounds__(256) void k_bi5f(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KS5)
    bi5f_tile<P>(pr, t_);
}

template <int P>
__global__ __launch_bounds__(256) void k_bi5(const Prob *__restrict__ probs, int nprob, int remap) {
    WD_KERNEL_PROLOGUE(KS5)
    bi5_tile<P>(pr, t_);
}

// x_lo <- 0 (a fill kernel rather than a memset, so it can sit in a graph)
__global__ void k_zero(uint4 *p, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

// ------------------------------------------------------------- launchers
// Profiling: while set, phase A/B/C tile kernels are launched with these
// start/stop events, which the runtime records at the kernel's own begin and
// end (no marker packets around the launch).
static thread_local hipEvent_t t_ev_start = nullptr, t_ev_stop = nullptr;
#define WD_TIMED_LAUNCH_LDS(K, grid, blk, lds, st, ...)                                            \
    do {                                                                                         \
        if (t_ev_start) hipExtLaunchKernelGGL(K, grid, blk, lds, st, t_ev_start, t_ev_stop, 0, __VA_ARGS__); \
        else hipLaunchKernelGGL(K, grid, blk, lds, st, __VA_ARGS__);                              \
    } while (0)
#define WD_TIMED_LAUNCH(K, grid, blk, st, ...) WD_TIMED_LAUNCH_LDS(K, grid, blk, 0, st, __VA_ARGS__)

// hop order 3 (pipelined) or 1 (one hop at a time) for the phase kernels;
// the plane-blocked (XY) variants exist for up to 2 rhs per thread (1 in FP64)
// reconstruct-12 variants: FP32 storage, plane or site blocks, 1 or 2 rhs per thread
template <int P, int ORD, bool B>
static void launch_AB_r12(int nr, int xy, int grid, int blk, hipStream_t st, const Prob *d, int n, int remap, int par, int first) {
    const dim3 gr(grid), bl(blk);
    if constexpr (P == P32) {
        if (xy) {
            if (nr == 2) {
                if (B) WD_TIMED_LAUNCH((k_phaseB<P, 2, ORD, true, true>), gr, bl, st, d, n, remap, par, first);
                else WD_TIMED_LAUNCH((k_phaseA<P, 2, ORD, true, true>), gr, bl, st, d, n, remap, par, first);
            } else {
                if (B) WD_TIMED_LAUNCH((k_phaseB<P, 1, ORD, true, true>), gr, bl, st, d, n, remap, par, first);
                else WD_TIMED_LAUNCH((k_phaseA<P, 1, ORD, true, true>), gr, bl, st, d, n, remap, par, first);
            }
        } else if (nr == 2) {
            if (B) WD_TIMED_LAUNCH((k_phaseB<P, 2, ORD, false, true>), gr, bl, st, d, n, remap, par, first);
            else WD_TIMED_LAUNCH((k_phaseA<P, 2, ORD, false, true>), gr, bl, st, d, n, remap, par, first);
        } else {
            if (B) WD_TIMED_LAUNCH((k_phaseB<P, 1, ORD, false, true>), gr, bl, st, d, n, remap, par, first);
            else WD_TIMED_LAUNCH((k_phaseA<P, 1, ORD, false, true>), gr, bl, st, d, n, remap, par, first);
        }
    }
}

// nontemporal-stream variants: FP64, plane blocks (1 rhs per thread) or site blocks (1 or 2)
template <int P, int ORD, bool B>
static void launch_AB_nt(int nr, int xy, int grid, int blk, hipStream_t st, const Prob *d, int n, int remap, int par, int first) {
    const dim3 gr(grid), bl(blk);
    if constexpr (P == P64) {
        if (xy) {
            if (B) WD_TIMED_LAUNCH((k_phaseB<P, 1, ORD, true, false, 1>), gr, bl, st, d, n, remap, par, first);
            else WD_TIMED_LAUNCH((k_phaseA<P, 1, ORD, true, false, 1>), gr, bl, st, d, n, remap, par, first);
        } else if (nr == 2) {
            if (B) WD_TIMED_LAUNCH((k_phaseB<P, 2, ORD, false, false, 1>), gr, bl, st, d, n, remap, par, first);
            else WD_TIMED_LAUNCH((k_phaseA<P, 2, ORD, false, false, 1>), gr, bl, st, d, n, remap, par, first);
        } else {
            if (B) WD_TIMED_LAUNCH((k_phaseB<P, 1, ORD, false, false, 1>), gr, bl, st, d, n, remap, par, first);
            else WD_TIMED_LAUNCH((k_phaseA<P, 1, ORD, false, false, 1>), gr, bl, st, d, n, remap, par, first);
        }
    }
}

template <int P, int ORD, bool B>
static void launch_AB_o(int nr, int xy, int lds, int r12, int nt, int grid, int blk, hipStream_t st, const Prob *d,
                        int n, int remap, int par, int first) {
    const dim3 gr(grid), bl(blk);
    if (r12) {
        launch_AB_r12<P, ORD, B>(nr, xy, grid, blk, st, d, n, remap, par, first);
        return;
    }
    if (nt == 1) {
        launch_AB_nt<P, ORD, B>(nr, xy, grid, blk, st, d, n, remap, par, first);
        return;
    }
    if (xy == 2) {
        if constexpr (P != P64) {
            if (B) WD_TIMED_LAUNCH_LDS((k_phaseB_zm<P, ORD>), gr, bl, lds, st, d, n, remap);
            else WD_TIMED_LAUNCH_LDS((k_phaseA_zm<P, ORD>), gr, bl, lds, st, d, n, remap);
        }
        return;
    }
    if (xy) {
        if (nr == 2 && P != P64) {
            if (B) WD_TIMED_LAUNCH((k_phaseB<P, 2, ORD, true>), gr, bl, st, d, n, remap, par, first);
            else WD_TIMED_LAUNCH((k_phaseA<P, 2, ORD, true>), gr, bl, st, d, n, remap, par, first);
        } else {
            if (B) WD_TIMED_LAUNCH((k_phaseB<P, 1, ORD, true>), gr, bl, st, d, n, remap, par, first);
            else WD_TIMED_LAUNCH((k_phaseA<P, 1, ORD, true>), gr, bl, st, d, n, remap, par, first);
        }
        return;
    }
    if (nr == 1) {
        if (B) WD_TIMED_LAUNCH((k_phaseB<P, 1, ORD, false>), gr, bl, st, d, n, remap, par, first);
        else WD_TIMED_LAUNCH((k_phaseA<P, 1, ORD, false>), gr, bl, st, d, n, remap, par, first);
    } else if (nr == 2) {
        if (B) WD_TIMED_LAUNCH((k_phaseB<P, 2, ORD, false>), gr, bl, st, d, n, remap, par, first);
        else WD_TIMED_LAUNCH((k_phaseA<P, 2, ORD, false>), gr, bl, st, d, n, remap, par, first);
    } else {
        if (B) WD_TIMED_LAUNCH((k_phaseB<P, 4, ORD, false>), gr, bl, st, d, n, remap, par, first);
        else WD_TIMED_LAUNCH((k_phaseA<P, 4, ORD, false>), gr, bl, st, d, n, remap, par, first);
    }
}
// hop order 5 (the memory hops z and t first, then the LDS hops x and y):
// plane-blocked variants with one rhs per thread, by the streams' cache policy
template <int P, int POL, bool R12, bool MP, bool B>
static void launch_AB_5(const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int edge) {
    const dim3 gr(k.grid), bl(k.block);
    if (B) WD_TIMED_LAUNCH((k_phaseB<P, 1, 5, true, R12, POL, MP>), gr, bl, st, d, n, k.remap, par, edge);
    else WD_TIMED_LAUNCH((k_phaseA<P, 1, 5, true, R12, POL, MP>), gr, bl, st, d, n, k.remap, par, edge);
}
template <int P, bool B>
static void launch_AB_o5(const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int edge) {
    const bool mp = k.planes > 1;   // several planes per block: FP32 and FP16 storage
    if constexpr (P == P64) {
        if (k.nt == 0) launch_AB_5<P, 0, false, false, B>(k, st, d, n, par, edge);
        else if (k.nt == 1) launch_AB_5<P, 1, false, false, B>(k, st, d, n, par, edge);
        else launch_AB_5<P, 2, false, false, B>(k, st, d, n, par, edge);
    } else if (P == P32 && k.r12) {
        if (k.nt == 3) mp ? launch_AB_5<P, 3, P == P32, true, B>(k, st, d, n, par, edge)
                          : launch_AB_5<P, 3, P == P32, false, B>(k, st, d, n, par, edge);
        else mp ? launch_AB_5<P, 0, P == P32, true, B>(k, st, d, n, par, edge)
                : launch_AB_5<P, 0, P == P32, false, B>(k, st, d, n, par, edge);
    } else {
        if (k.nt == 3) mp ? launch_AB_5<P, 3, false, true, B>(k, st, d, n, par, edge)
                          : launch_AB_5<P, 3, false, false, B>(k, st, d, n, par, edge);
        else mp ? launch_AB_5<P, 0, false, true, B>(k, st, d, n, par, edge)
                : launch_AB_5<P, 0, false, false, B>(k, st, d, n, par, edge);
    }
}

template <int P, bool B>
static void launch_split(const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int edge) {
    const dim3 gr(k.grid), bl(k.block);
    if constexpr (P == P32)
        if (k.r12) {
            WD_TIMED_LAUNCH_LDS((k_phase_split<P, true, B>), gr, bl, k.lds, st, d, n, k.remap, par, edge);
            return;
        }
    WD_TIMED_LAUNCH_LDS((k_phase_split<P, false, B>), gr, bl, k.lds, st, d, n, k.remap, par, edge);
}

// site blocks with x_lo updated in pairs (site_pair; FP64: nontemporal streams)
template <int P, bool B>
static void launch_pair(const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int edge) {
    const dim3 gr(k.grid), bl(k.block);
    auto go = [&](auto a, auto b) {
        if (B) WD_TIMED_LAUNCH(b, gr, bl, st, d, n, k.remap, par, edge);
        else WD_TIMED_LAUNCH(a, gr, bl, st, d, n, k.remap, par, edge);
    };
    constexpr int POL = P == P64 ? 1 : 0;
    if (P == P32 && k.r12)
        go(k_phaseA<P, 1, 3, false, P == P32, POL, false, true>, k_phaseB<P, 1, 3, false, P == P32, POL, false, true>);
    else go(k_phaseA<P, 1, 3, false, false, POL, false, true>, k_phaseB<P, 1, 3, false, false, POL, false, true>);
}

template <int P>
static void launch_A(const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int first) {
    if (k.split) {
        launch_split<P, false>(k, st, d, n, par, first);
        return;
    }
    if (k.pair && !k.xy) {
        launch_pair<P, false>(k, st, d, n, par, first);
        return;
    }
    if (k.ordered == 5) launch_AB_o5<P, false>(k, st, d, n, par, first);
    else if (k.ordered == 3)
        launch_AB_o<P, 3, false>(k.nr, k.xy, k.lds, k.r12, k.nt, k.grid, k.block, st, d, n, k.remap, par, first);
    else launch_AB_o<P, 1, false>(k.nr, k.xy, k.lds, k.r12, k.nt, k.grid, k.block, st, d, n, k.remap, par, first);
}
template <int P>
static void launch_B(const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int last) {
    if (k.split) {
        launch_split<P, true>(k, st, d, n, par, last);
        return;
    }
    if (k.pair && !k.xy) {
        launch_pair<P, true>(k, st, d, n, par, last);
        return;
    }
    if (k.ordered == 5) launch_AB_o5<P, true>(k, st, d, n, par, last);
    else if (k.ordered == 3)
        launch_AB_o<P, 3, true>(k.nr, k.xy, k.lds, k.r12, k.nt, k.grid, k.block, st, d, n, k.remap, par, last);
    else launch_AB_o<P, 1, true>(k.nr, k.xy, k.lds, k.r12, k.nt, k.grid, k.block, st, d, n, k.remap, par, last);
}
template <int P, bool ZX = false>
static void launch_R2(int nr, int xy, int grid, int blk, hipStream_t st, const Prob *d, int n, int remap) {
    if (xy) hipLaunchKernelGGL((k_ru2<P, 1, true, ZX>), dim3(grid), dim3(blk), 0, st, d, n, remap);
    else if (nr == 1) hipLaunchKernelGGL((k_ru2<P, 1, false, ZX>), dim3(grid), dim3(blk), 0, st, d, n, remap);
    else hipLaunchKernelGGL((k_ru2<P, 2, false, ZX>), dim3(grid), dim3(blk), 0, st, d, n, remap);
}

// plane blocks (xy): hop order 5, one rhs per thread, the reconstruct-12
// links in FP32 when the gauge has them
template <int P, bool S4, bool F>
static void launch_BS(const KindShape &k, hipStream_t st, const Prob *d, int n, int first) {
    const dim3 gr(k.grid), bl(k.block);
    if (k.xy) {
        if constexpr (P == P32)
            if (k.r12) {
                hipLaunchKernelGGL((k_bi_stencil<P, 1, S4, 5, true, true, F>), gr, bl, 0, st, d, n, k.remap, first);
                return;
            }
        hipLaunchKernelGGL((k_bi_stencil<P, 1, S4, 5, true, false, F>), gr, bl, 0, st, d, n, k.remap, first);
    } else if (k.nr == 1) hipLaunchKernelGGL((k_bi_stencil<P, 1, S4, 1, false, false, F>), gr, bl, 0, st, d, n, k.remap, first);
    else if (k.nr == 2) hipLaunchKernelGGL((k_bi_stencil<P, 2, S4, 1, false, false, F>), gr, bl, 0, st, d, n, k.remap, first);
    else hipLaunchKernelGGL((k_bi_stencil<P, 4, S4, 1, false, false, F>), gr, bl, 0, st, d, n, k.remap, first);
}
// fused: the fused iteration's kernels (first: a chunk's first iteration)
template <int P>
static void launch_bicg(int kind, const KindShape &k, hipStream_t st, const Prob *d, int n, int fused, int first) {
    const dim3 gr(k.grid), bl(k.block);
    switch (kind) {
    case KS1: hipLaunchKernelGGL(k_bi1<P>, gr, bl, 0, st, d, n, 0); break;
    case KS2:
        if (fused) launch_BS<P, false, true>(k, st, d, n, first);
        else launch_BS<P, false, false>(k, st, d, n, 0);
        break;
    case KS3:
        if (fused) hipLaunchKernelGGL((k_bi3<P, true>), gr, bl, 0, st, d, n, 0);
        else hipLaunchKernelGGL((k_bi3<P, false>), gr, bl, 0, st, d, n, 0);
        break;
    case KS4:
        if (fused) launch_BS<P, true, true>(k, st, d, n, 0);
        else launch_BS<P, true, false>(k, st, d, n, 0);
        break;
    case KS5:
        if (fused) hipLaunchKernelGGL(k_bi5f<P>, gr, bl, 0, st, d, n, 0);
        else hipLaunchKernelGGL(k_bi5<P>, gr, bl, 0, st, d, n, 0);
        break;
    }
}

static void launch_kind_tiles(int kind, int inner, const KindShape &k, hipStream_t st, const Prob *d, int nprob,
                              int par = -1, int first = 0);

static void launch_finish(int kind, hipStream_t st, const Prob *d, int nprob) {
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(1024), 0, st, d, nprob, kind);
}

// The finish after the tiles of `kind`.  Phase B by k_phaseB (not even-odd,
// not z-marching) completes phase A's reduction in its blocks: then phase A
// has no finish and phase B's finishes both.
static void launch_finish_after(int kind, const LaunchSet &ls, hipStream_t st, const Prob *d, int nprob) {
    const bool fa = !ls.eo && ls.k[KB].xy != 2;
    if (kind == KA && fa) return;
    launch_finish(kind == KB && fa ? (KB | FIN_AB) : kind, st, d, nprob);
}

// The even-odd hops of phases A and B, one kernel of the kind with the template
// arguments given (links R12, half-plane blocks XY).  par, edge: as for
// k_phaseA and k_phaseB.
template <int P, int NR, bool R12, bool XY>
static void launch_eo_AB(int kind, const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int edge) {
    const dim3 gr(k.grid), bl(k.block);
    const size_t lds = XY ? k.lds : 0;   // the half-plane's spinors
    switch (kind) {
    case KEA1: hipLaunchKernelGGL((k_eo_hop1<P, NR, true, R12, XY>), gr, bl, lds, st, d, n, k.remap, par, edge); break;
    case KEB1: hipLaunchKernelGGL((k_eo_hop1<P, NR, false, R12, XY>), gr, bl, lds, st, d, n, k.remap, par, edge); break;
    case KA: hipLaunchKernelGGL((k_eo_phaseA<P, NR, R12, XY>), gr, bl, lds, st, d, n, k.remap, par, edge); break;
    case KB: hipLaunchKernelGGL((k_eo_phaseB<P, NR, R12, XY>), gr, bl, lds, st, d, n, k.remap, par, edge); break;
    }
}
// even-odd kernels of the stencil kinds: half-plane blocks (one rhs per thread)
// or site blocks (1 or 2); the reconstruct-12 links in FP32 where the gauge has them
template <int P>
static void launch_eo(int kind, const KindShape &k, hipStream_t st, const Prob *d, int n, int par, int edge) {
    const dim3 gr(k.grid), bl(k.block);
    const bool two = k.nr >= 2;
    if (kind == KER2A) {
        if (two) hipLaunchKernelGGL((k_eo_ru2a<2>), gr, bl, 0, st, d, n, k.remap);
        else hipLaunchKernelGGL((k_eo_ru2a<1>), gr, bl, 0, st, d, n, k.remap);
    } else if (kind == KR2) {
        if (two) hipLaunchKernelGGL((k_eo_ru2b<P, 2>), gr, bl, 0, st, d, n, k.remap);
        else hipLaunchKernelGGL((k_eo_ru2b<P, 1>), gr, bl, 0, st, d, n, k.remap);
    } else if (P == P32 && k.r12) {   // R12: FP32 only
        if (k.xy) launch_eo_AB<P, 1, P == P32, true>(kind, k, st, d, n, par, edge);
        else if (two) launch_eo_AB<P, 2, P == P32, false>(kind, k, st, d, n, par, edge);
        else launch_eo_AB<P, 1, P == P32, false>(kind, k, st, d, n, par, edge);
    } else {
        if (k.xy) launch_eo_AB<P, 1, false, true>(kind, k, st, d, n, par, edge);
        else if (two) launch_eo_AB<P, 2, false, false>(kind, k, st, d, n, par, edge);
        else launch_eo_AB<P, 1, false, false>(kind, k, st, d, n, par, edge);
    }
}

void launch_kind(int kind, int inner, const LaunchSet &ls, hipStream_t st, const Prob *d, int nprob, int par,
                 int first) {
    const KindShape &k = ls.k[kind];
    if (k.grid <= 0) return;
    if (kind == KC && ls.qrec) return;   // phase A forms the direction in q
    const bool reduces = kind == KA || kind == KB || kind == KR2 || kind == KN || kind == KS2 || kind == KS4 ||
                         kind == KS5;
    const bool eo_kind = kind == KA || kind == KB || kind == KR2 || kind == KEA1 || kind == KEB1 || kind == KER2A;
    if (ls.eo && eo_kind) {
        if (inner == P64) launch_eo<P64>(kind, k, st, d, nprob, par, first);
        else if (inner == P32) launch_eo<P32>(kind, k, st, d, nprob, par, first);
        else launch_eo<P16>(kind, k, st, d, nprob, par, first);
    } else {
        launch_kind_tiles(kind, inner, k, st, d, nprob, par, first);
    }
    // with the fused finish, phase A finishes the previous iteration and a
    // trailing finish the chunk's last (launch_iterations)
    if (reduces && !(par >= 0 && kind != KR2 && kind != KN)) launch_finish_after(kind, ls, st, d, nprob);
}

// The first true residual of a solve (R2).  x_zero: x64 is zero (no initial
// guess), so r = eta is formed without the FP64 stencil (bitwise the same).
void launch_first_residual(int inner, const LaunchSet &ls, hipStream_t st, const Prob *d, int nprob, bool x_zero) {
    if (!x_zero) {
        if (ls.eo) launch_kind(KER2A, inner, ls, st, d, nprob);
        launch_kind(KR2, inner, ls, st, d, nprob);
        return;
    }
    const KindShape &k = ls.k[KR2];
    if (k.grid <= 0) return;
    if (ls.eo) {   // one rhs per thread: nothing shared between fields without the hops
        const dim3 gr(k.grid), bl(k.block);
        const bool two = k.nr >= 2;
        auto zx = [&](auto one, auto pair) {
            hipLaunchKernelGGL(two ? pair : one, gr, bl, 0, st, d, nprob, k.remap);
        };
        if (inner == P64) zx(k_eo_ru2b<P64, 1, true>, k_eo_ru2b<P64, 2, true>);
        else if (inner == P32) zx(k_eo_ru2b<P32, 1, true>, k_eo_ru2b<P32, 2, true>);
        else zx(k_eo_ru2b<P16, 1, true>, k_eo_ru2b<P16, 2, true>);
        launch_finish(KR2, st, d, nprob);
        return;
    }
    if (inner == P64) launch_R2<P64, true>(k.nr, k.xy, k.grid, k.block, st, d, nprob, k.remap);
    else if (inner == P32) launch_R2<P32, true>(k.nr, k.xy, k.grid, k.block, st, d, nprob, k.remap);
    else launch_R2<P16, true>(k.nr, k.xy, k.grid, k.block, st, d, nprob, k.remap);
    launch_finish(KR2, st, d, nprob);
}

void launch_iterations(int inner, const LaunchSet &ls, hipStream_t st, const Prob *d, int nprob, int K) {
    if (ls.fused) {
        for (int it = 0; it < K; ++it) {
            if (ls.eo) launch_kind(KEA1, inner, ls, st, d, nprob, it & 1, 0);
            launch_kind(KA, inner, ls, st, d, nprob, it & 1, it == 0);
            if (ls.eo) launch_kind(KEB1, inner, ls, st, d, nprob, it & 1, 0);
            launch_kind(KB, inner, ls, st, d, nprob, it & 1, it == K - 1);
        }
        hipLaunchKernelGGL(k_finish, dim3(1), dim3(1024), 0, st, d, nprob,
                           KB | FIN_AB | FIN_TRAIL | ((K & 1) << 12) | (ls.eo || ls.k[KB].pair ? 0 : FIN_SINGLE));
        return;
    }
    for (int it = 0; it < K; ++it) {
        if (ls.eo) launch_kind(KEA1, inner, ls, st, d, nprob);
        launch_kind(KA, inner, ls, st, d, nprob);
        if (ls.eo) launch_kind(KEB1, inner, ls, st, d, nprob);
        launch_kind(KB, inner, ls, st, d, nprob);
        launch_kind(KC, inner, ls, st, d, nprob);
    }
}

static void launch_kind_tiles(int kind, int inner, const KindShape &k, hipStream_t st, const Prob *d, int nprob,
                              int par, int first) {
    switch (kind) {
    case KA:
        if (inner == P64) launch_A<P64>(k, st, d, nprob, par, first);
        else if (inner == P32) launch_A<P32>(k, st, d, nprob, par, first);
        else launch_A<P16>(k, st, d, nprob, par, first);
        break;
    case KB:
        if (inner == P64) launch_B<P64>(k, st, d, nprob, par, first);
        else if (inner == P32) launch_B<P32>(k, st, d, nprob, par, first);
        else launch_B<P16>(k, st, d, nprob, par, first);
        break;
    case KC:
        if (inner == P64) WD_TIMED_LAUNCH(k_phaseC<P64>, dim3(k.grid), dim3(k.block), st, d, nprob, 0);
        else if (inner == P32) WD_TIMED_LAUNCH(k_phaseC<P32>, dim3(k.grid), dim3(k.block), st, d, nprob, 0);
        else WD_TIMED_LAUNCH(k_phaseC<P16>, dim3(k.grid), dim3(k.block), st, d, nprob, 0);
        break;
    case KR1:
        if (inner == P64) hipLaunchKernelGGL(k_ru1<P64>, dim3(k.grid), dim3(k.block), 0, st, d, nprob, 0);
        else if (inner == P32) hipLaunchKernelGGL(k_ru1<P32>, dim3(k.grid), dim3(k.block), 0, st, d, nprob, 0);
        else hipLaunchKernelGGL(k_ru1<P16>, dim3(k.grid), dim3(k.block), 0, st, d, nprob, 0);
        break;
    case KR2:
        if (inner == P64) launch_R2<P64>(k.nr, k.xy, k.grid, k.block, st, d, nprob, k.remap);
        else if (inner == P32) launch_R2<P32>(k.nr, k.xy, k.grid, k.block, st, d, nprob, k.remap);
        else launch_R2<P16>(k.nr, k.xy, k.grid, k.block, st, d, nprob, k.remap);
        break;
    case KN:
        hipLaunchKernelGGL(k_norm, dim3(k.grid), dim3(k.block), 0, st, d, nprob, 0);
        break;
    case KS1: case KS2: case KS3: case KS4: case KS5:
        if (inner == P64) launch_bicg<P64>(kind, k, st, d, nprob, par >= 0, first);
        else if (inner == P32) launch_bicg<P32>(kind, k, st, d, nprob, par >= 0, first);
        else launch_bicg<P16>(kind, k, st, d, nprob, par >= 0, first);
        break;
    }
}

void launch_summary(hipStream_t st, const Prob *d, int nprob, int *out, const int *abort_flag) {
    hipLaunchKernelGGL(k_summary, dim3(1), dim3(MAX_RHS), 0, st, d, nprob, out, abort_flag);
}

void launch_zero(void *p, size_t bytes, hipStream_t st) {
    const size_t n16 = bytes / 16;
    const int grid = (int)std::min<size_t>((n16 + 255) / 256, 4096);
    if (grid > 0) hipLaunchKernelGGL(k_zero, dim3(grid), dim3(256), 0, st, (uint4 *)p, n16);
}

// ------------------------------------------------------------- host plan
static size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

WsLayout ws_layout(int64_t V, int nrhs, int inner, int method, int eo) {
    WsLayout L;
    size_t o = 0;
    const int64_t Vf = eo ? V / 2 : V;   // sites of a vector
    L.prob = o; o += al256(sizeof(Prob));
    L.scal = o; o += al256(sizeof(Scal) * nrhs);
    L.scal2 = o; o += al256(sizeof(Scal) * nrhs);
    L.bar = o; o += BAR_BYTES;
    L.summary = o; o += 256 + al256(sizeof(SumHist) * MAX_RHS);
    L.part = o; o += al256((size_t)((V + 63) / 64) * nrhs * PSTRIDE * sizeof(double));
    L.eta64 = o; o += al256(spinor_bytes(WD_F64, Vf, nrhs));
    L.x64 = o; o += al256(spinor_bytes(WD_F64, Vf, nrhs));
    const int xp = inner == WD_F16N ? WD_F32 : inner;
    L.xlo = o; o += al256(spinor_bytes(xp, Vf, nrhs));
    L.r = o; o += al256(spinor_bytes(inner, Vf, nrhs));
    L.p = o; o += al256(spinor_bytes(inner, Vf, nrhs));
    L.q = o; o += al256(spinor_bytes(inner, Vf, nrhs));   // BiCGSTAB: v
    L.bscal = L.rh = L.sv = L.tv = 0;
    L.eta_o = L.tmp = L.w64 = 0;
    if (eo) {
        L.eta_o = o; o += al256(spinor_bytes(WD_F64, Vf, nrhs));
        L.tmp = o; o += al256(spinor_bytes(inner, Vf, nrhs));
        L.w64 = o; o += al256(spinor_bytes(WD_F64, Vf, nrhs));
    }
    if (method == METHOD_BICGSTAB) {
        L.bscal = o; o += al256(sizeof(BScal) * nrhs);
        L.rh = o; o += al256(spinor_bytes(inner, V, nrhs));
        L.sv = o; o += al256(spinor_bytes(inner, V, nrhs));
        L.tv = o; o += al256(spinor_bytes(inner, V, nrhs));
    }
    L.least = o;
    L.bi_part2 = L.bi_rec = 0;
    if (method == METHOD_BICGSTAB) {
        L.bi_part2 = o; o += al256((size_t)((V + 63) / 64) * nrhs * BI_NP2 * sizeof(double));
        L.bi_rec = o; o += al256(3 * sizeof(BiRec) * nrhs);
    }
    L.total = o;
    return L;
}

// Launch shapes of every kernel kind for one problem (tiles start at 0).
bool unfused_requested() {
    const char *v = getenv("WD_CG_UNFUSED");
    return v && *v && strcmp(v, "0") != 0;
}

// bytes of the fields an iteration touches: r, q in two buffers, x_lo
static size_t iterated_bytes(int inner, int64_t Vf, int nrhs) {
    return 3 * spinor_bytes(inner, Vf, nrhs) + spinor_bytes(inner == WD_F16N ? WD_F32 : inner, Vf, nrhs);
}

// Cache policy (see ld) of the phases' streaming accesses, by whether the fields
// an iteration touches (r, q in two buffers, x_lo) fit the 256 MB MALL.  They do:
// plain (0), but device-scope accesses (2) in FP64 from 128 MB on, which leave
// the L2 to the gathered field: whole solves, plain against device-scope, 12^4 x 12
// 12.55 -> 12.28 ms (nontemporal 13.3), 8 x 8 x 14 x 28 x 10 21.7 -> 20.9, 16^4 x 4
// 16.3 -> 15.8, 14^4 x 8 19.6 -> 19.2, 12 x 12 x 16 x 20 x 5 15.6 -> 15.3, 14 x 10 x
// 12 x 24 x 5 13.78 -> 13.72, and by 1 to 2 % on four lattices more in the window;
// 14^4 x 2, of which the L2s hold a good part, 5.62 -> 5.85 ms.  In FP32 device-scope accesses are not kept: 14^4 x 16 15.7 ->
// 15.5 ms, but 14 x 10 x 12 x 24 x 5 6.54 -> 7.02, 8 x 8 x 14 x 28 x 10 9.8 -> 10.4
// ms.  They do not fit: FP64 nontemporal (1), 14^4 x 16 plain 33.8, device-scope
// 34.0, nontemporal 30.8 ms; FP32 and FP16N nontemporal loads with device-scope
// stores (3), 16^3 x 32 x 6 FP32 20.8 -> 19.3 ms (nontemporal both ways 19.9), x 12
// FP16N 30.5 -> 29.1 ms; below that size 14^4 x 16 FP32 takes 17.3 ms with it: it
// gives up the MALL's copies.
static int stream_policy(int inner, size_t bytes) {
    if (bytes <= (size_t)256 << 20) return inner == WD_F64 && bytes >= (size_t)128 << 20 ? 2 : 0;
    return inner == WD_F64 ? 1 : 3;
}

void plan_shapes(const wd_gauge *g, int nrhs, int inner, LaunchSet &ls, Prob &pr) {
    const int V = (int)g->V;
    const int np = g->dims[0] * g->dims[1];
    const Geom geo = make_geom(g);
    ShapeKey ka{{g->dims[0], g->dims[1], g->dims[2], g->dims[3]}, inner, nrhs, 1, FAM_CG_A};
    ShapeKey kb = ka;
    kb.dag = 0;
    kb.fam = FAM_CG_B;
    ShapeKey kr = kb;
    kr.prec = WD_F64;
    kr.fam = FAM_CG_R;
    Shape sa = shape_lookup(ka), sb = shape_lookup(kb), sr = shape_lookup(kr);
    if (sr.nr > 2) sr.nr = 2;
    // stencil kinds: A (D^dagger), B, S2 and S4 (D), R2 (FP64 D); the rest stream
    // even-odd: the first half hops take the shape of their phase
    const Shape *st[NKIND] = {&sa, &sb, nullptr, nullptr, &sr, nullptr, nullptr, &sb, nullptr, &sb, nullptr,
                              &sa, &sb, &sr};
    const int Vf = pr.vf;
    ls.eo = pr.eo;
    const size_t iterated = iterated_bytes(inner, Vf, nrhs);
    const int policy = stream_policy(inner, iterated);
    for (int k = 0; k < NKIND; ++k) {
        KindShape &ks = ls.k[k];
        if (st[k]) {
            ks.block = st[k]->block;
            ks.nr = st[k]->nr;
            ks.remap = st[k]->remap;
            ks.ordered = (k == KA || k == KB) && (st[k]->ordered == 3 || st[k]->ordered == 5) ? st[k]->ordered : 1;
            const int strip = (st[k]->strip > 0 && st[k]->strip < g->dims[2]) ? st[k]->strip : 0;
            ks.order = strip | (st[k]->gmajor ? 1 << 16 : 0) | (st[k]->fpass << 24);
            // plane-blocked phases A and B, reliable update and BiCGSTAB
            // stencils: one xy-plane of 64..256 sites per block (the
            // partial-sum buffer holds one entry per 64 sites)
            ks.xy = (k == KA || k == KB || k == KR2 || k == KS2 || k == KS4) && st[k]->xylds && np >= 64 &&
                    np <= 256 && !pr.eo;
            if (pr.eo) {   // the half-lattice kernels: lexicographic order (half-plane blocks below)
                ks.order = 0;
                if (ks.nr > 2) ks.nr = 2;
            }
            if (ks.xy) {
                ks.block = 256;
                if (ks.nr > 2) ks.nr = 2;
                if (inner == WD_F64 || k == KR2) ks.nr = 1;   // FP64 planes: one rhs per thread
                ks.order |= 1 << 17;
            }
            // z-marching columns of planes (FP32 and FP16 storage, one rhs per
            // tile); strip = number of z-chunks, by default enough for about
            // three tiles per compute unit with chunks of at least two planes
            if (ks.xy && st[k]->xylds == 2 && inner != WD_F64 && g->dims[2] >= 2 && k != KS2 && k != KS4) {
                const int Lz = g->dims[2], Lt = g->dims[3];
                int nzc = st[k]->strip > 0 ? std::min(st[k]->strip, Lz)
                                           : std::min((768 + Lt * nrhs - 1) / (Lt * nrhs), Lz / 2);
                if (nzc < 1) nzc = 1;
                ks.xy = 2;
                ks.nr = 1;
                ks.order = nzc;
                ks.lds = 2 * 6 * np * 16;   // two planes of 6 float4 per site
            }
            // cache policy of phases A and B's streams: the plane-blocked kernels with
            // hop order 5, and nontemporal streams in the other FP64 ones
            if ((k == KA || k == KB) && ks.xy != 2 && !pr.eo) {
                const bool five = ks.xy == 1 && ks.ordered == 5 && ks.nr == 1;
                ks.nt = five || policy == 1 ? policy : 0;
                if (ks.nt == 1 && ks.nr > 2) ks.nr = 2;
            }
            // reconstruct-12 links for phases A and B (FP32; plane or site blocks, <= 2 rhs per thread;
            // even-odd: both half-lattice hops of each phase)
            if ((k == KA || k == KB || (pr.eo && (k == KEA1 || k == KEB1))) && pr.U12 && ks.xy != 2) {
                ks.r12 = 1;
                if (ks.nr > 2) ks.nr = 2;
            }
            // BiCGSTAB's stencils on plane blocks: hop order 5, one rhs per
            // thread, the reconstruct-12 links where the gauge has them (FP32)
            if ((k == KS2 || k == KS4) && ks.xy == 1) {
                ks.nr = 1;
                ks.ordered = 5;
                ks.r12 = pr.U12 != nullptr;
            }
            // even-odd: the phases' half-lattice hops on half-plane blocks (the
            // Lx Ly / 2 sites of one parity on an xy-plane, 64..256 of them),
            // one rhs per thread, hop order 5.  FP16N, whose coding keeps the
            // phases bound by issue: site blocks from more than one to two
            // half-plane blocks per compute unit, whatever the phases' shapes ask
            // for.  Whole solves, site against half-plane blocks (of 128): 16 x 16 x
            // 8 x 9 x 4 (288 blocks) 3.97 -> 4.42, 16 x 16 x 8 x 8 x 6 (384) 3.85 ->
            // 4.37, 16^3 x 32 x 1 (512) 4.98 -> 5.76 ms; but 16^4 x 1 (256) 3.68 ->
            // 3.62, 16 x 16 x 12 x 12 x 4 (576) 5.20 -> 4.97, 16 x 16 x 10 x 16 x 4
            // (640) 5.38 -> 5.09, 16^4 x 3 (768) 5.42 -> 5.23, 16^3 x 32 x 4 (2048)
            // 9.25 -> 9.08 ms
            if (pr.eo && (k == KA || k == KB || k == KEA1 || k == KEB1)) {
                const int nh = np / 2;
                const int64_t hb = (int64_t)V / np * nrhs;
                const bool idle = inner == WD_F16N && hb > 256 && hb <= 512;
                ks.xy = st[k]->xylds && nh >= 64 && nh <= 256 && !idle ? 1 : 0;
                ks.order = 0;
                if (ks.xy) {
                    ks.block = (nh + 63) & ~63;
                    ks.nr = 1;
                    ks.ordered = 5;
                    ks.lds = nh * (inner == WD_F64 ? 192 : 96);   // the half-plane in LDS
                }
            }
            // hop order 5 exists for plane blocks with one rhs per thread
            if (ks.ordered == 5 && !(ks.xy == 1 && ks.nr == 1)) ks.ordered = 3;
            // several z-adjacent planes per block (FP32 / FP16 storage, hop order 5);
            // the block is rounded up to whole wavefronts for the block sums
            ks.planes = 1;
            if ((k == KA || k == KB) && ks.xy == 1 && ks.nr == 1 && ks.ordered == 5 && !pr.eo) {
                const int kp = xy_planes(*st[k], geo, inner, 1);
                if (kp > 1) {
                    ks.planes = kp;
                    ks.block = (kp * np + 63) & ~63;
                    ks.order |= kp << 18;
                }
                // direction split: at most one plane block per compute unit, or two
                // of 64 sites.  Whole solves, plain against split: 8^4 FP32 1 / 8
                // fields 2.10 -> 1.83, 2.55 -> 2.31 ms (16 fields, 1024 blocks, 2.82
                // -> 2.69; FP16N none), FP64 x 4 2.56 -> 2.35, 10x10x8x8 x 3 2.37 ->
                // 2.12, 14^4 x 1 (196 blocks) 2.83 -> 2.75 ms; but 12^4 x 2 (288
                // blocks of 768 threads) 2.97 -> 4.22 ms: the second round of blocks
                const int npr = (np + 63) & ~63, lds = split_lds_bytes(inner, np), blocks = V / np * nrhs;
                if (kp == 1 && blocks <= (np == 64 ? 512 : 256) && lds <= 65536 &&
                    4 * npr <= (inner == WD_F64 ? 512 : 1024)) {
                    ks.split = 1;
                    ks.block = 4 * npr;
                    ks.lds = lds;
                }
            }
            if ((k == KA || k == KB) && !pr.eo)
                ks.pair = ks.xy == 1 ||
                          (ks.xy == 0 && site_pair(inner, ks.ordered, ks.nr, iterated, (int64_t)Vf * nrhs));
        } else {
            ks.block = 256;
            ks.nr = 1;
            ks.remap = 0;
            ks.order = 0;
            ks.xy = 0;
        }
        pr.sorder[k] = ks.order;
        pr.nsb[k] = ks.xy == 2 ? ks.order * g->dims[3] : ks.xy ? V / (np * ks.planes) : (Vf + ks.block - 1) / ks.block;
        pr.ng[k] = (nrhs + ks.nr - 1) / ks.nr;
        pr.t0[k] = 0;
        pr.nt[k] = pr.nsb[k] * pr.ng[k];
        ks.grid = pr.nt[k];
    }
    // phase A by k_phaseA or the even-odd kernels (not z-marching) carries the
    // direction as q
    ls.qrec = ls.eo || ls.k[KA].xy != 2;
    // phase A completes the previous iteration's finish: plane or site blocks
    // with phase A's reduction inside phase B, even-odd or not (not
    // z-marching).  WD_CG_UNFUSED=1 selects the iteration with finish launches
    // instead (the same arithmetic; kept for comparisons), and so do shapes set
    // for one phase only that pair x_lo's updates differently.
    ls.fused = ls.k[KA].xy != 2 && ls.k[KB].xy != 2 && ls.k[KA].pair == ls.k[KB].pair && !unfused_requested();
}

// The persistent kernel runs phases A and B with one block shape, site blocks
// and one hop at a time.  FP32 and FP16 storage with one rhs per thread (the
// default shapes), or a launch limited to max_cus compute units: one
// 1024-thread block per compute unit (all of them, or max_cus), the
// reconstruct-12 links in FP32 where the gauge has them.  Otherwise (FP64,
// several rhs per thread): phase B's block size, as many blocks as are
// resident at once, complete links.  Its phase A forms the direction as q (no
// p and no phase C).  ls.pcus: the compute-unit limit of the first kind of
// launch (0 for the second).
void plan_persistent(LaunchSet &ls, Prob &pr, int64_t V, int nrhs, int inner, int max_cus) {
    const bool cus = max_cus > 0 || (inner != WD_F64 && ls.k[KB].nr == 1);
    ls.pcus = max_cus > 0 ? max_cus : cus ? (1 << 30) : 0;
    const int blk = cus ? 1024 : ls.k[KB].block;
    ls.qrec = 1;   // the persistent kernel's phase A carries the direction as q too
    ls.fused = 0;  // it finishes each iteration at its own grid barriers
    int nr = cus ? 1 : ls.k[KB].nr;
    if (inner == WD_F64 && nr > 2) nr = 2;
    const int kinds[2] = {KA, KB};
    for (int k : kinds) {
        KindShape &ks = ls.k[k];
        ks.block = blk;
        ks.nr = nr;
        ks.remap = 0;
        ks.ordered = 1;
        // z-marching: the order held the chunk count; no plane blocks
        ks.order = ks.xy == 2 ? 0 : ks.order & ~(1 << 17) & ~(7 << 18);
        ks.xy = 0;
        ks.planes = 1;
        ks.split = 0;
        ks.pair = 0;
        ks.lds = 0;
        ks.r12 = cus && inner == WD_F32 && pr.U12 != nullptr;
        ks.nt = 0;
        pr.sorder[k] = ks.order;
        pr.nsb[k] = (int)((V + blk - 1) / blk);
        pr.ng[k] = (nrhs + nr - 1) / nr;
        pr.nt[k] = pr.nsb[k] * pr.ng[k];
        ks.grid = pr.nt[k];
    }
}

// Fill the problem record of a solve whose workspace starts at ws.
void fill_prob(Prob &pr, const wd_gauge *g, double m0, int nrhs, const wd_cg_params &p,
               char *ws, const WsLayout &L) {
    pr.g = make_geom(g);
    pr.diag = 4.0 + m0;
    pr.eo = even_odd(p, g->dims);
    pr.vf = pr.eo ? (int)(g->V / 2) : (int)g->V;
    pr.eo_c = 0.25 / pr.diag;
    pr.tol2 = p.tol * p.tol;
    pr.nrhs = nrhs;
    pr.max_iter = p.max_iter;
    pr.ru_every = p.reliable_every;
    pr.method = p.method;
    pr.U_lo = g->U[p.inner];
    pr.U12 = p.inner == WD_F32 ? g->U12[WD_F32] : nullptr;
    pr.U64 = g->U[WD_F64];
    pr.x_lo = ws + L.xlo;
    pr.r = ws + L.r;
    pr.p = ws + L.p;
    pr.q = ws + L.q;
    pr.x64 = ws + L.x64;
    pr.eta64 = ws + L.eta64;
    pr.part = (double *)(ws + L.part);
    pr.psb = (int)((g->V + 63) / 64);   // the buffer's site blocks per column (ws_layout)
    pr.sc = (Scal *)(ws + L.scal);
    pr.sc2 = (Scal *)(ws + L.scal2);
    pr.v = ws + L.q;
    pr.rh = L.rh ? ws + L.rh : nullptr;
    pr.sv = L.sv ? ws + L.sv : nullptr;
    pr.tv = L.tv ? ws + L.tv : nullptr;
    pr.bs = L.bscal ? (BScal *)(ws + L.bscal) : nullptr;
    pr.part2 = L.bi_part2 ? (double *)(ws + L.bi_part2) : nullptr;
    pr.rec2 = L.bi_rec ? (BiRec *)(ws + L.bi_rec) : nullptr;
    pr.rec3 = pr.rec2 ? pr.rec2 + nrhs : nullptr;
    pr.recm = pr.rec2 ? pr.rec3 + nrhs : nullptr;
    pr.eta_o = L.eta_o ? ws + L.eta_o : nullptr;
    pr.tmp = L.tmp ? ws + L.tmp : nullptr;
    pr.w64 = L.w64 ? ws + L.w64 : nullptr;
}

void init_scalars(std::vector<Scal> &sc, int nrhs) {
    sc.assign(nrhs, Scal());
    for (auto &c : sc) {
        memset(&c, 0, sizeof(c));
        c.rho = 1.0;
        c.rho_old = 1.0;
        c.state = ST_FROZEN;   // the first reliable update computes r = eta - D x0
        c.restart = 1;
    }
}

// ------------------------------------------------------------ graph cache
// Every field of every kernel kind's launch shape is part of the key (the hop
// order, the LDS size, the link copy and the streaming hint select different
// kernels), so a changed shape never replays a graph of the old kernels.
struct GraphKey {
    const void *ws;
    int dims[4], nrhs, inner, K, persistent, method, max_cus;
    KindShape shp[NKIND];
    bool operator<(const GraphKey &o) const { return memcmp(this, &o, sizeof(*this)) < 0; }
};
static_assert(sizeof(KindShape) == 13 * sizeof(int), "KindShape must be plain ints (compared bytewise)");

struct GraphEntry {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    uint64_t last_use = 0;
};

static std::mutex g_graph_mu;
static std::map<GraphKey, GraphEntry> g_graphs;
static uint64_t g_graph_clock = 0;
static int64_t g_graphs_built = 0;   // chunk graphs captured since the library was loaded
static std::map<int, hipStream_t> g_capture_streams;

static hipStream_t capture_stream() {
    int dev = 0;
    (void)hipGetDevice(&dev);
    auto it = g_capture_streams.find(dev);
    if (it != g_capture_streams.end()) return it->second;
    hipStream_t s = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return nullptr;
    g_capture_streams[dev] = s;
    return s;
}

// Graph of one chunk: K iterations, then the reliable update and the summary.
// `record` enqueues the kernels of the chunk on the capture stream.
template <typename F>
static int get_graph(const GraphKey &key, F record, hipGraphExec_t *out) {
    std::lock_guard<std::mutex> lk(g_graph_mu);
    auto it = g_graphs.find(key);
    if (it != g_graphs.end()) {
        it->second.last_use = ++g_graph_clock;
        *out = it->second.exec;
        return WD_OK;
    }
    if (g_graphs.size() >= 32) {   // evict the least recently used
        auto victim = g_graphs.begin();
        for (auto j = g_graphs.begin(); j != g_graphs.end(); ++j)
            if (j->second.last_use < victim->second.last_use) victim = j;
        (void)hipGraphExecDestroy(victim->second.exec);
        (void)hipGraphDestroy(victim->second.graph);
        g_graphs.erase(victim);
    }
    hipStream_t cs = capture_stream();
    WD_CHECK(cs, WD_EHIP, "could not create the capture stream");
    WD_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    record(cs);
    GraphEntry e;
    hipError_t err = hipStreamEndCapture(cs, &e.graph);
    if (err != hipSuccess) return fail(WD_EHIP, "graph capture failed: %s", hipGetErrorString(err));
    err = hipGraphInstantiate(&e.exec, e.graph, nullptr, nullptr, 0);
    if (err != hipSuccess) {
        (void)hipGraphDestroy(e.graph);
        return fail(WD_EHIP, "graph instantiation failed: %s", hipGetErrorString(err));
    }
    e.last_use = ++g_graph_clock;
    g_graphs[key] = e;
    ++g_graphs_built;
    *out = e.exec;
    return WD_OK;
}

int cg_status_of(int st) {
    switch (st) {
    case ST_DONE: return WD_OK;
    case ST_BREAKDOWN: return WD_EBREAKDOWN;
    default: return WD_ENOTCONV;
    }
}

// ------------------------------------------------------------- profiling
static std::atomic<int> g_prof_on{0};
static std::mutex g_prof_mu;
struct ProfEntry {
    int64_t launches = 0;
    double ms = 0, bytes = 0;
};
static ProfEntry g_prof[3];   // phases A, B, C
static const char *g_prof_names[3] = {"cg_phaseA", "cg_phaseB", "cg_phaseC"};

// One chunk launched kernel by kernel, back to back, every phase-A/B/C tile
// kernel launched with start/stop events.  The number of fields that iterated in each
// launch is recovered after the chunk from the per-field iteration counters:
// an active field iterates without gaps from the start of the chunk until it
// freezes, so field i took part in iteration j of the chunk iff j < d_i, where
// d_i is its iteration count advance over the chunk (and skipped phase C of
// the iteration in which it froze).
static int profiled_chunk(int inner, const LaunchSet &ls, hipStream_t st, const Prob *dprob, int K,
                          int nrhs, int64_t V, void *dscal, bool r12) {
    std::vector<hipEvent_t> ev(6 * K);   // start and end of every A, B, C tile kernel
    for (auto &e : ev) WD_HIP(hipEventCreate(&e));
    std::vector<Scal> before(nrhs), after(nrhs);
    const double G = (double)link_bytes(inner, V, r12);
    const double S = (double)spinor_bytes(inner, V, 1);
    const double SX = (double)spinor_bytes(inner == WD_F16N ? WD_F32 : inner, V, 1);
    int rc = WD_OK;
    if (hipMemcpyAsync(before.data(), dscal, sizeof(Scal) * nrhs, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        rc = fail(WD_EHIP, "profiling copy failed");
    if (!rc) {
        for (int it = 0; it < K; ++it) {
            const int kinds[3] = {KA, KB, KC};
            for (int q = 0; q < (ls.qrec ? 2 : 3); ++q) {
                t_ev_start = ev[6 * it + 2 * q];
                t_ev_stop = ev[6 * it + 2 * q + 1];
                if (ls.fused)   // the sequence launch_iterations records
                    launch_kind_tiles(kinds[q], inner, ls.k[kinds[q]], st, dprob, 1, it & 1, it == (q == 0 ? 0 : K - 1));
                else launch_kind_tiles(kinds[q], inner, ls.k[kinds[q]], st, dprob, 1);
                t_ev_start = t_ev_stop = nullptr;
                if (kinds[q] != KC && !ls.fused) launch_finish_after(kinds[q], ls, st, dprob, 1);
            }
        }
        if (ls.fused)
            hipLaunchKernelGGL(k_finish, dim3(1), dim3(1024), 0, st, dprob, 1, KB | FIN_AB | FIN_TRAIL | ((K & 1) << 12));
        if (hipMemcpyAsync(after.data(), dscal, sizeof(Scal) * nrhs, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            rc = fail(WD_EHIP, "profiling copy failed");
    }
    if (!rc) {
        std::vector<int> d(nrhs), froze(nrhs);
        for (int i = 0; i < nrhs; ++i) {
            d[i] = after[i].iters - before[i].iters;
            froze[i] = (d[i] > 0 && after[i].state != ST_ACTIVE) ? 1 : 0;
        }
        std::lock_guard<std::mutex> lk(g_prof_mu);
        for (int it = 0; it < K; ++it) {
            int nact = 0, nc = 0, nq = 0;
            for (int i = 0; i < nrhs; ++i) {
                nact += it < d[i];
                nc += it < d[i] - froze[i];
                nq += it < d[i] && !(it == 0 && before[i].restart);   // phase A reads the old q
            }
            // phase B's x_lo: in every iteration, or paired (fused finish) two
            // iterations' updates in the launches of parity 1 (which read both q)
            const double bx = !ls.fused || !ls.k[KB].pair ? 2.0 * SX
                              : (it & 1) ? S + 2.0 * SX : it == K - 1 ? 2.0 * SX : 0.0;
            const double bytes[3] = {G + nact * 2.0 * S + (ls.qrec ? nq * S : 0.0), G + nact * (3.0 * S + bx),
                                     nc * 3.0 * S};
            const int cnt[3] = {nact, nact, ls.qrec ? 0 : nc};
            for (int k = 0; k < 3; ++k) {
                if (cnt[k] == 0) continue;
                float ms = 0;
                hipEventElapsedTime(&ms, ev[6 * it + 2 * k], ev[6 * it + 2 * k + 1]);
                g_prof[k].launches += 1;
                g_prof[k].ms += ms;
                g_prof[k].bytes += bytes[k];
            }
        }
    }
    for (auto &e : ev) (void)hipEventDestroy(e);
    return rc;
}

// Pinned host staging for the solve driver's small copies (problem record,
// scalar records, chunk summary), one buffer per host thread, kept for the
// life of the thread: copies from pageable memory go through the runtime's
// own staging and left the GPU idle for tens of microseconds each, and a
// pinned allocation per solve costs as much.  A solve reuses the buffer only
// after the previous solve on the thread has synchronised its stream (a solve
// that returned an error early may leave a copy in flight, which reads the
// buffer only for that failed solve).
static char *host_stage(size_t bytes) {
    thread_local char *buf = nullptr;
    thread_local size_t cap = 0;
    if (cap < bytes) {
        if (buf) (void)hipHostFree(buf);
        buf = nullptr;
        cap = 0;
        if (hipHostMalloc((void **)&buf, bytes, hipHostMallocDefault) != hipSuccess) return nullptr;
        cap = bytes;
    }
    return buf;
}

// The solve driver shared by wd_cg_solve and wd_cg_solve_batch.
int cg_run(const wd_gauge *g, double m0, const void *src, void *sol, int nrhs, const wd_cg_params &p,
           void *ws, size_t ws_bytes, wd_cg_report *reps, hipStream_t st) {
    const auto t_start = std::chrono::steady_clock::now();
    const int64_t V = g->V;
    const int eo = even_odd(p, g->dims);
    const WsLayout L = ws_layout(V, nrhs, p.inner, p.method, eo);
    WD_CHECK(ws_bytes >= L.least, WD_ENOMEM, "workspace of %zu bytes, %zu needed", ws_bytes, L.least);
    char *w = (char *)ws;
    Prob hp;
    memset(&hp, 0, sizeof(hp));
    fill_prob(hp, g, m0, nrhs, p, w, L);
    LaunchSet ls;
    plan_shapes(g, nrhs, p.inner, ls, hp);
    const Prob *dprob = (const Prob *)(w + L.prob);
    int *dsum = (int *)(w + L.summary);

    const int K = p.chunk > 0 ? p.chunk : (p.reliable_every > 0 ? p.reliable_every : 50);
    const bool bicg = p.method == METHOD_BICGSTAB;
    // the fused iteration needs the pieces after L.least
    ls.bi_fused = bicg && ws_bytes >= L.total && !unfused_requested();
    const int persistent = (p.persistent == 1 && !bicg) ? 1 : 0;
    if (persistent) plan_persistent(ls, hp, V, nrhs, p.inner, p.max_cus);
    for (int k = 0; k < NKIND; ++k)   // kernels launched one by one are compiled for <= 256 threads
                                      // (phases A and B: multi-plane <= 512, direction-split <= 1024)
        WD_CHECK(ls.k[k].block <= 256 || (persistent && (k == KA || k == KB)) ||
                     (ls.k[k].planes > 1 && ls.k[k].block <= 512 && (k == KA || k == KB)) ||
                     (ls.k[k].split && ls.k[k].block <= 1024 && (k == KA || k == KB)),
                 WD_EINVAL, "kernel kind %d planned with %d threads per block", k, ls.k[k].block);
    for (int k = 0; k < NKIND; ++k)   // every kind's partial sums fit the buffer
        WD_CHECK(hp.nsb[k] <= (V + 63) / 64, WD_EINVAL, "kernel kind %d has %d site blocks, the partial-sum "
                 "buffer holds %lld", k, hp.nsb[k], (long long)((V + 63) / 64));

    // upload the problem record and the initial scalars
    std::vector<Scal> sc;
    init_scalars(sc, nrhs);
    // staging: problem record, scalar records, summary (pinned, see host_stage)
    const size_t st_scal = (sizeof(Prob) + 255) & ~size_t(255), st_sum = st_scal + ((sizeof(Scal) * nrhs + 255) & ~size_t(255));
    char *stage = host_stage(st_sum + 256);
    WD_CHECK(stage, WD_ENOMEM, "pinned host staging of %zu bytes", st_sum + 256);
    memcpy(stage, &hp, sizeof(hp));
    memcpy(stage + st_scal, sc.data(), sizeof(Scal) * nrhs);
    WD_HIP(hipMemcpyAsync((void *)dprob, stage, sizeof(hp), hipMemcpyHostToDevice, st));
    WD_HIP(hipMemcpyAsync(w + L.scal, stage + st_scal, sizeof(Scal) * nrhs, hipMemcpyHostToDevice, st));
    WD_HIP(hipMemsetAsync(w + L.bar, 0, BAR_BYTES, st));
    // fields
    const int64_t Vf = hp.vf;
    int rc = WD_OK;
    if (eo) {   // even and odd halves of the source (and of x0: its odd half is not used)
        launch_eo_split(dprob, Vf, nrhs, src, w + L.eta64, w + L.eta_o, st);
        if (p.use_x0) launch_eo_split(dprob, Vf, nrhs, sol, w + L.x64, w + L.w64, st);
        else launch_zero(w + L.x64, spinor_bytes(WD_F64, Vf, nrhs), st);
    } else {
        rc = launch_pack_spinor(WD_F64, src, w + L.eta64, (int)V, nrhs, st);
        if (rc) return rc;
        if (p.use_x0) rc = launch_pack_spinor(WD_F64, sol, w + L.x64, (int)V, nrhs, st);
        else launch_zero(w + L.x64, spinor_bytes(WD_F64, V, nrhs), st);
        if (rc) return rc;
    }
    launch_zero(w + L.xlo, spinor_bytes(p.inner == WD_F16N ? WD_F32 : p.inner, Vf, nrhs), st);
    if (bicg) launch_zero(w + L.bscal, al256(sizeof(BScal) * nrhs), st);
    // |eta|, (even-odd: the Schur system's source), first true residual, p = r
    // (BiCGSTAB: its first stage S1 does that)
    launch_kind(KN, p.inner, ls, st, dprob, 1);
    if (eo) {
        launch_eo_source(dprob, Vf, nrhs, st);
    }
    launch_first_residual(p.inner, ls, st, dprob, 1, !p.use_x0);
    if (!bicg) launch_kind(KC, p.inner, ls, st, dprob, 1);
    const int *dabort = persistent ? (const int *)(w + L.bar + BAR_ABORT) : nullptr;
    launch_summary(st, dprob, 1, dsum, dabort);
    WD_HIP(hipGetLastError());

    GraphKey key;
    memset(&key, 0, sizeof(key));
    key.ws = ws;
    for (int d = 0; d < 4; ++d) key.dims[d] = g->dims[d];
    key.nrhs = nrhs;
    key.inner = p.inner;
    key.persistent = persistent;
    key.max_cus = p.max_cus;
    key.method = p.method | (eo << 4) | (ls.fused << 5) | (ls.bi_fused << 6);
    for (int k = 0; k < NKIND; ++k) key.shp[k] = ls.k[k];
    // the graph of a chunk of Kc iterations (cached per length)
    auto chunk_graph = [&](int Kc, hipGraphExec_t *exec) -> int {
        key.K = Kc;
        int rec_rc = WD_OK;
        const int r = get_graph(key, [&](hipStream_t cs) {
            if (bicg) {
                if (ls.bi_fused) {
                    launch_kind(KS1, p.inner, ls, cs, dprob, 1);   // fields that restart
                    for (int it = 0; it < Kc; ++it)
                        for (int k = KS2; k <= KS5; ++k) launch_kind(k, p.inner, ls, cs, dprob, 1, 0, it == 0);
                    launch_finish(KS5 | FIN_TRAIL_BI, cs, dprob, 1);
                } else {
                    for (int it = 0; it < Kc; ++it)
                        for (int k = KS1; k <= KS5; ++k) launch_kind(k, p.inner, ls, cs, dprob, 1);
                }
                launch_kind(KR1, p.inner, ls, cs, dprob, 1);
                launch_kind(KR2, p.inner, ls, cs, dprob, 1);
                launch_summary(cs, dprob, 1, dsum, dabort);
                return;
            }
            if (persistent) rec_rc = record_persistent_chunk(p.inner, ls, cs, dprob, 1, Kc, w + L.bar, ls.pcus);
            else launch_iterations(p.inner, ls, cs, dprob, 1, Kc);
            launch_kind(KR1, p.inner, ls, cs, dprob, 1);
            if (eo) launch_kind(KER2A, p.inner, ls, cs, dprob, 1);
            launch_kind(KR2, p.inner, ls, cs, dprob, 1);
            launch_kind(KC, p.inner, ls, cs, dprob, 1);
            launch_summary(cs, dprob, 1, dsum, dabort);
        }, exec);
        return r ? r : rec_rc;
    };

    int *hsum = (int *)(stage + st_sum);
    WD_HIP(hipMemcpyAsync(hsum, dsum, 3 * sizeof(int), hipMemcpyDeviceToHost, st));
    WD_HIP(hipStreamSynchronize(st));
    // Chunks of K iterations, except where the library picks the length
    // (p.chunk == 0): once the summary estimates that the active fields need
    // fewer, the chunk is cut to that many plus 3, rounded up to a multiple of
    // 8 (a few graph lengths), so a solve does not idle through most of a
    // chunk after its fields converge.  Chunk boundaries only decide when the
    // host looks: the results are bitwise the same for any lengths.
    const bool adaptive = p.chunk == 0;
    // every chunk of K either converges a field or spends K iterations of it (fused
    // BiCGSTAB: or restarts, at most one after each iteration)
    const int64_t budget = (int64_t)K * (p.max_iter / K + 2 * (p.max_iter / (K * 4) + 4)) * (ls.bi_fused ? 2 : 1);
    const bool prof = g_prof_on.load() != 0 && !persistent && !bicg && !eo;
    int Kc = K;
    for (int64_t run = 0; run < budget && hsum[0] > 0; run += Kc) {
        hipError_t e = hipSuccess;
        if (prof) {
            rc = profiled_chunk(p.inner, ls, st, dprob, Kc, nrhs, V, w + L.scal, ls.k[KB].r12 != 0);
            if (rc) return rc;
            launch_kind(KR1, p.inner, ls, st, dprob, 1);
            launch_kind(KR2, p.inner, ls, st, dprob, 1);
            launch_kind(KC, p.inner, ls, st, dprob, 1);
            launch_summary(st, dprob, 1, dsum, dabort);
        } else {
            hipGraphExec_t exec = nullptr;
            rc = chunk_graph(Kc, &exec);
            if (rc) return rc;
            e = hipGraphLaunch(exec, st);
        }
        if (e == hipSuccess) e = hipMemcpyAsync(hsum, dsum, 3 * sizeof(int), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return fail(WD_EHIP, "chunk replay failed: %s", hipGetErrorString(e));
        if (persistent && hsum[1] != 0) return fail(WD_EHIP, "persistent kernel grid barrier timed out");
        const int need = hsum[2];
        Kc = (adaptive && need >= 0 && need + 3 < K) ? std::min(K, std::max(8, (need + 3 + 7) / 8 * 8)) : K;
    }
    // solution out (even-odd: x_o from x_e), scalars back
    if (eo) {
        launch_eo_merge(dprob, Vf, nrhs, sol, st);
        WD_HIP(hipGetLastError());
    } else {
        rc = launch_unpack_spinor(WD_F64, w + L.x64, sol, (int)V, nrhs, st);
        if (rc) return rc;
    }
    WD_HIP(hipMemcpyAsync(stage + st_scal, w + L.scal, sizeof(Scal) * nrhs, hipMemcpyDeviceToHost, st));
    WD_HIP(hipStreamSynchronize(st));
    memcpy(sc.data(), stage + st_scal, sizeof(Scal) * nrhs);
    int first_bad = WD_OK;
    for (int i = 0; i < nrhs; ++i) {
        if (sc[i].zero_src) WD_HIP(hipMemsetAsync((char *)sol + (size_t)i * V * 192, 0, (size_t)V * 192, st));
    }
    WD_HIP(hipStreamSynchronize(st));
    const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
    for (int i = 0; i < nrhs; ++i) {
        const Scal &c = sc[i];
        wd_cg_report &r = reps[i];
        memset(&r, 0, sizeof(r));
        r.status = cg_status_of(c.state);
        r.iters = c.iters;
        r.reliable_updates = c.n_ru;
        r.true_rel_res = c.eta2 > 0 ? sqrt(c.true2 / c.eta2) : 0.0;
        r.iter_rel_res = c.eta2 > 0 ? sqrt(c.rho / c.eta2) : 0.0;
        r.seconds = secs;
        if (r.status != WD_OK && first_bad == WD_OK) first_bad = r.status;
    }
    if (first_bad != WD_OK)
        fail(first_bad, "%s", first_bad == WD_EBREAKDOWN ? "a field broke down" : "a field did not converge");
    return first_bad;
}

int check_params(const wd_cg_params *p) {
    WD_CHECK(p, WD_EINVAL, "null params");
    WD_CHECK(p->tol > 0 && p->tol < 1, WD_EINVAL, "tol %g out of (0, 1)", p->tol);
    WD_CHECK(p->max_iter >= 1, WD_EINVAL, "max_iter %d < 1", p->max_iter);
    WD_CHECK(p->reliable_every >= 0, WD_EINVAL, "reliable_every %d < 0", p->reliable_every);
    WD_CHECK(p->inner >= 0 && p->inner <= 2, WD_EINVAL, "unknown inner precision %d", p->inner);
    WD_CHECK(p->chunk >= 0 && p->chunk <= 1000, WD_EINVAL, "chunk %d out of range", p->chunk);
    WD_CHECK(p->persistent >= -1 && p->persistent <= 1, WD_EINVAL, "persistent %d", p->persistent);
    WD_CHECK(p->method == METHOD_CGNE || p->method == METHOD_BICGSTAB, WD_EINVAL, "unknown method %d", p->method);
    WD_CHECK(p->method == METHOD_CGNE || p->persistent != 1, WD_EINVAL,
             "the persistent kernel runs CG only");
    WD_CHECK(p->precondition == WD_PRECOND_NONE || p->precondition == WD_PRECOND_EO, WD_EINVAL,
             "unknown preconditioning %d", p->precondition);
    WD_CHECK(p->precondition == WD_PRECOND_NONE || (p->method == METHOD_CGNE && p->persistent != 1), WD_EINVAL,
             "even-odd preconditioning runs CG without the persistent kernel");
    WD_CHECK(p->max_cus >= 0, WD_EINVAL, "max_cus %d < 0", p->max_cus);
    WD_CHECK(p->max_cus == 0 || (p->persistent == 1 && p->method == METHOD_CGNE), WD_EINVAL,
             "max_cus needs the persistent CG kernel (persistent = 1)");
    WD_CHECK(p->max_cus == 0 || p->inner != WD_F64, WD_EINVAL, "max_cus needs an FP32 or FP16N inner iteration");
    return WD_OK;
}

}  // namespace wd

using namespace wd;

extern "C" {

void wd_cg_default_params(wd_cg_params *p) {
    if (!p) return;
    memset(p, 0, sizeof(*p));
    p->tol = 1e-10;
    p->max_iter = 20000;
    p->reliable_every = 50;
    p->inner = WD_F32;
    p->use_x0 = 0;
    p->persistent = -1;
    p->chunk = 0;
    p->method = METHOD_CGNE;
}

size_t wd_cg_workspace_bytes(const wd_gauge *g, int32_t nrhs, const wd_cg_params *p) {
    if (!g || !p || nrhs < 1 || nrhs > MAX_RHS || p->inner < 0 || p->inner > 2) return 0;
    if (p->method != METHOD_CGNE && p->method != METHOD_BICGSTAB) return 0;
    if (p->precondition != WD_PRECOND_NONE && p->precondition != WD_PRECOND_EO) return 0;
    return ws_layout(g->V, nrhs, p->inner, p->method, even_odd(*p, g->dims)).total;
}

int wd_cg_solve_batch(const wd_gauge *g, double m0, const void *src, void *sol, int32_t nrhs,
                      const wd_cg_params *p, void *ws, size_t ws_bytes, wd_cg_report *reps, void *stream) {
    clear_error();
    WD_CHECK(g && src && sol && ws && reps, WD_EINVAL, "null argument");
    WD_CHECK(nrhs >= 1 && nrhs <= MAX_RHS, WD_EINVAL, "nrhs %d out of range 1..%d", nrhs, MAX_RHS);
    WD_CHECK(m0 > -4.0 && m0 < 1e6, WD_EINVAL, "m0 %g out of range", m0);
    int rc = check_params(p);
    if (rc) return rc;
    WD_CHECK(g->U[p->inner], WD_EINVAL, "gauge handle holds no links in precision %d", p->inner);
    WD_CHECK(src != sol, WD_EINVAL, "src and sol must not overlap");
    WD_CHECK(p->precondition != WD_PRECOND_EO || g->dims[0] % 2 == 0, WD_EINVAL,
             "even-odd preconditioning needs an even Lx (got %d)", g->dims[0]);
    rc = require_gfx950();
    if (rc) return rc;
    return cg_run(g, m0, src, sol, nrhs, *p, ws, ws_bytes, reps, (hipStream_t)stream);
}

int wd_cg_solve(const wd_gauge *g, double m0, const void *src, void *sol, const wd_cg_params *p,
                void *ws, size_t ws_bytes, wd_cg_report *rep, void *stream) {
    return wd_cg_solve_batch(g, m0, src, sol, 1, p, ws, ws_bytes, rep, stream);
}

int wd_tune_cg(const wd_gauge *g, double m0, int32_t inner, const void *src, int32_t nrhs, int32_t iters,
               wd_tune_result *best, void *stream) {
    clear_error();
    WD_CHECK(g && src && best, WD_EINVAL, "null argument");
    WD_CHECK(inner >= 0 && inner <= 2 && g->U[inner], WD_EINVAL, "no links in precision %d", inner);
    WD_CHECK(nrhs >= 1 && nrhs <= MAX_RHS, WD_EINVAL, "nrhs %d out of range 1..%d", nrhs, MAX_RHS);
    WD_CHECK(iters >= 1 && iters <= 1000, WD_EINVAL, "iters %d out of range 1..1000", iters);
    WD_CHECK(m0 > -4.0 && m0 < 1e6, WD_EINVAL, "m0 %g out of range", m0);
    int rc = require_gfx950();
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    wd_cg_params p;
    wd_cg_default_params(&p);
    p.inner = inner;
    p.max_iter = iters;        // every field runs exactly `iters` iterations (tol is out of reach)
    p.tol = 1e-15;
    p.reliable_every = 0;
    p.chunk = iters;
    p.persistent = 0;
    const size_t wsb = wd_cg_workspace_bytes(g, nrhs, &p);
    const size_t fb = (size_t)g->V * 192 * nrhs;
    void *ws = nullptr, *x = nullptr;
    WD_HIP(hipMalloc(&ws, wsb));
    if (hipMalloc(&x, fb) != hipSuccess) {
        (void)hipFree(ws);
        return fail(WD_ENOMEM, "tuner scratch of %zu bytes", fb);
    }
    std::vector<double> ref(fb / 8), got(fb / 8);
    std::vector<wd_cg_report> reps(nrhs);
    const int Lz = g->dims[2], np = g->dims[0] * g->dims[1];
    const Geom geo = make_geom(g);
    const ShapeKey ka{{g->dims[0], g->dims[1], g->dims[2], g->dims[3]}, inner, nrhs, 1, FAM_CG_A};
    ShapeKey kb = ka;
    kb.dag = 0;
    kb.fam = FAM_CG_B;
    const Shape keep_a = shape_lookup(ka), keep_b = shape_lookup(kb);
    // candidates: plane or site blocks, rhs per thread, hop order, z-strip width
    std::vector<Shape> cand;
    for (int xy = 1; xy >= 0; --xy) {
        if (xy && (np < 64 || np > 256)) continue;
        for (int nr = 1; nr <= 2; ++nr) {
            if (xy && nr == 2 && inner == WD_F64) continue;
            for (int ord : {5, 3, 1})
                for (int strip : {4, 0, 2, 7}) {
                    if (strip >= Lz) continue;
                    if (ord == 5 && !(xy && nr == 1)) continue;   // memory hops first: plane blocks
                    Shape s = default_shape(kb);
                    s.block = 256;
                    s.nr = nr;
                    s.ordered = ord;
                    s.strip = strip;
                    s.xylds = xy;
                    s.gmajor = 0;
                    s.occ = 0;
                    s.planes = 1;
                    cand.push_back(s);
                    s.planes = 2;   // two z-adjacent planes per block, where they fit
                    if (ord == 5 && xy_planes(s, geo, inner, 1) == 2) cand.push_back(s);
                }
        }
    }
    double best_ms = 1e30;
    Shape bests = keep_b;
    int nref = 0;
    for (size_t c = 0; c < cand.size() && rc == WD_OK; ++c) {
        shape_store(ka, cand[c]);
        shape_store(kb, cand[c]);
        int r = cg_run(g, m0, src, x, nrhs, p, ws, wsb, reps.data(), st);   // warm-up: graph capture
        if (r != WD_OK && r != WD_ENOTCONV) { rc = r; break; }
        float t[3];
        for (int k = 0; k < 3 && rc == WD_OK; ++k) {
            hipEvent_t e0, e1;
            WD_HIP(hipEventCreate(&e0));
            WD_HIP(hipEventCreate(&e1));
            (void)hipEventRecord(e0, st);
            r = cg_run(g, m0, src, x, nrhs, p, ws, wsb, reps.data(), st);
            (void)hipEventRecord(e1, st);
            (void)hipEventSynchronize(e1);
            (void)hipEventElapsedTime(&t[k], e0, e1);
            (void)hipEventDestroy(e0);
            (void)hipEventDestroy(e1);
            if (r != WD_OK && r != WD_ENOTCONV) rc = r;
        }
        if (rc) break;
        std::sort(t, t + 3);
        // the iterate must agree with the first candidate's (rounding order differs)
        WD_HIP(hipMemcpy(c == 0 ? ref.data() : got.data(), x, fb, hipMemcpyDeviceToHost));
        bool ok = true;
        if (c == 0) {
            nref = 1;
        } else {
            double d2 = 0, r2 = 0;
            for (size_t k = 0; k < ref.size(); ++k) {
                const double d = got[k] - ref[k];
                d2 += d * d;
                r2 += ref[k] * ref[k];
            }
            ok = d2 <= 1e-6 * r2;   // relative difference <= 1e-3
        }
        if (ok && t[1] < best_ms) {
            best_ms = t[1];
            bests = cand[c];
        }
    }
    (void)hipFree(ws);
    (void)hipFree(x);
    if (rc != WD_OK || !nref) {
        shape_store(ka, keep_a);
        shape_store(kb, keep_b);
        return rc ? rc : fail(WD_EHIP, "no CG launch shape could be timed");
    }
    shape_store_persist(ka, bests, best_ms * 1e3);
    shape_store_persist(kb, bests, best_ms * 1e3);
    memset(best, 0, sizeof(*best));
    best->block = bests.block;
    best->rhs_per_thread = bests.nr;
    best->xcd_remap = bests.remap;
    best->hop_order = bests.ordered;
    best->rhs_loop = bests.rloop;
    best->site_order = encode_order(bests);
    best->us = best_ms * 1e3;
    return WD_OK;
}

int wd_cg_graph_stats(int64_t *built, int32_t *cached) {
    clear_error();
    WD_CHECK(built && cached, WD_EINVAL, "null argument");
    std::lock_guard<std::mutex> lk(g_graph_mu);
    *built = g_graphs_built;
    *cached = (int32_t)g_graphs.size();
    return WD_OK;
}

int wd_profile_enable(int32_t on) {
    clear_error();
    g_prof_on.store(on ? 1 : 0);
    return WD_OK;
}

int wd_profile_reset(void) {
    clear_error();
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (auto &e : g_prof) e = ProfEntry();
    return WD_OK;
}

int wd_profile_read(wd_kernel_stat *out, int32_t max_n, int32_t *n) {
    clear_error();
    WD_CHECK(n && (out || max_n == 0), WD_EINVAL, "null argument");
    std::lock_guard<std::mutex> lk(g_prof_mu);
    *n = 3;
    for (int k = 0; k < 3 && k < max_n; ++k) {
        memset(&out[k], 0, sizeof(out[k]));
        strncpy(out[k].name, g_prof_names[k], sizeof(out[k].name) - 1);
        out[k].launches = g_prof[k].launches;
        out[k].total_ms = g_prof[k].ms;
        out[k].bytes_total = g_prof[k].bytes;
    }
    return WD_OK;
}

}  // extern "C"
