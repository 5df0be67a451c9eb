// Device side of BiCGSTAB on D itself -- one of the other Krylov methods the
// paper lists for the Dirac equation (arXiv 2111.14958, Sec. 1) -- on the same
// machinery as the CG: per-field scalars in device memory, fixed-order
// last-block reductions, the FP64 reliable update R1/R2 of cg_core.h.
//
// One iteration (van der Vorst's BiCGSTAB, shadow residual r_hat):
//   S1  p = r + beta (p - omega v)        (p = r, r_hat = r after a restart)
//   S2  v = D p,        <r_hat, v>  -> alpha = rho / <r_hat, v>
//   S3  s = r - alpha v
//   S4  t = D s,        <t, s>, <t, t>  -> omega = <t, s> / <t, t>
//   S5  x += alpha p + omega s, r = s - omega t,
//       <r_hat, r>, |r|^2  -> rho, beta = (rho / rho_old)(alpha / omega), tests
// <a, b> = sum conj(a) b.  A reliable update restarts with r_hat = r = eta - D x;
// a (near) breakdown |<r_hat, r>| <= 1e-6 |r_hat| |r| restarts with r_hat = r.
//
// Fused iteration (BiRec records; the default): four launches, every
// reduction completed by the launch that needs it, instead of five stages and
// three one-block finishes:
//   F2  completes |r|^2: counters, state, tests;  v = D p,  <r_hat, v>
//   S3  alpha;  s = r - alpha v
//   F4  t = D s,  <t, s>, <t, t>, <r_hat, s>, <r_hat, t>
//   F5  omega, rho = <r_hat, s> - omega <r_hat, t>, beta;  x += alpha p + omega s,
//       r = s - omega t,  p = r + beta (p - omega v),  |r|^2
// rho of the new residual is known before it is formed, so S5 and the next S1
// are one pass (8 spinor streams instead of 11).  The test for a near breakdown
// needs |r|^2, which F2 completes when p is formed already, so a field that
// restarts sits out the rest of that round of launches and S3 sets p = r_hat = r
// (F5's p cannot stay: p - r = rho / (omega <r_hat, v>) (p_old - omega v), and
// <r_hat, v> is small where the rho before was).  At a chunk's end a trailing
// finish closes the last iteration into the final records, and the next chunk's
// S1 sets p = r_hat = r, as it does after a reliable update: the iterates are the
// same wherever chunks end.
// (rho does not see the rounding of the stored r.  Against <r_hat, r> over 1056
// fields of 4^4 to 12^4 stopped at 1e-10, mean change in FP32 and FP16N: iterations
// 0.03 +- 0.04 and -0.02 +- 0.06, error against an FP64 solution at 1e-14 -4.5 +-
// 2.0 % and -0.7 +- 1.4 %; in FP64 neither changed on 180 fields.)
// The five-stage iteration remains for workspaces without the fused one's
// records.  12^4 x 4 FP32, where launches and latency bound: a solve 4.36 -> 3.61
// ms, 3.33 ms with the last chunk cut to the estimated need.
#pragma once

#include "cg_core.h"

namespace wd {

struct dc { double re, im; };
__device__ __forceinline__ dc dmul(dc a, dc b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ dc ddiv(dc a, dc b) {
    const double d = b.re * b.re + b.im * b.im;
    return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}
__device__ __forceinline__ bool dfinite(dc a) { return a.re == a.re && a.im == a.im && fabs(a.re) < 1e300 && fabs(a.im) < 1e300; }
__device__ __forceinline__ dc ld(const double v[2]) { return {v[0], v[1]}; }
__device__ __forceinline__ void st(double v[2], dc a) { v[0] = a.re; v[1] = a.im; }

// Records of the fused iteration: each launch reads one array and writes
// another (a launch's blocks all read what its site block 0 replaces).
// What a chunk does not change stays in the final records (Scal, BScal).
struct alignas(16) BiRec {
    double rr, ri;   // rho
    double ar, ai;   // alpha
    double wr, wi;   // omega
    double br, bi;   // beta
    double rh2, r2;  // |r_hat|^2, |r|^2
    int state, iters, since_ru;   // state: ST_*, or BI_RESTART in the round of launches that restarts the field
};
constexpr int BI_RESTART = 5;
// columns of the fused iteration's partials: pr.part slots 0, 1 <r_hat, v>, 2
// |r|^2; pr.part2 <t, s>, <t, t>, <r_hat, s>, <r_hat, t>
constexpr int BI_R2 = 2, BI_NP2 = 7;
__device__ __forceinline__ double *part2_col(const Prob &pr, int i, int k) {
    return pr.part2 + ((size_t)k * pr.nrhs + i) * pr.psb;
}
// sum of a column of nsb partials by one wavefront, in sum_all's order
__device__ __forceinline__ double wave_col_sum(const double *col, int nsb) {
    const int lane = threadIdx.x & 63;
    double a[4], x = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = lane + 64 * k < nsb ? col[lane + 64 * k] : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) x += a[k];
    for (int b = lane + 256; b < nsb; b += 64) x += col[b];
    return wave_sum(x);
}

// The end of an iteration of an active field (c: F5's record, read field by
// field), with |r|^2 = r2 of the residual F5 stored
__device__ __forceinline__ void bi_end(const Prob &pr, const BiRec &c, double stop2, double r2, BiRec &o) {
    o.ar = c.ar, o.ai = c.ai, o.wr = c.wr, o.wi = c.wi, o.br = c.br, o.bi = c.bi;
    o.rr = c.rr, o.ri = c.ri, o.rh2 = c.rh2, o.r2 = c.r2;
    o.state = c.state == BI_RESTART ? ST_ACTIVE : c.state;   // a restart is no iteration
    o.iters = c.iters, o.since_ru = c.since_ru;
    if (c.state != ST_ACTIVE) return;
    o.r2 = r2;
    o.iters += 1;
    o.since_ru += 1;
    if (!(r2 < 1e300) || !dfinite(dc{o.rr, o.ri})) o.state = ST_BREAKDOWN;
    else if (r2 <= stop2 || o.iters >= pr.max_iter || (pr.ru_every > 0 && o.since_ru >= pr.ru_every))
        o.state = ST_FROZEN;
    else if (o.rr * o.rr + o.ri * o.ri <= 1e-12 * o.rh2 * r2) {   // see bi5_finish
        o.state = BI_RESTART;
        o.rr = r2;
        o.ri = 0.0;
        o.rh2 = r2;
    }
}

// The finish of the previous iteration inside F2's blocks: begin issues the
// loads (before the plane staging, whose latency covers them), reduce (before
// its barrier) sums |r|^2, decide gives the fields that iterate (not those that
// restart).  first: the records are final.
template <int NR> struct BiBegin {
    const Prob &pr;
    const int rhs0, first;
    unsigned act0;   // fields that iterated before this launch's finish, or restarted
    double a[NR][4];
    __device__ __forceinline__ BiBegin(const Prob &p, int r0, int fi) : pr(p), rhs0(r0), first(fi) {
        act0 = 0;
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (rhs0 + j < pr.nrhs) {
                const int st = first ? pr.sc[rhs0 + j].state : pr.recm[rhs0 + j].state;
                if (st == ST_ACTIVE || st == BI_RESTART) act0 |= 1u << j;
            }
    }
    __device__ __forceinline__ void begin() {
        if (!first && act0) col_issue<NR>(pr, rhs0, act0, a, BI_R2, pr.nsb[KS5]);
    }
    __device__ __forceinline__ void reduce(double *r2) {
        if (!first && act0) col_reduce<NR>(pr, rhs0, act0, a, r2, BI_R2, pr.nsb[KS5]);
    }
    __device__ __forceinline__ unsigned decide(int sb, const double *r2, int *go) {
        if (threadIdx.x < NR) {
            const int j = threadIdx.x, i = rhs0 + j;
            go[j] = 0;
            if (i < pr.nrhs) {
                BiRec o;
                if (first) {   // S1 has formed p and r_hat of a field that restarts
                    const Scal &c = pr.sc[i];
                    const BScal &b = pr.bs[i];
                    o.rr = b.rho[0], o.ri = b.rho[1], o.ar = b.alpha[0], o.ai = b.alpha[1];
                    o.wr = b.omega[0], o.wi = b.omega[1], o.br = b.beta[0], o.bi = b.beta[1];
                    o.rh2 = b.rh2, o.r2 = c.rho;
                    o.state = c.state, o.iters = c.iters, o.since_ru = c.since_ru;
                } else {
                    bi_end(pr, pr.recm[i], pr.sc[i].stop2, act0 >> j & 1 ? r2[j] : 0.0, o);
                }
                go[j] = o.state == ST_ACTIVE;
                if (sb == 0) pr.rec2[i] = o;
            }
        }
        __syncthreads();
        unsigned act = 0;
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (go[j]) act |= 1u << j;
        return act;
    }
};

// p = r_hat = r at site s of field i
template <int P>
__device__ __forceinline__ void bi_restart(const Prob &pr, int i, int s) {
    typedef typename real_of<P>::type R;
    FieldPtr fr{pr.r, pr.g.V, pr.nrhs}, fp{pr.p, pr.g.V, pr.nrhs}, fh{pr.rh, pr.g.V, pr.nrhs};
    cx<R> r[12];
    Spinor<P>::load(fr, i, s, r);
    Spinor<P>::store(fh, i, s, r);
    Spinor<P>::store(fp, i, s, r);
}

// ------------------------------------------------------------- S1, streaming
template <int P>
__device__ __forceinline__ void bi1_tile(const Prob &pr, int t) {
    typedef typename real_of<P>::type R;
    const int sb = t / pr.nrhs, i = t - sb * pr.nrhs;
    const int s = sb * blockDim.x + threadIdx.x;
    const Scal &c = pr.sc[i];
    if (c.state != ST_ACTIVE || !c.pending_p || s >= pr.g.V) return;
    if (c.restart) {
        bi_restart<P>(pr, i, s);
        return;
    }
    FieldPtr fr{pr.r, pr.g.V, pr.nrhs}, fp{pr.p, pr.g.V, pr.nrhs};
    cx<R> r[12];
    Spinor<P>::load(fr, i, s, r);
    FieldPtr fv{pr.v, pr.g.V, pr.nrhs};
    const dc b = ld(pr.bs[i].beta), w = ld(pr.bs[i].omega);
    const R br = (R)b.re, bi = (R)b.im, wr = (R)w.re, wi = (R)w.im;
    cx<R> p[12], v[12];
    Spinor<P>::load(fp, i, s, p);
    Spinor<P>::load(fv, i, s, v);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        // d = p - omega v ; p = r + beta d
        const cx<R> d = {p[k].re - (wr * v[k].re - wi * v[k].im), p[k].im - (wr * v[k].im + wi * v[k].re)};
        p[k] = {r[k].re + (br * d.re - bi * d.im), r[k].im + (br * d.im + bi * d.re)};
    }
    Spinor<P>::store(fp, i, s, p);
}

// ------------------------------------------- S2 / S4, stencil plus reductions
// S2: out = v = D p, partials <r_hat, v> (2 numbers).
// S4: out = t = D s, partials <t, s> (2) and <t, t> (1).
// XY: one xy-plane per block, its input spinors staged in LDS (the x and y
// hops and the site's own spinor read them there); ORD: hop order as in the
// CG phases (5 = the memory hops z and t first); R12: links from the
// reconstruct-12 copy.
// F: the fused iteration's F2 (first: a chunk's first iteration) and F4.
template <int P, int NR, bool S4, int ORD = 1, bool XY = false, bool R12 = false, bool F = false>
__device__ __forceinline__ void bi_stencil_tile(const Prob &pr, int t, int first = 0) {
    typedef typename real_of<P>::type R;
    typedef typename LdsSpinor<P>::word W;
    __shared__ W xy[XY ? NR * LdsWords<P>::value * 256 : 1];
    const int K = S4 ? KS4 : KS2;
    int sb, grp, s;
    stencil_tile<XY>(pr, K, t, sb, grp, s);
    const int rhs0 = grp * NR;
    unsigned act = 0;
    BiBegin<NR> bb(pr, rhs0, F && !S4 ? first : 1);   // used by F2 alone (first: no fused records to read)
    __shared__ double r2[NR];
    __shared__ int go[NR];
    if constexpr (F && S4) {
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (rhs0 + j < pr.nrhs && pr.rec3[rhs0 + j].state == ST_ACTIVE) act |= 1u << j;
    } else if constexpr (F) {
        act = bb.act0;
        bb.begin();
    }
    else act = rhs_mask<NR>(pr, rhs0, ST_ACTIVE);
    constexpr int NP = F && S4 ? BI_NP2 : 3;   // numbers per field
    double part[NP * NR];
#pragma unroll
    for (int j = 0; j < NP * NR; ++j) part[j] = 0.0;
    const Geom g = pr.g;
    const int np = g.S[2];   // sites of a plane
    FieldPtr fin{S4 ? pr.sv : pr.p, g.V, pr.nrhs}, fout{S4 ? pr.tv : pr.v, g.V, pr.nrhs};
    if constexpr (F && !S4) {
        if (XY && act) stage_plane<P, NR>(fin, rhs0, act, s, g.V, xy, np, [&]() { bb.reduce(r2); });
        else if (act) {
            bb.reduce(r2);
            __syncthreads();
        }
        act = bb.decide(sb, r2, go);
    } else if (XY && act) stage_plane<P, NR>(fin, rhs0, act, s, g.V, xy, np);   // act is uniform over the block
    if (act && s < g.V) {
        FieldPtr fh{pr.rh, g.V, pr.nrhs};
        const void *U = R12 ? pr.U12 : pr.U_lo;
        cx<R> acc[NR][12];
        hopping<P, false, NR, ORD, XY, false, false, R12>(g, s, U, fin, rhs0, act, acc, nullptr, xy,
                                                          s - (int)threadIdx.x, np);
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            if (act >> j & 1) {
                cx<R> self[12], o[12], a[12];
                if constexpr (XY) LdsSpinor<P>::get(xy, np, j, threadIdx.x, self);
                else Spinor<P>::load(fin, rhs0 + j, s, self);
                wilson_finish<R>((R)pr.diag, self, acc[j], o);
                Spinor<P>::store(fout, rhs0 + j, s, o);
                if (S4) {
#pragma unroll
                    for (int k = 0; k < 12; ++k) a[k] = self[k];   // s
                } else {
                    Spinor<P>::load(fh, rhs0 + j, s, a);            // r_hat
                }
                if constexpr (F && S4) {   // all seven sums component by component
                    cx<R> h[12];
                    Spinor<P>::load(fh, rhs0 + j, s, h);
                    double u[BI_NP2] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int k = 0; k < 12; ++k) {
                        const dc t = {(double)o[k].re, (double)o[k].im}, v = {(double)a[k].re, (double)a[k].im},
                                 w = {(double)h[k].re, (double)h[k].im};
                        u[0] += t.re * v.re + t.im * v.im;   // <t, s> = sum conj(t) s
                        u[1] += t.re * v.im - t.im * v.re;
                        u[2] += (double)norm2(o[k]);
                        u[3] += w.re * v.re + w.im * v.im;   // <r_hat, s>
                        u[4] += w.re * v.im - w.im * v.re;
                        u[5] += w.re * t.re + w.im * t.im;   // <r_hat, t>
                        u[6] += w.re * t.im - w.im * t.re;
                        // the next component's conversions wait for these sums
                        if (k < 11) asm volatile("" : "+v"(o[k + 1].re), "+v"(a[k + 1].re), "+v"(h[k + 1].re) : "v"(u[0]), "v"(u[3]), "v"(u[6]));
                    }
#pragma unroll
                    for (int k = 0; k < BI_NP2; ++k) part[NP * j + k] = u[k];
                } else {
                    double re = 0, im = 0, nn = 0;
#pragma unroll
                    for (int k = 0; k < 12; ++k) {
                        if (S4) {   // <t, s> = sum conj(t) s
                            re += (double)o[k].re * a[k].re + (double)o[k].im * a[k].im;
                            im += (double)o[k].re * a[k].im - (double)o[k].im * a[k].re;
                            nn += (double)norm2(o[k]);
                        } else {    // <r_hat, v> = sum conj(r_hat) v
                            re += (double)a[k].re * o[k].re + (double)a[k].im * o[k].im;
                            im += (double)a[k].re * o[k].im - (double)a[k].im * o[k].re;
                        }
                    }
                    part[NP * j] = re;
                    part[NP * j + 1] = im;
                    part[NP * j + 2] = nn;
                }
            }
        }
    }
    if (act) {
        block_sum<NP * NR>(part);
        if (threadIdx.x == 0)
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (act >> j & 1) {
                    if constexpr (F && S4) {
                        for (int k = 0; k < NP; ++k) part2_col(pr, rhs0 + j, k)[sb] = part[NP * j + k];
                    } else {   // the fused iteration's slot 2 holds |r|^2
                        for (int k = 0; k < (F ? 2 : 3); ++k) part_at(pr, sb, rhs0 + j, k) = part[NP * j + k];
                    }
                }
    }
}

__device__ __forceinline__ void bi2_finish(const Prob &pr) {
    __shared__ double sums[MAX_SUMS];
    sum_all(pr, pr.nsb[KS2], 2, sums);
    for (int i = threadIdx.x; i < pr.nrhs; i += blockDim.x) {
        Scal &c = pr.sc[i];
        if (c.state == ST_ACTIVE) {
            const dc rv = {sums[2 * i], sums[2 * i + 1]};
            if (!dfinite(rv) || (rv.re == 0.0 && rv.im == 0.0)) c.state = ST_BREAKDOWN;
            else st(pr.bs[i].alpha, ddiv(ld(pr.bs[i].rho), rv));
        }
        c.pending_p = 0;
        c.restart = 0;
    }
}

__device__ __forceinline__ void bi4_finish(const Prob &pr) {
    __shared__ double sums[MAX_SUMS];
    sum_all(pr, pr.nsb[KS4], 3, sums);
    for (int i = threadIdx.x; i < pr.nrhs; i += blockDim.x) {
        Scal &c = pr.sc[i];
        if (c.state != ST_ACTIVE) continue;
        const double re = sums[3 * i], im = sums[3 * i + 1], tt = sums[3 * i + 2];
        {
            const dc w = {re / tt, im / tt};
            if (!finite_pos(tt) || !dfinite(w) || (w.re == 0.0 && w.im == 0.0)) c.state = ST_BREAKDOWN;
            else st(pr.bs[i].omega, w);
        }
    }
}

// ------------------------------------------------------------- S3, streaming
// F (the fused iteration): alpha formed here from F2's sums; a field that restarts
// gets p = r_hat = r instead
template <int P, bool F = false>
__device__ __forceinline__ void bi3_tile(const Prob &pr, int t) {
    typedef typename real_of<P>::type R;
    const int sb = t / pr.nrhs, i = t - sb * pr.nrhs;
    const int s = sb * blockDim.x + threadIdx.x;
    dc a;
    if constexpr (F) {
        __shared__ double sum[2], al[2];
        __shared__ int go;
        const BiRec &c = pr.rec2[i];
        const bool live = c.state == ST_ACTIVE;   // uniform over the block
        const int w = threadIdx.x >> 6;
        if (live && w < 2) {
            const double x = wave_col_sum(part_col(pr, i, w), pr.nsb[KS2]);
            if ((threadIdx.x & 63) == 0) sum[w] = x;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int state = c.state;
            dc na = {c.ar, c.ai};
            if (live) {
                const dc rv = {sum[0], sum[1]};
                if (!dfinite(rv) || (rv.re == 0.0 && rv.im == 0.0)) state = ST_BREAKDOWN;
                else na = ddiv(dc{c.rr, c.ri}, rv);
            }
            go = state;
            al[0] = na.re;
            al[1] = na.im;
            if (sb == 0) {
                BiRec &o = pr.rec3[i];
                o.rr = c.rr, o.ri = c.ri, o.ar = na.re, o.ai = na.im, o.wr = c.wr, o.wi = c.wi;
                o.br = c.br, o.bi = c.bi, o.rh2 = c.rh2, o.r2 = c.r2;
                o.state = state, o.iters = c.iters, o.since_ru = c.since_ru;
            }
        }
        __syncthreads();
        if (s >= pr.g.V) return;
        if (go == BI_RESTART) bi_restart<P>(pr, i, s);
        if (go != ST_ACTIVE) return;
        a = dc{al[0], al[1]};
    } else {
        if (pr.sc[i].state != ST_ACTIVE || s >= pr.g.V) return;
        a = ld(pr.bs[i].alpha);
    }
    FieldPtr fr{pr.r, pr.g.V, pr.nrhs}, fv{pr.v, pr.g.V, pr.nrhs}, fs{pr.sv, pr.g.V, pr.nrhs};
    const R ar = (R)a.re, ai = (R)a.im;
    cx<R> r[12], v[12];
    Spinor<P>::load(fr, i, s, r);
    Spinor<P>::load(fv, i, s, v);
#pragma unroll
    for (int k = 0; k < 12; ++k)
        r[k] = {r[k].re - (ar * v[k].re - ai * v[k].im), r[k].im - (ar * v[k].im + ai * v[k].re)};
    Spinor<P>::store(fs, i, s, r);
}

// ------------------------------------------------- S5, streaming + reductions
// x_lo += alpha p + omega s ; r = s - omega t ; partials <r_hat, r>, |r|^2
template <int P>
__device__ __forceinline__ void bi5_tile(const Prob &pr, int t) {
    typedef typename real_of<P>::type R;
    constexpr int XP = XPrec<P>::value;
    typedef typename real_of<XP>::type RX;
    const int sb = t / pr.nrhs, i = t - sb * pr.nrhs;
    const int s = sb * blockDim.x + threadIdx.x;
    if (pr.sc[i].state != ST_ACTIVE) return;   // uniform over the block
    double part[3] = {0.0, 0.0, 0.0};
    if (s < pr.g.V) {
        FieldPtr fp{pr.p, pr.g.V, pr.nrhs}, fs{pr.sv, pr.g.V, pr.nrhs}, ft{pr.tv, pr.g.V, pr.nrhs};
        FieldPtr fr{pr.r, pr.g.V, pr.nrhs}, fh{pr.rh, pr.g.V, pr.nrhs}, fx{pr.x_lo, pr.g.V, pr.nrhs};
        const dc a = ld(pr.bs[i].alpha), w = ld(pr.bs[i].omega);
        cx<R> p[12], sv[12], tv[12], h[12];
        cx<RX> x[12];
        Spinor<P>::load(fp, i, s, p);
        Spinor<P>::load(fs, i, s, sv);
        Spinor<P>::load(ft, i, s, tv);
        Spinor<XP>::load(fx, i, s, x);
        const RX axr = (RX)a.re, axi = (RX)a.im, wxr = (RX)w.re, wxi = (RX)w.im;
        const R wr = (R)w.re, wi = (R)w.im;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const RX pr_ = (RX)p[k].re, pi_ = (RX)p[k].im, sr = (RX)sv[k].re, si = (RX)sv[k].im;
            x[k] = {x[k].re + (axr * pr_ - axi * pi_) + (wxr * sr - wxi * si),
                    x[k].im + (axr * pi_ + axi * pr_) + (wxr * si + wxi * sr)};
            p[k] = {sv[k].re - (wr * tv[k].re - wi * tv[k].im), sv[k].im - (wr * tv[k].im + wi * tv[k].re)};
        }
        Spinor<XP>::store(fx, i, s, x);
        Spinor<P>::store(fr, i, s, p);     // the new residual (stored values)
        Spinor<P>::load(fh, i, s, h);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            part[0] += (double)h[k].re * p[k].re + (double)h[k].im * p[k].im;
            part[1] += (double)h[k].re * p[k].im - (double)h[k].im * p[k].re;
            part[2] += (double)norm2(p[k]);
        }
    }
    block_sum<3>(part);
    if (threadIdx.x == 0)
        for (int k = 0; k < 3; ++k) part_at(pr, sb, i, k) = part[k];
}

// F5 of the fused iteration: omega, rho and beta from F4's sums, then x_lo, r
// and the next p in one pass; partial |r|^2 (of the stored r)
template <int P>
__device__ __forceinline__ void bi5f_tile(const Prob &pr, int t) {
    typedef typename real_of<P>::type R;
    constexpr int XP = XPrec<P>::value;
    typedef typename real_of<XP>::type RX;
    const int sb = t / pr.nrhs, i = t - sb * pr.nrhs;
    const int s = sb * blockDim.x + threadIdx.x;
    __shared__ double sum[BI_NP2], sc[6];
    __shared__ int go;
    const BiRec &c = pr.rec3[i];
    const bool live = c.state == ST_ACTIVE;   // uniform over the block
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (live)
        for (int k = w; k < BI_NP2; k += nw) {
            const double x = wave_col_sum(part2_col(pr, i, k), pr.nsb[KS4]);
            if ((threadIdx.x & 63) == 0) sum[k] = x;
        }
    __syncthreads();
    if (threadIdx.x == 0) {
        int state = c.state;
        const dc al = {c.ar, c.ai};
        dc om = {c.wr, c.wi}, rho = {c.rr, c.ri}, be = {c.br, c.bi};
        if (live) {
            om = dc{sum[0] / sum[2], sum[1] / sum[2]};
            if (!finite_pos(sum[2]) || !dfinite(om) || (om.re == 0.0 && om.im == 0.0)) state = ST_BREAKDOWN;
            else {
                const dc ot = dmul(om, dc{sum[5], sum[6]}), old = rho;
                rho = dc{sum[3] - ot.re, sum[4] - ot.im};
                be = dmul(ddiv(rho, old), ddiv(al, om));
            }
        }
        go = state == ST_ACTIVE;
        sc[0] = al.re, sc[1] = al.im, sc[2] = om.re, sc[3] = om.im, sc[4] = be.re, sc[5] = be.im;
        if (sb == 0) {
            BiRec &o = pr.recm[i];
            o.rr = rho.re, o.ri = rho.im, o.ar = al.re, o.ai = al.im, o.wr = om.re, o.wi = om.im;
            o.br = be.re, o.bi = be.im, o.rh2 = c.rh2, o.r2 = c.r2;
            o.state = state, o.iters = c.iters, o.since_ru = c.since_ru;
        }
    }
    __syncthreads();
    if (!go) return;
    double part[1] = {0.0};
    if (s < pr.g.V) {
        FieldPtr fp{pr.p, pr.g.V, pr.nrhs}, fs{pr.sv, pr.g.V, pr.nrhs}, ft{pr.tv, pr.g.V, pr.nrhs};
        FieldPtr fr{pr.r, pr.g.V, pr.nrhs}, fv{pr.v, pr.g.V, pr.nrhs}, fx{pr.x_lo, pr.g.V, pr.nrhs};
        cx<R> p[12], sv[12], tv[12], v[12];
        cx<RX> x[12];
        Spinor<P>::load(fp, i, s, p);
        Spinor<P>::load(fs, i, s, sv);
        Spinor<XP>::load(fx, i, s, x);
        const RX axr = (RX)sc[0], axi = (RX)sc[1], wxr = (RX)sc[2], wxi = (RX)sc[3];
        const R wr = (R)sc[2], wi = (R)sc[3], br = (R)sc[4], bi = (R)sc[5];
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const RX pr_ = (RX)p[k].re, pi_ = (RX)p[k].im, sr = (RX)sv[k].re, si = (RX)sv[k].im;
            x[k] = {x[k].re + (axr * pr_ - axi * pi_) + (wxr * sr - wxi * si),
                    x[k].im + (axr * pi_ + axi * pr_) + (wxr * si + wxi * sr)};
        }
        Spinor<XP>::store(fx, i, s, x);
        Spinor<P>::load(ft, i, s, tv);
        Spinor<P>::load(fv, i, s, v);
#pragma unroll
        for (int k = 0; k < 12; ++k)   // the new residual
            sv[k] = {sv[k].re - (wr * tv[k].re - wi * tv[k].im), sv[k].im - (wr * tv[k].im + wi * tv[k].re)};
        Spinor<P>::store(fr, i, s, sv);     // stored values from here on
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            part[0] += (double)norm2(sv[k]);
            // d = p - omega v ; p = r + beta d
            const cx<R> d = {p[k].re - (wr * v[k].re - wi * v[k].im), p[k].im - (wr * v[k].im + wi * v[k].re)};
            p[k] = {sv[k].re + (br * d.re - bi * d.im), sv[k].im + (br * d.im + bi * d.re)};
        }
        Spinor<P>::store(fp, i, s, p);
    }
    block_sum<1>(part);
    if (threadIdx.x == 0) part_at(pr, sb, i, BI_R2) = part[0];
}

// The trailing finish of a chunk of fused iterations: the last F5's records and
// |r|^2 into the final records.  p is formed already; a field that restarts has
// S1 set p = r_hat = r.
__device__ __forceinline__ void bi_trail_finish(const Prob &pr) {
    __shared__ double sums[MAX_SUMS];
    sum_all(pr, pr.nsb[KS5], 1, sums, BI_R2);
    const int i = threadIdx.x;
    if (i >= pr.nrhs) return;
    Scal &c = pr.sc[i];
    BScal &b = pr.bs[i];
    BiRec o;
    bi_end(pr, pr.recm[i], c.stop2, sums[i], o);
    b.rho[0] = o.rr, b.rho[1] = o.ri, b.alpha[0] = o.ar, b.alpha[1] = o.ai;
    b.omega[0] = o.wr, b.omega[1] = o.wi, b.beta[0] = o.br, b.beta[1] = o.bi;
    b.rh2 = o.rh2;
    c.rho = o.r2;
    const bool restart = o.state == BI_RESTART;
    c.state = restart ? ST_ACTIVE : o.state;
    c.iters = o.iters;
    c.since_ru = o.since_ru;
    c.restart = c.pending_p = restart;
}

__device__ __forceinline__ void bi5_finish(const Prob &pr) {
    __shared__ double sums[MAX_SUMS];
    sum_all(pr, pr.nsb[KS5], 3, sums);
    for (int i = threadIdx.x; i < pr.nrhs; i += blockDim.x) {
        Scal &c = pr.sc[i];
        if (c.state != ST_ACTIVE) continue;
        const double re = sums[3 * i], im = sums[3 * i + 1], r2 = sums[3 * i + 2];
        {
            BScal &b = pr.bs[i];
            const dc rho_new = {re, im};
            st(b.rho_old, ld(b.rho));
            st(b.rho, rho_new);
            st(b.beta, dmul(ddiv(rho_new, ld(b.rho_old)), ddiv(ld(b.alpha), ld(b.omega))));
            c.rho = r2;
            c.iters += 1;
            c.since_ru += 1;
            if (!(r2 < 1e300) || !dfinite(rho_new)) c.state = ST_BREAKDOWN;
            else if (r2 <= c.stop2 || c.iters >= pr.max_iter ||
                     (pr.ru_every > 0 && c.since_ru >= pr.ru_every))
                c.state = ST_FROZEN;
            else {
                // (near) breakdown, <r_hat, r> ~ 0: restart in place with
                // r_hat = p = r (the iterated residual), rho = |r|^2.  A point
                // source meets it after one iteration: with r_hat = r0 = e_k, s
                // has no component along e_k and, since (1 - gamma)(1 + gamma) = 0,
                // neither has t = D s.
                if (rho_new.re * rho_new.re + rho_new.im * rho_new.im <= 1e-12 * b.rh2 * r2) {
                    c.restart = 1;
                    b.rho[0] = r2;
                    b.rho[1] = 0.0;
                    b.rh2 = r2;
                }
                c.pending_p = 1;
            }
        }
    }
}

}  // namespace wd
