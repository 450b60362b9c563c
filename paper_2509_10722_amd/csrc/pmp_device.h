// Device-side building blocks shared by the PMP kernels: reductions, the
// proximal operators of Section III-E and the per-stream / per-link updates
// of the compact over-relaxed iteration (Section III-D, III-G).
#pragma once

#include "pmp_internal.h"

#include <cmath>

namespace pmp {

__device__ __forceinline__ int ld_stream(const int *p) { return __builtin_nontemporal_load(p); }

// The XCD this wave runs on.
__device__ __forceinline__ int xcc_id()
{
    return __builtin_amdgcn_s_getreg(20 | (3 << 11));   // HW_REG_XCC_ID, 4 bits
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Sum over a workgroup of NT threads in a fixed order; the result is valid in
// thread 0.  `sh` holds NT / 64 doubles.
template <int NT>
__device__ __forceinline__ double block_sum_n(double v, double *sh)
{
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) r += sh[i];
    }
    __syncthreads();
    return r;
}

__device__ __forceinline__ double block_sum(double v, double *sh) { return block_sum_n<kBlock>(v, sh); }

// Fixed-point term of a long row's sum (Dev::fx_shift): x 2^F rounded to an
// integer (x >= 0 and below 2^62 / (row length) after scaling, by the choice of F).
__device__ __forceinline__ long long fx_term(double x, double scale)
{
    return __double2ll_rn(x * scale);
}

// Exact int64 sum over a workgroup of NT threads (valid in thread 0); `sh`
// holds NT / 64 doubles, reused as int64.
template <int NT = kBlock>
__device__ __forceinline__ long long block_sum_ll(long long v, double *sh)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    long long *s = (long long *)sh;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) s[wid] = v;
    __syncthreads();
    long long r = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < NT / 64; ++i) r += s[i];
    __syncthreads();
    return r;
}

// Stage tab[idx[i]] for i < cnt into LDS with a workgroup of NT threads, in
// three steps so that a caller can issue its other loads between them: load
// every lane's share of the index stream, issue all its gathers (up to
// CAP / NT per lane in flight together), write LDS.  Rounds past cnt are
// skipped by the whole workgroup.
template <typename T, int NT = kBlock, int CAP = kCap>
struct GatherStage {
    static constexpr int R = CAP / NT;
    int id[R];
    T val[R];
    __device__ __forceinline__ void load_indices(const int *__restrict__ idx, int cnt)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            id[r] = -1;
            if (r * NT < cnt) {
                const int i = r * NT + threadIdx.x;
                if (i < cnt) id[r] = ld_stream(idx + i);
            }
        }
    }
    __device__ __forceinline__ void gather(const T *__restrict__ tab, int cnt)
    {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r * NT < cnt) val[r] = id[r] >= 0 ? tab[id[r]] : T(0);
    }
    __device__ __forceinline__ void store(T *sh, int cnt) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r * NT < cnt && id[r] >= 0) sh[r * NT + threadIdx.x] = val[r];
    }
};

template <typename T, int NT = kBlock, int CAP = kCap>
__device__ __forceinline__ void gather_stage(const int *__restrict__ idx,
                                             const T *__restrict__ tab, T *sh, int cnt)
{
    GatherStage<T, NT, CAP> g;
    g.load_indices(idx, cnt);
    g.gather(tab, cnt);
    g.store(sh, cnt);
}

// FP64 sum of sh[b..e) in a fixed order: four interleaved partial sums
// (entries b + 4i + r go to sum r), the tail into the first, then
// (s0 + s1) + (s2 + s3).  Four independent chains hide the LDS and add
// latency of one lane's run; every kernel that sums a staged run uses this
// order, so their results agree bit for bit.
template <typename T>
__device__ __forceinline__ double run_sum(const T *sh, int b, int e)
{
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int k = b;
    for (; k + 3 < e; k += 4) {
        s0 += (double)sh[k];
        s1 += (double)sh[k + 1];
        s2 += (double)sh[k + 2];
        s3 += (double)sh[k + 3];
    }
    for (; k < e; ++k) s0 += (double)sh[k];
    return (s0 + s1) + (s2 + s3);
}

// The same sum by four neighbouring lanes (sub = 0..3), one partial sum each;
// valid in all four.
template <typename T>
__device__ __forceinline__ double run_sum4(const T *sh, int b, int e, int sub)
{
    const int body = b + ((e - b) & ~3);
    double s = 0.0;
    int k = b + sub;
    for (; k + 12 < body; k += 16) {
        const T t0 = sh[k], t1 = sh[k + 4], t2 = sh[k + 8], t3 = sh[k + 12];
        s += (double)t0;
        s += (double)t1;
        s += (double)t2;
        s += (double)t3;
    }
    for (; k < body; k += 4) s += (double)sh[k];
    if (sub == 0)
        for (k = body; k < e; ++k) s += (double)sh[k];
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    return s;
}

// Last + 1 group of four entries of a run that ends at entry e1 (up to 2^31 - 1).
__host__ __device__ __forceinline__ int quads_end(int e1) { return (e1 >> 2) + ((e1 & 3) != 0); }

// Entries of one lane of a workgroup that strides over cnt of them, in rounds
// of eight: round(k) where k, k + kBlock, ... k + 7 kBlock are all there, then
// last(k) for the rest.  Counts go up to 2^31 - 1; in unsigned no sum wraps.
template <typename R, typename L>
__host__ __device__ __forceinline__ void strided_rounds(unsigned cnt, unsigned lane, R round, L last)
{
    unsigned k = lane;
    for (; k + 7u * kBlock < cnt; k += 8u * kBlock) round(k);
    if (k < cnt) last(k);
}

// Sum of tab[idx[k]] over k = b + threadIdx.x, + kBlock, ... below e, added in
// that order, in FP64 or (term: FP64 -> int64) in integers; eight gathers per
// lane in flight.
template <typename T, typename A, typename F>
__device__ __forceinline__ A strided_sum(const int *__restrict__ idx, const T *tab, int b, int e,
                                         F term)
{
    A acc = 0;
    const int *p = idx + b;
    const unsigned cnt = (unsigned)(e - b);
    auto round = [&](unsigned k) {
        int id[8];
        T v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) id[r] = ld_stream(p + k + r * kBlock);
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = tab[id[r]];
#pragma unroll
        for (int r = 0; r < 8; ++r) acc += term((double)v[r]);
    };
    auto last = [&](unsigned k) {
        int id[8];
        T v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) id[r] = k + r * kBlock < cnt ? ld_stream(p + k + r * kBlock) : -1;
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = id[r] >= 0 ? tab[id[r]] : T(0);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (id[r] >= 0) acc += term((double)v[r]);
    };
    strided_rounds(cnt, threadIdx.x, round, last);
    return acc;
}

// The per-stream and per-link updates below are shared by every layout, whose
// results are to agree bit for bit: the compiler does not contract their
// expressions (which it would do differently from kernel to kernel), and each
// fused multiply-add is written out.

// Proximal operator of one traffic stream with L terminals and sum of
// arguments S (Section III-E), clipped to the box; irho = 1 / rho.  wsig > 0: log utility
// with weight wsig (alpha2 = false) or -w / x with weight wsig (alpha2 =
// true); wsig < 0: linear utility with weight -wsig.  For S < 0 the log root
// uses the equal form 2w / (rho (sqrt(S^2 + 4wL/rho) - S)).  The -w / x prox
// is the positive root of L x^3 - S x^2 - w / rho = 0, reached by Newton's
// method from max(S/L, 0) + (w / (rho L))^(1/3), where the cubic is
// nonnegative and convex, so the iterates decrease monotonically.
//
// FP64 divides and square roots are what the epilogues spend their time on
// (one wave64 FP64 instruction a clock and CU, about 12 for a divide, 20 for
// a root): every closed form is one quotient num / den, so a stream costs one
// divide and, with a log utility, one root (four divides before).
__device__ __forceinline__ double prox_stream(double S, int L, double wsig, double irho,
                                              double lo, double hi, bool alpha2 = false)
{
#pragma clang fp contract(off)
    if (L == 0) return hi;
    double x;
    const double dl = (double)L;
    const double q = fabs(wsig) * irho;   // w / rho
    if (alpha2) {
        x = (S > 0.0 ? S / dl : 0.0) + cbrt(q / dl);
        for (int it = 0; it < 100; ++it) {
            const double g = (dl * x - S) * x * x - q;
            const double nx = x - g / ((3.0 * dl * x - 2.0 * S) * x);
            if (!(nx < x)) break;
            x = nx;
        }
    } else {
        double num = S + q, den = dl;     // linear
        if (wsig > 0.0) {                 // log
            const double disc = sqrt(__builtin_fma(S, S, 4.0 * (dl * q)));
            num = S < 0.0 ? 2.0 * q : S + disc;
            den = S < 0.0 ? disc - S : 2.0 * dl;
        }
        x = num / den;
    }
    return fmin(fmax(x, lo), hi);
}

// A check also screens the state it writes: a non-finite entry can leave the
// residuals finite (the box clip and the slack prox's max discard NaN), so
// it turns the partial sum into NaN, which finalize reports as
// PMP_ERR_NUMERIC.
__device__ __forceinline__ double screen(double part, double v)
{
    return isfinite(v) ? part : __builtin_nan("");
}

template <typename T>
__device__ __forceinline__ bool is_alpha2(const Dev<T> &d, int j)
{
    return d.util != nullptr && d.util[j] == PMP_UTIL_ALPHA2;
}

// One stream's update: new rate and a from the summed link values.
template <typename T>
__device__ __forceinline__ void stream_core(double a, double wsig, int L, double vsum, double irho,
                                            double lo, double hi, double alpha, bool alpha2, T &xt,
                                            T &at)
{
#pragma clang fp contract(off)
    const double S = __builtin_fma((double)L, a, vsum);
    xt = (T)prox_stream(S, L, wsig, irho, lo, hi, alpha2);
    at = (T)__builtin_fma(alpha, (double)xt, (1.0 - alpha) * a);
}

template <typename T, bool CHECK>
__device__ __forceinline__ double stream_update(const Dev<T> &d, int j, int L, double vsum,
                                                double irho)
{
    T xt, at;
    stream_core<T>((double)d.a[j], (double)d.wsig[j], L, vsum, irho, d.lo, d.hi, d.alpha,
                   is_alpha2(d, j), xt, at);
    double part = 0.0;
    if (CHECK) {                       // dual residual: sum_j L_j (dx_j)^2
        const double dx = (double)xt - (double)d.x[j];
        part = screen((double)L * dx * dx, (double)at);
    }
    d.x[j] = xt;
    d.a[j] = at;
    return part;
}

// Per-link inputs of the link update, loaded ahead of it so that the loads
// of several links can be in flight before any of their stores.
struct LinkIn {
    double c, u, b, zs;
    double yp, pp;   // saved y and ps of the previous iteration (checks only)
};

template <typename T, int MODE>
__device__ __forceinline__ LinkIn link_load(const Dev<T> &d, int l)
{
    LinkIn in{(double)d.c[l], (double)d.u[l], (double)d.b[l], (double)d.zs[l], 0.0, 0.0};
    if (MODE == kCheck) {
        in.yp = d.y_prev[l];
        in.pp = d.ps_prev[l];
    }
    return in;
}

// One link's update: new b, u, zs (and v = b - u, returned) and the slack prox
// ps from the link sum y; a check adds the link's residual terms.
template <typename T, bool CHECK>
__device__ __forceinline__ T link_core(double al, int deg, double y, const LinkIn &in, T &bt,
                                       T &ut, T &zt, double &ps, double &r2, double &s2)
{
#pragma clang fp contract(off)
    const double c = in.c, u = in.u, b = in.b, zs = in.zs;
    ps = fmax(zs - u, -c);                              // slack prox
    const double cnt = (double)deg + 1.0;               // |l| = d_l + 1
    const double pbar = (y + ps) / cnt;                 // link average
    bt = (T)__builtin_fma(-al, pbar, (1.0 - al) * b);
    ut = (T)__builtin_fma(al, pbar, u);
    zt = (T)__builtin_fma(al, ps - pbar, (1.0 - al) * zs);
    if (CHECK) {
        // ||r||^2 = sum_l |l| pbar_l^2 and, with D the change since the
        // previous iteration, the link part of ||s||^2 / rho^2:
        // sum_{j on l} (Dx_j - Dpbar)^2 + (Dps - Dpbar)^2
        //   = [sum_j Dx_j^2] + d Dpbar^2 - 2 Dpbar Dy + (Dps - Dpbar)^2,
        // the bracket being added on the stream side.
        const double yp = in.yp, pp = in.pp;
        const double dpb = pbar - (yp + pp) / cnt;
        const double dy = y - yp, dps = ps - pp;
        r2 += screen(cnt * pbar * pbar, (double)bt + (double)ut + (double)zt);
        s2 += (double)deg * dpb * dpb - 2.0 * dpb * dy + (dps - dpb) * (dps - dpb);
    }
    return (T)((double)bt - (double)ut);
}

template <typename T, int MODE, bool WRITE_V = true>
__device__ __forceinline__ double link_update_in(const Dev<T> &d, int l, int deg, double y,
                                               const LinkIn &in, double &r2, double &s2)
{
    T bt, ut, zt;
    double ps;
    const T vt = link_core<T, MODE == kCheck>(d.alpha, deg, y, in, bt, ut, zt, ps, r2, s2);
    if (d.mu_out) d.mu_out[l] = in.zs - in.u > -in.c ? 1 : 0;   // ps's branch, for reverse mode
    d.b[l] = bt;
    d.zs[l] = zt;
    d.u[l] = ut;
    if (WRITE_V) d.v[l] = vt;
    if (MODE != kPlain) {
        d.y_prev[l] = y;
        d.ps_prev[l] = ps;
    }
    return (double)vt;
}

template <typename T, int MODE, bool WRITE_V = true>
__device__ __forceinline__ double link_update(const Dev<T> &d, int l, int deg, double y,
                                            double &r2, double &s2)
{
    return link_update_in<T, MODE, WRITE_V>(d, l, deg, y, link_load<T, MODE>(d, l), r2, s2);
}

// A balancing step's rescale u <- (rho_old / rho_new) u (eq. (18)); returns v = b - u.
template <typename T>
__device__ __forceinline__ T link_rescale(T b, T &u, double ratio)
{
#pragma clang fp contract(off)
    u = (T)((double)u * ratio);
    return (T)((double)b - (double)u);
}

// ---- reverse mode (one reversed iteration; see pmp_adjoint.hip) ------------

// Per-link and per-stream inputs of a reversed iteration, loaded ahead of the
// sums they are combined with.
struct AdjLinkIn {
    double B, Z, U, cbar;
    bool mu;
    // without a mask (no link step in this kernel) only B and U are needed
    __device__ __forceinline__ void load(const AdjDev &a, int l, const uint8_t *mask)
    {
        B = a.B[l];
        U = a.U[l];
        Z = cbar = 0.0;
        mu = false;
        if (mask) {
            Z = a.Z[l];
            cbar = a.cbar[l];
            mu = mask[l] != 0;
        }
    }
};

// Returns the link's ybar.
__device__ __forceinline__ double adj_link_step(const AdjDev &a, int l, int deg, double alpha,
                                                const AdjLinkIn &in)
{
    const double B = in.B, Z = in.Z, U = in.U;
    const double inv = 1.0 / ((double)deg + 1.0);
    const double pbb = alpha * (U - B - Z);
    const double psb = alpha * Z + pbb * inv;
    const double m1 = in.mu ? 1.0 : 0.0;
    const double ybar = pbb * inv;
    a.ybar[l] = ybar;
    a.cbar[l] = in.cbar - (1.0 - m1) * psb;
    a.B[l] = (1.0 - alpha) * B;
    a.Z[l] = (1.0 - alpha) * Z + m1 * psb;
    a.U[l] = U - m1 * psb;
    return ybar;
}

template <typename T>
struct AdjStreamIn {
    double A, ext, wbar, x, wsig;
    bool a2;
    __device__ __forceinline__ void load(const Dev<T> &d, const AdjDev &a, const T *xt, int j, int last)
    {
        A = a.A[j];
        ext = last ? a.ext[j] : 0.0;
        wbar = a.wbar[j];
        x = (double)xt[j];
        wsig = (double)d.wsig[j];
        a2 = is_alpha2(d, j);
    }
};

// Returns the stream's Sbar.
template <typename T>
__device__ __forceinline__ double adj_stream_step(const Dev<T> &d, const AdjDev &a,
                                                  const AdjStreamIn<T> &in, int j, int L,
                                                  double ysum, double rho)
{
    const double xbar = d.alpha * in.A + ysum + in.ext;
    const double x = in.x, wsig = in.wsig;
    double sbar = 0.0;
    if (L > 0 && x > d.lo && x < d.hi) {
        double dS, dw;
        if (in.a2) {
            // rho L x^3 - rho S x^2 - w = 0:  dx/dS = rho x^3 / (rho L x^3 + 2w),
            // dx/dw = x / (rho L x^3 + 2w)
            const double den = rho * (double)L * x * x * x + 2.0 * wsig;
            dS = rho * x * x * x / den;
            dw = x / den;
        } else if (wsig > 0.0) {
            const double den = rho * (double)L * x * x + wsig;
            dS = rho * x * x / den;
            dw = x / den;
        } else {
            dS = 1.0 / (double)L;
            dw = 1.0 / (rho * (double)L);
        }
        sbar = xbar * dS;
        a.wbar[j] = in.wbar + xbar * dw;
    }
    a.A[j] = (1.0 - d.alpha) * in.A + (double)L * sbar;
    a.Sbar[j] = sbar;
    return sbar;
}

// ---- residual reduction, stop rule and rho balancing ---------------------

// Thread 0 of the check-finalize kernel: residual norms (Section III-F), the
// stop rule, and residual balancing of rho (Section III-G).  nrm (or NULL):
// sums of squares of p, z and u over all terminals, for the relative part
// of the stop rule: ||r|| < eps_abs sqrt(J) + eps_rel max(||p||, ||z||) and
// ||s|| < eps_abs sqrt(J) + eps_rel ||rho u||.
// c: the control block, h: the history entry of this check.
__device__ inline void finalize(Ctl *c, HistEntry &h, long long delta, int stop, double sr,
                                double ss, const double *nrm = nullptr)
{
    const double rho = c->rho;
    const long long it = c->iter + delta;
    const double r = sqrt(sr);
    const double s = rho * sqrt(ss > 0.0 ? ss : (ss == ss ? 0.0 : ss));   // keeps a NaN
    double tol_r = c->eps_tol, tol_s = c->eps_tol;
    if (nrm && c->eps_rel > 0.0) {
        c->p_norm = sqrt(fmax(nrm[0], 0.0));
        c->z_norm = sqrt(fmax(nrm[1], 0.0));
        c->u_norm = rho * sqrt(fmax(nrm[2], 0.0));
        tol_r += c->eps_rel * fmax(c->p_norm, c->z_norm);
        tol_s += c->eps_rel * c->u_norm;
    }
    c->iter = it;
    c->r_norm = r;
    c->s_norm = s;
    c->ratio = 1.0;
    h.iter = it;
    h.r_norm = r;
    h.s_norm = s;
    h.rho = rho;
    c->nhist += 1;
    if (!isfinite(r) || !isfinite(s)) {
        c->status = PMP_ERR_NUMERIC;
        c->done = 1;
    } else if (stop && r < tol_r && s < tol_s) {
        c->status = PMP_OK;
        c->done = 1;
    } else if (c->adapt_every > 0 && it % c->adapt_every == 0) {
        double rn = rho;
        if (r > c->mu * s) rn = c->gamma * rho;
        else if (s > c->mu * r) rn = rho / c->gamma;
        c->ratio = rho / rn;
        c->rho = rn;
        c->irho = 1.0 / rn;
    }
}

}  // namespace pmp
