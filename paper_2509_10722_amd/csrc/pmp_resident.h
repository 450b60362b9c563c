// PMP iterations of a small instance held on chip.
//
// A network of some thousand links and streams gives each pass of the gather
// layout well under a microsecond of work, yet the two passes of an iteration
// take 4-5 us each: a chain of dependent global loads (done flag, block table,
// pointers, indices, gathered values, state) and a launch.  Here a few
// workgroups run as many iterations as the call asks in one launch.  Every
// lane keeps one stream and one link: its state and the first kSlots entries
// of its index list stay in registers, and the vector it gathers from (v in
// the stream phase, x in the link phase) sits whole in LDS.
//
// One workgroup (up to kRT streams and links) needs only its own barriers.
// Several workgroups exchange x and v through memory and meet at a barrier
// after each phase.  They all run on one XCD and so share its L2: a store is
// in that L2 once the wave's vmcnt is down, and a load of agent scope passes
// by the L1, so neither needs a cache writeback or invalidate.  Such a barrier
// takes about 0.6 us; with stores of agent scope,
// which workgroups on several XCDs would need, the exchange takes 5-10 us.
//
// Roll call: 8 G workgroups are launched for a group of G.  Each takes a
// ticket of the XCD it runs on (by the pigeonhole principle some XCD deals G
// tickets once all have started), the first XCD to deal G wins, and the rest
// leave.  All members are then running, so the phase barriers complete.  If
// no XCD gets that far in kRollTicks (the GPU is shared with other long
// kernels), the workgroups that have started on the XCD with the most of them
// run this launch's iterations, rows dealt out in turn and everything read
// from memory; a launch has about a thousand iterations at most (launch_resident's
// callers), so the next one soon calls the roll again.  30,000 x 30,000: 41 us an
// iteration on 24 of the 30 workgroups, 62 on 8, 113 on 4, 392 on one alone.
//
// What bounds it is latency: LDS round trips, the barriers, the FP64 divide
// and root of the prox.  Measured on MI355X, us an iteration against the two
// gather passes: 200 links x 1,000 streams 2.0 (9.1) in FP64, 2.1 (9.5) in
// FP32; 8,000 x 8,000 with 64,000 nonzeros 5.2 (9.8); 30,000 x 30,000 with
// 300,000 nonzeros 7.5 (11.3).  The largest side has 32,768 rows (a lane each in 32
// workgroups); the LDS holds 40,696 in FP32, 20,344 in FP64.
//
// Every sum keeps the gather layout's order (run_sum) and every update its
// arithmetic (stream_core, link_core), so the iterates are the same bit for
// bit; only the order of the residual sums of a check is its own.
//
// Part of pmp_kernels.hip, which includes it.
#pragma once

#include "pmp_device.h"

#include <algorithm>

namespace pmp {

namespace {

constexpr int kRT = 1024;             // lanes of a workgroup
constexpr int kRWaves = kRT / 64;
constexpr int kSlots = 16;            // index entries per lane and side in registers
constexpr int kResMaxGroup = 32;      // workgroups of a group: one per CU of an XCD
constexpr int kResSteps1 = 4, kResSteps4 = 12;       // steps past the slots (resident_plan)
constexpr size_t kResLds = 159 * 1024;               // LDS for the staged vectors
constexpr unsigned long long kRollTicks = 400000;    // 4 ms of the 100 MHz wall clock
constexpr unsigned kResPolls = 1u << 26;             // bound of a phase barrier's wait
// ResSync::win: nobody yet; XCD + 1 of a whole group; being closed; a barrier
// gave up, no more launches; kFew + 8 (g - 1) + XCD: its first g workgroups
constexpr unsigned kOpen = 0, kClosing = 97, kGone = 98, kFew = 99;

template <typename V>
__device__ __forceinline__ V ld_agent(const V *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One lane's part of one segment (route or link row) of L entries, summed in
// run_sum's order: four partial sums over the body (the first L & ~3 entries),
// the tail into the first of them.  Q = 1: one lane has all four.  Q = 4: lane
// `sub` has one, lane 0 the tail too.  The first 16 of its body entries and
// the tail are kept as 16-bit indices in registers; a slot without an entry
// points at tab[zero], which holds 0, so the sum has no branches that differ
// between lanes (adding +0 changes nothing).
struct Seg {
    int b, L;                        // first entry, entries of the segment
    int nb, sub;                     // entries of each partial sum's body
    int steps;                       // the wave's most body slots (Q = 1: of each sum; Q = 4: fours)
    unsigned pk[kSlots / 2], tl[2];  // two indices a word: body, tail
    __device__ __forceinline__ void init(const int *ptr, const int *idx, int row, bool valid, bool q4,
                                         int s, int zero)
    {
        b = valid ? ptr[row] : 0;
        L = valid ? ptr[row + 1] - b : 0;
        sub = s;
        nb = L / 4;
        const int body = q4 ? nb : 4 * nb, ntail = q4 && s ? 0 : L - 4 * nb;
        auto at = [&](int i) { return (unsigned)(i < body ? idx[q4 ? b + 4 * i + s : b + i] : zero); };
        auto tail = [&](int i) { return (unsigned)(i < ntail ? idx[b + 4 * nb + i] : zero); };
#pragma unroll
        for (int i = 0; i < kSlots; i += 2) pk[i / 2] = at(i) | at(i + 1) << 16;
        tl[0] = tail(0) | tail(1) << 16;
        tl[1] = tail(2);
        int w = min((body + 3) / 4, kSlots / 4);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) w = max(w, __shfl_xor(w, off, 64));
        steps = __builtin_amdgcn_readfirstlane(w);
    }
    __device__ __forceinline__ int slot(int i) const
    {
        return (int)(i & 1 ? pk[i / 2] >> 16 : pk[i / 2] & 0xffffu);
    }
    // The loads of N fours of body slots and of the tail in flight together.
    template <int N, typename T>
    __device__ __forceinline__ double sum_n(const T *tab, const int *idx, bool q4) const
    {
        T v[4 * N + 1];
#pragma unroll
        for (int i = 0; i < 4 * N; ++i) v[i] = tab[slot(i)];
        const T t0 = tab[tl[0] & 0xffffu], t1 = tab[tl[0] >> 16], t2 = tab[tl[1]];
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        if (!q4) {
#pragma unroll
            for (int i = 0; i < 4 * N; i += 4) {
                s0 += (double)v[i];
                s1 += (double)v[i + 1];
                s2 += (double)v[i + 2];
                s3 += (double)v[i + 3];
            }
            for (int k = kSlots; k < 4 * nb; k += 4) {      // a long segment's further entries
                const int *p = idx + b + k;
                const int i0 = p[0], i1 = p[1], i2 = p[2], i3 = p[3];
                s0 += (double)tab[i0];
                s1 += (double)tab[i1];
                s2 += (double)tab[i2];
                s3 += (double)tab[i3];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4 * N; ++i) s0 += (double)v[i];
            for (int k = kSlots; k < nb; ++k) s0 += (double)tab[idx[b + 4 * k + sub]];
        }
        s0 += (double)t0;
        s0 += (double)t1;
        s0 += (double)t2;
        if (!q4) return (s0 + s1) + (s2 + s3);
        s0 += __shfl_xor(s0, 1, 64);
        s0 += __shfl_xor(s0, 2, 64);
        return s0;
    }
    // run_sum of tab over the segment, valid in all its lanes.
    template <typename T>
    __device__ __forceinline__ double sum(const T *tab, const int *idx, bool q4) const
    {
        switch (steps) {        // uniform in the wave
        case 0: return sum_n<0, T>(tab, idx, q4);
        case 1: return sum_n<1, T>(tab, idx, q4);
        case 2: return sum_n<2, T>(tab, idx, q4);
        case 3: return sum_n<3, T>(tab, idx, q4);
        default: return sum_n<4, T>(tab, idx, q4);
        }
    }
};

// Copy src[0..cnt) (written by the group's workgroups before the barrier) to
// LDS and append a zero: 16 bytes a lane straight into LDS, agent scope, all
// in flight at once.  Reads up to 15 bytes past the end, which the workspace's
// 256-byte padding of each vector covers.
template <typename T>
__device__ __forceinline__ void stage(const T *src, T *dst, int cnt)
{
    typedef __attribute__((address_space(1))) const void gvoid;
    typedef __attribute__((address_space(3))) void lvoid;
    constexpr int kSc1 = 16;             // cache policy bit: agent scope
    const int quads = (cnt * (int)sizeof(T) + 15) / 16;
    const int wave = threadIdx.x & ~63;
    for (int i = wave; i < quads; i += kRT)
        if (i + (int)(threadIdx.x & 63) < quads)
            __builtin_amdgcn_global_load_lds((gvoid *)((const char *)src + 16 * (size_t)(i + (threadIdx.x & 63))),
                                             (lvoid *)((char *)dst + 16 * (size_t)i), 16, 0, kSc1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) dst[cnt] = T(0);
    __syncthreads();
}

// Barrier of the group's workgroups (`epoch` counts them); false if it gave
// up.  Every workgroup stores its epoch in its own word, and one wave of each
// reads all the words until they have it: no chain of atomic adds.  A wait of
// more than kResPolls polls ends the launch: `abort` makes the others leave too,
// and closes the roll calls of the launches after it, since the workgroups may
// stand at different phases of an iteration and their words at different
// barriers; the host's word has the calls that read the iterate say so
// (pmp_set_state clears both).
__device__ __forceinline__ bool group_sync(ResSync *rs, int *failed, int role, int G, unsigned epoch, int *s_ok)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores are in the L2
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        if (lane == 0)
            __hip_atomic_store(&rs->flag[role], epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        bool ok = true;
        unsigned polls = 0;
        while (!__all(lane >= G || (int)(ld_agent(&rs->flag[lane]) - epoch) >= 0))
            if (++polls > kResPolls || ld_agent(&rs->abort)) {
                if (lane == 0) {
                    atomicExch(&rs->abort, 1u);
                    __hip_atomic_store(failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                }
                ok = false;
                break;
            }
        if (lane == 0) *s_ok = ok;
    }
    __syncthreads();
    return *s_ok != 0;
}

// Reduce r2, ss and (relative rule) the norms q over the workgroup into
// out[0..5) (thread 0).
__device__ __forceinline__ void reduce_parts(double r2, double ss, bool rel, const double *q,
                                             double *sred, double *out)
{
    r2 = block_sum_n<kRT>(r2, sred);
    ss = block_sum_n<kRT>(ss, sred);
    if (threadIdx.x == 0) {
        out[0] = r2;
        out[1] = ss;
    }
    if (rel)
        for (int k = 0; k < 3; ++k) {
            const double t = block_sum_n<kRT>(q[k], sred);
            if (threadIdx.x == 0) out[2 + k] = t;
        }
}

// run_sum of tab[idx[b..e)) from memory (tab: written by the group).
template <typename T>
__device__ __forceinline__ double run_sum_idx(const T *tab, const int *idx, int b, int e)
{
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int k = b;
    for (; k + 3 < e; k += 4) {
        const T t0 = ld_agent(tab + idx[k]), t1 = ld_agent(tab + idx[k + 1]);
        const T t2 = ld_agent(tab + idx[k + 2]), t3 = ld_agent(tab + idx[k + 3]);
        s0 += (double)t0;
        s1 += (double)t1;
        s2 += (double)t2;
        s3 += (double)t3;
    }
    for (; k < e; ++k) s0 += (double)ld_agent(tab + idx[k]);
    return (s0 + s1) + (s2 + s3);
}

// The group's partials of a check, added in the same order by each workgroup
// (thread 0).
__device__ __forceinline__ void add_parts(ResSync *rs, int G, double *parts)
{
    for (int k = 0; k < 5; ++k) {
        double t = 0.0;
        for (int g = 0; g < G; ++g) t += ld_agent(&rs->part[g][k]);
        parts[k] = t;
    }
}

// The iterations by a smaller group than they were laid out for, from memory.
template <typename T>
__device__ bool run_few(const Dev<T> &d, ResSync *rs, int role, int G, unsigned &epoch, Ctl &c, HistEntry &h,
                        double *sred, double *parts, int *s_ok, int iters, int end, int ce, int adapt)
{
    const int first = role * kRT + (int)threadIdx.x, step = G * kRT;
    const long long it0 = c.iter;
    for (int i = 1; i <= iters; ++i) {
        const long long it = it0 + i;
        const bool stop = ce > 0 && it % ce == 0;
        const bool check = i == end || stop || (adapt > 0 && it % adapt == 0);
        const bool rel = check && c.eps_rel > 0.0;
        const double irho = c.irho;
        double ss = 0.0, r2 = 0.0, q[3] = {0.0, 0.0, 0.0};
        for (int j = first; j < d.n; j += step) {
            const int b = d.col_ptr[j], L = d.col_ptr[j + 1] - b;
            const double acc = run_sum_idx<T>(d.v, d.row_idx, b, b + L);
            ss += stream_update<T, true>(d, j, L, acc, irho);
            if (rel) {
                const double xj = (double)d.x[j], aj = (double)d.a[j];
                q[0] += (double)L * xj * xj;
                q[1] += (double)L * aj * aj;
            }
        }
        if (!group_sync(rs, d.res_failed, role, G, ++epoch, s_ok)) return false;
        for (int l = first; l < d.m; l += step) {
            const int b = d.row_ptr[l], deg = d.row_ptr[l + 1] - b;
            const double acc = run_sum_idx<T>(d.x, d.col_idx, b, b + deg);
            link_update<T, kCheck>(d, l, deg, acc, r2, ss);
            if (rel) {
                const double dg = (double)deg, bl = (double)d.b[l], z = (double)d.zs[l], ul = (double)d.u[l];
                q[0] += d.ps_prev[l] * d.ps_prev[l];
                q[1] += z * z - dg * bl * bl - 2.0 * bl * z;
                q[2] += (dg + 1.0) * ul * ul;
            }
        }
        if (check) reduce_parts(r2, ss, rel, q, sred, rs->part[role]);
        if (!group_sync(rs, d.res_failed, role, G, ++epoch, s_ok)) return false;
        if (!check) continue;
        if (threadIdx.x == 0) {
            add_parts(rs, G, parts);
            finalize(&c, h, it - c.iter, stop ? 1 : 0, parts[0], parts[1], rel ? parts + 2 : nullptr);
            if (role == 0) d.hist[(c.nhist - 1) % kHist] = h;
        }
        __syncthreads();
        if (c.ratio != 1.0) {
            for (int l = first; l < d.m; l += step) {
                T ut = d.u[l];
                d.v[l] = link_rescale<T>(d.b[l], ut, c.ratio);
                d.u[l] = ut;
            }
            if (!group_sync(rs, d.res_failed, role, G, ++epoch, s_ok)) return false;
        }
        if (c.done) break;
    }
    return true;
}

// `iters` iterations from the state in memory.  Residuals (and rho balancing
// where due) at iteration counts that are multiples of adapt_every and at the
// iteration `end` (0: at none); with ce > 0 at multiples of ce too, where the
// stop rule ends the run.  ONE: a single workgroup, which ends in a check; else a
// group of G on one XCD.
template <typename T, bool ONE>
__global__ __launch_bounds__(kRT) void k_resident(Dev<T> d, ResSync *rs, int G, int iters, int end,
                                                  int ce, int adapt)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Ctl c;
    __shared__ HistEntry h;
    __shared__ double sred[kRWaves], parts[5];
    __shared__ int s_role, s_size, s_ok;
    __shared__ long long s_last;            // iteration count at the end
    const int tid = threadIdx.x, m = d.m, n = d.n;
    if (ONE) {
        if (d.ctl->done) return;
    } else {
        if (tid == 0) {
            int role = -1, size = 0;
            if (!ld_agent(&d.ctl->done)) {
                const unsigned x = (unsigned)xcc_id() % 8u;
                const unsigned t = atomicAdd(&rs->cnt[x * 64], 1u);
                if (t == (unsigned)G - 1u) atomicCAS(&rs->win, kOpen, x + 1u);
                const unsigned long long t0 = wall_clock64();
                unsigned w;
                while ((w = ld_agent(&rs->win)) == kOpen || w == kClosing)
                    if (w == kOpen && wall_clock64() - t0 > kRollTicks &&
                        atomicCAS(&rs->win, kOpen, kClosing) == kOpen) {
                        // (every ticket's workgroup runs and waits in this loop)
                        unsigned most = 0, on = 0;
                        for (unsigned k = 0; k < 8; ++k) {
                            const unsigned g = min(ld_agent(&rs->cnt[k * 64]), (unsigned)G);
                            if (g > most) {
                                most = g;
                                on = k;
                            }
                        }
                        atomicExch(&rs->win, kFew + 8u * (most - 1u) + on);
                    }
                if (w == x + 1u) size = G;
                else if (w >= kFew && (w - kFew) % 8u == x) size = (int)((w - kFew) / 8u + 1u);
                if (t < (unsigned)size) role = (int)t;
            }
            s_size = size;
            s_role = role;
        }
        __syncthreads();
    }
    const int role = ONE ? 0 : s_role;
    if (role >= 0) {
        if (tid == 0) {
            c = *d.ctl;
            s_last = c.iter + iters;
        }
        __syncthreads();
    }
    // barriers are numbered on from the last launch: the words need no reset
    unsigned epoch = ONE || role < 0 ? 0u : rs->base;
    bool ok = true;
    if (!ONE && role >= 0 && s_size < G) {
        // The instance is the kernel's first argument, read here through a pointer
        // the compiler knows nothing of: it loads what run_few uses in this branch,
        // and the iterations below keep those registers (82 -> 39 of them spilled;
        // 8,000 x 8,000 5.34 -> 5.16 us an iteration).
        const Dev<T> *dp = (const Dev<T> *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(dp));
        ok = run_few<T>(*dp, rs, role, s_size, epoch, c, h, sred, parts, &s_ok, iters, end, ce, adapt);
    } else if (role >= 0) {
        T *xs = (T *)lds;
        T *vs = ONE ? xs + ((n + 8) & ~7) : xs;   // a group needs one of them at a time
        // this workgroup's streams [s0, s1) and links [l0, l1)
        const int ns = (n + G - 1) / G, nl = (m + G - 1) / G;
        const int s0 = min(n, role * ns), s1 = min(n, s0 + ns);
        const int l0 = min(m, role * nl), l1 = min(m, l0 + nl);
        const bool sq = 4 * ns <= kRT, lq = 4 * nl <= kRT;     // four lanes a segment
        const int j = s0 + (sq ? tid / 4 : tid), l = l0 + (lq ? tid / 4 : tid);
        const bool has_s = j < s1, has_l = l < l1;
        const bool own_s = has_s && !(sq && tid % 4), own_l = has_l && !(lq && tid % 4);
        Seg sseg, lseg;
        T a = T(0), w = T(0), b = T(0), zs = T(0), u = T(0), cap = T(0), xo = T(0);
        double yp = 0.0, pp = 0.0;
        bool a2 = false;
        sseg.init(d.col_ptr, d.row_idx, j, has_s, sq, tid % 4, m);
        lseg.init(d.row_ptr, d.col_idx, l, has_l, lq, tid % 4, n);
        if (has_s) {
            a = d.a[j];
            w = d.wsig[j];
            a2 = is_alpha2(d, j);
            xo = d.x[j];
        }
        if (has_l) {
            b = d.b[l];
            zs = d.zs[l];
            u = d.u[l];
            cap = d.c[l];
            yp = d.y_prev[l];
            pp = d.ps_prev[l];
        }
        stage<T>(d.v, vs, m);
        if (ONE && tid == 0) xs[n] = T(0);
        const long long it0 = c.iter;
        // iterations to the next check with a stop test and to the next
        // balancing one (counted down: a 64-bit remainder costs a microsecond
        // an iteration)
        int to_stop = ce > 0 ? ce - (int)(it0 % ce) : 0;
        int to_adapt = adapt > 0 ? adapt - (int)(it0 % adapt) : 0;
        for (int i = 1; i <= iters; ++i) {
            const bool stop = --to_stop == 0, balance = --to_adapt == 0;
            if (stop) to_stop = ce;
            if (balance) to_adapt = adapt;
            const bool check = (ONE ? i == iters : i == end) || stop || balance;
            const double irho = c.irho;
            double ss = 0.0, r2 = 0.0;
            if (has_s) {
                T xt, at;
                stream_core<T>((double)a, (double)w, sseg.L, sseg.sum<T>(vs, d.row_idx, sq), irho, d.lo,
                               d.hi, d.alpha, a2, xt, at);
                if (own_s) {
                    if (check) {
                        const double dx = (double)xt - (double)xo;
                        ss += screen((double)sseg.L * dx * dx, (double)at);
                    }
                    if (ONE) xs[j] = xt;
                    else d.x[j] = xt;
                }
                xo = xt;
                a = at;
            }
            if (ONE) {
                __syncthreads();
            } else {
                if (!(ok = group_sync(rs, d.res_failed, role, G, ++epoch, &s_ok))) break;
                stage<T>(d.x, xs, n);
            }
            if (has_l) {
                const double y = lseg.sum<T>(xs, d.col_idx, lq);
                const LinkIn in{(double)cap, (double)u, (double)b, (double)zs, yp, pp};
                double ps, rl = 0.0, sl = 0.0;
                const T vt = check ? link_core<T, true>(d.alpha, lseg.L, y, in, b, u, zs, ps, rl, sl)
                                   : link_core<T, false>(d.alpha, lseg.L, y, in, b, u, zs, ps, rl, sl);
                yp = y;
                pp = ps;
                if (own_l) {
                    r2 += rl;
                    ss += sl;
                    if (ONE) vs[l] = vt;
                    else d.v[l] = vt;
                }
            }
            if (check) {
                double q[3] = {0.0, 0.0, 0.0};
                const bool rel = c.eps_rel > 0.0;
                if (rel) {              // the norms of k_rel_norms, from registers
                    if (own_s) {
                        const double L = (double)sseg.L;
                        q[0] += L * (double)xo * (double)xo;
                        q[1] += L * (double)a * (double)a;
                    }
                    if (own_l) {
                        const double dg = (double)lseg.L, bl = (double)b, z = (double)zs;
                        q[0] += pp * pp;
                        q[1] += z * z - dg * bl * bl - 2.0 * bl * z;
                        q[2] += (dg + 1.0) * (double)u * (double)u;
                    }
                }
                reduce_parts(r2, ss, rel, q, sred, ONE ? parts : rs->part[role]);
            }
            if (ONE) {
                __syncthreads();
            } else {
                if (!(ok = group_sync(rs, d.res_failed, role, G, ++epoch, &s_ok))) break;
                stage<T>(d.v, vs, m);
            }
            if (check) {
                // every workgroup takes the same decisions on its own copy of
                // the control block
                if (tid == 0) {
                    if (!ONE) add_parts(rs, G, parts);
                    finalize(&c, h, it0 + i - c.iter, stop ? 1 : 0, parts[0], parts[1],
                             c.eps_rel > 0.0 ? parts + 2 : nullptr);
                    if (role == 0) d.hist[(c.nhist - 1) % kHist] = h;
                }
                __syncthreads();
                const double ratio = c.ratio;
                if (ratio != 1.0) {     // rho changed: u <- (rho_old / rho_new) u (eq. (18))
                    const T vt = link_rescale<T>(b, u, ratio);
                    if (own_l) {
                        if (ONE) vs[l] = vt;
                        else d.v[l] = vt;
                    }
                    if (ONE) {
                        __syncthreads();
                    } else {
                        if (!(ok = group_sync(rs, d.res_failed, role, G, ++epoch, &s_ok))) break;
                        stage<T>(d.v, vs, m);
                    }
                }
                if (c.done) break;      // the same in every lane and workgroup
            }
        }
        if (own_s) {
            d.x[j] = xo;
            d.a[j] = a;
        }
        if (own_l) {
            d.b[l] = b;
            d.zs[l] = zs;
            d.u[l] = u;
            d.v[l] = (T)((double)b - (double)u);
            d.y_prev[l] = yp;
            d.ps_prev[l] = pp;
        }
    }
    if (tid == 0 && role == 0 && ok) {
        if (!c.done) c.iter = s_last;
        *d.ctl = c;
        if (!ONE) rs->base = epoch;
    }
    // the last workgroup to leave clears the counters for the next launch
    if (!ONE && tid == 0) {
        if (atomicAdd(&rs->exits, 1u) == gridDim.x - 1u) {
            for (int k = 0; k < 8; ++k) atomicExch(&rs->cnt[k * 64], 0u);
            atomicExch(&rs->win, ld_agent(&rs->abort) ? kGone : kOpen);
            atomicExch(&rs->exits, 0u);
        }
    }
}

size_t resident_lds(int m, int n, int G, size_t sz)
{
    // a zero behind each vector, 16-byte steps
    return (G > 1 ? (size_t)std::max(m, n) + 8 : (size_t)m + (size_t)n + 24) * sz;
}

}  // namespace

int resident_plan(int m, int n, int longest_link, int longest_route, size_t sz)
{
    // Register slots hold 16 entries of a lane's segment and its tail; beyond
    // that every step (four entries, or one of a four-lane segment) loads
    // indices from memory.  Few such steps cost less than the passes' launches
    // (4 lanes a segment, 11 steps: 7.4 against 11.9 us an iteration), many do
    // not (9 steps of one-lane segments: 12.9 against 12.3 us).
    auto fits = [](int rows, int longest) {
        if (4 * rows <= kRT) return longest / 4 - kSlots <= kResSteps4;
        return rows <= kRT && (longest / 4 * 4 - kSlots + 3) / 4 <= kResSteps1;
    };
    for (int G = 1; G <= kResMaxGroup; ++G)
        if (fits((n + G - 1) / G, longest_route) && fits((m + G - 1) / G, longest_link))
            return resident_lds(m, n, G, sz) <= kResLds ? G : 0;
    return 0;
}

// More than 64 KiB of LDS has to be asked for (a call small instances save).
template <typename T>
hipError_t resident_configure(const Dev<T> &d)
{
    if (resident_lds(d.m, d.n, d.resident, sizeof(T)) <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(d.resident == 1 ? (const void *)k_resident<T, true> : (const void *)k_resident<T, false>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLds);
}

template <typename T>
void launch_resident(const Dev<T> &d, int iters, bool end_check, int ce, int adapt, hipStream_t s)
{
    const int end = end_check ? iters : 0;
    const int G = d.resident;
    const size_t lds = resident_lds(d.m, d.n, G, sizeof(T));
    if (G == 1)
        hipLaunchKernelGGL((k_resident<T, true>), dim3(1), dim3(kRT), lds, s, d, d.rsync, 1, iters, end, ce, adapt);
    else
        hipLaunchKernelGGL((k_resident<T, false>), dim3(8 * G), dim3(kRT), lds, s, d, d.rsync, G, iters, end,
                           ce, adapt);
}

template hipError_t resident_configure<float>(const Dev<float> &);
template hipError_t resident_configure<double>(const Dev<double> &);
template void launch_resident<float>(const Dev<float> &, int, bool, int, int, hipStream_t);
template void launch_resident<double>(const Dev<double> &, int, bool, int, int, hipStream_t);

}  // namespace pmp
