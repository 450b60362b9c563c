// Binned message exchange: the PMP iteration for large, unstructured R.
//
// On a random link-route pattern the gathers of the CSR/CSC passes hit a
// different cache line for nearly every nonzero, and random 4-byte gathers
// from an 80 MB vector run an order of magnitude below streaming bandwidth.
// This layout instead moves one message per nonzero through HBM in
// coalesced runs:
//   R is tiled into P x Q tiles (link block p: consecutive links holding
//   about nnz / P nonzeros, at most LB links; stream block q: SB consecutive
//   streams).  mx holds x_j for every nonzero, tile by tile in p-major
//   order; mv holds v_l in q-major order; both list a tile's nonzeros in the
//   same order (grouped by link), so entry k of tile (p, q) is the same
//   nonzero in both.
//   stream workgroup q: add its mv entries into FP64 LDS sums by local stream
//     index (six), run the stream epilogue (prox, relaxation), then write
//     x_j into mx tile by tile (one wave per tile).
//   link workgroup p: add its mx entries into FP64 LDS sums by local link
//     index (lix), run the link epilogue (slack prox, average, dual update),
//     then write v_l into mv tile by tile.
// The LDS sums are FP64 atomic adds of FP32 messages.  Every addend is a
// multiple of the smallest addend's FP32 ulp u, so while a sum stays below
// 2^53 u every partial sum is exact (for example up to 32 addends spanning
// less than 2^24 in magnitude, or 1000 spanning less than 2^19): the result
// then does not depend on the order of the adds and equals the sequential
// FP64 sum of the CSR/CSC kernels.  Beyond that the order of the adds moves
// the last bits only.
#include "pmp_device.h"

#include <algorithm>

namespace pmp {

namespace {

typedef double acc_t;   // LDS sums

// Tuning knobs (defaults measured on MI355X at the large size and on a
// congested instance):
//   PMP_BIN_RUNS    merge runs of one link index before the LDS adds
//   PMP_BIN_EMIT_U  tiles a wave emits per step
//   PMP_BIN_EPI     rows per lane whose epilogue inputs are loaded before
//                   any of them is updated
#ifndef PMP_BIN_RUNS
#define PMP_BIN_RUNS true
#endif
#ifndef PMP_BIN_EMIT_U
#define PMP_BIN_EMIT_U 4
#endif
#ifndef PMP_BIN_EPI
#define PMP_BIN_EPI 2
#endif

// Workgroups are handed to the 8 XCDs of the chip in turn (block b to XCD
// b mod 8).  Renumbered so that every XCD runs one contiguous range of
// blocks, neighbouring blocks write neighbouring tiles from the same L2, where
// the partly written cache lines at tile boundaries merge before write-back.
#ifndef PMP_BIN_XCD
#define PMP_BIN_XCD 1
#endif
__device__ __forceinline__ int xcd_block(int b, int nblocks)
{
    if (!PMP_BIN_XCD) return b;
    constexpr int X = 8;
    const int x = b % X, per = nblocks / X, rem = nblocks % X;
    return x * per + min(x, rem) + b / X;
}

// Stream blocks in descending rounds: dispatch round r (blocks [R r, R r + R),
// R = Dev::SR: one block per CU, or all of them when the GPU holds them all
// at once) takes the r-th range of R stream blocks from the top, and inside a round every XCD takes a run of
// consecutive blocks (so the tiles that neighbouring workgroups write are
// neighbours, as with xcd_block).  The link pass writes the v-message tiles in
// ascending stream-block order, so the first stream blocks read the tiles
// written last, which the 256 MB memory-side cache may still hold; likewise
// the last stream blocks write the x-message tiles that every link block
// reads first.  Measured on the large workload: stream pass 0.385 -> 0.368 ms,
// link pass 0.352 -> 0.336 ms, against xcd_block numbering (rounds of two
// blocks per CU; one per CU gains another 1%).
__device__ __forceinline__ int stream_block(int b, int nblocks, int R)
{
    constexpr int X = 8;
    const int r = b / R, i = b % R;
    const int top = nblocks - R * r;
    const int lo = max(0, top - R);
    const int cnt = top - lo;
    const int x = i % X, pos = i / X, per = cnt / X, rem = cnt % X;
    return lo + x * per + min(x, rem) + pos;
}

// Add messages msg[e0..e1) into acc[idx[e]] (FP64 LDS atomics).  FP32
// messages are read four at a time (16-byte message and 8-byte index loads,
// aligned; the arrays carry 4 entries of padding), entries outside
// [e0, e1) being masked.  Messages are loaded non-temporally; indices too,
// unless TIDX.
//
// RUNS (link side): inside a tile the x messages are grouped by link, so a
// link with many streams in the tile (a congested link) makes a long run of one
// local index, and its LDS adds would all hit one address.  When some lane's
// four entries share one index, the wave merges runs first: such a lane
// contributes the sum of its four entries, a segmented sum over the lanes
// (segments = maximal runs of equal indices) totals each run, and the last
// lane of a run adds it once.  The sums are FP64 sums of FP32 messages, exact
// under the same condition as the LDS adds, so the result does not change.
//
// FX (link side, FP32): an index carrying kLongBit belongs to a long row,
// whose slot holds an int64 fixed-point sum instead (Dev::fx_shift): the
// entry adds fx_term(x, fxs) with an integer atomic, and merged runs of such
// a row add the integer sum of their terms, so the row's total does not
// depend on the order of the adds.
template <bool RUNS, bool FX, typename V, typename K>
__device__ __forceinline__ void add_quad(const V &v, const K &k, int e, int e0, int e1, bool in, acc_t *acc, double fxs)
{
    const int lane = threadIdx.x & 63;
    if constexpr (RUNS) {
        const bool uni = in && e >= e0 && e + 3 < e1 && k.x == k.y && k.y == k.z && k.z == k.w;
        if (__ballot(uni) != 0) {
            int key = uni ? (int)k.x : -1 - lane;   // others: segments of their own
            const bool lng = FX && uni && (k.x & kLongBit);
            double sum = uni && !lng ? ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w) : 0.0;
            long long isum = 0;
            if (lng)
                isum = (fx_term((double)v.x, fxs) + fx_term((double)v.y, fxs)) +
                       (fx_term((double)v.z, fxs) + fx_term((double)v.w, fxs));
            const int prev = __shfl_up(key, 1, 64);
            int head = lane == 0 || prev != key;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const double so = __shfl_up(sum, off, 64);
                long long io = 0;
                if (FX) io = __shfl_up(isum, off, 64);
                const int ho = __shfl_up(head, off, 64);
                if (lane >= off) {
                    if (!head) {
                        sum += so;
                        isum += io;
                    }
                    head |= ho;
                }
            }
            const int next = __shfl_down(key, 1, 64);
            if (uni && (lane == 63 || next != key)) {
                if (lng) atomicAdd((unsigned long long *)&acc[key & kLocalMask], (unsigned long long)isum);
                else unsafeAtomicAdd(&acc[key & kLocalMask], (acc_t)sum);
            }
            in = in && !uni;
        }
    }
    auto add1 = [&](double x, unsigned key) {
        if (FX && (key & kLongBit))
            atomicAdd((unsigned long long *)&acc[key & kLocalMask], (unsigned long long)fx_term(x, fxs));
        else
            unsafeAtomicAdd(&acc[key & kLocalMask], (acc_t)x);
    };
    if (!in) return;
    if (e >= e0 && e < e1) add1((double)v.x, k.x);
    if (e + 1 >= e0 && e + 1 < e1) add1((double)v.y, k.y);
    if (e + 2 >= e0 && e + 2 < e1) add1((double)v.z, k.z);
    if (e + 3 >= e0 && e + 3 < e1) add1((double)v.w, k.w);
}

template <typename T, bool RUNS, bool FX = false, bool TIDX = false>
__device__ __forceinline__ void accumulate(const T *__restrict__ msg,
                                           const uint16_t *__restrict__ idx, int e0, int e1,
                                           acc_t *acc, double fxs = 0.0)
{
    if constexpr (sizeof(T) == 4) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        typedef unsigned short u4 __attribute__((ext_vector_type(4)));
        const f4 *m4 = (const f4 *)msg;
        const u4 *i4 = (const u4 *)idx;
        const int lane = threadIdx.x & 63;
        // every lane of a wave takes the same trips (the run merge is
        // wave-wide); a lane past the end loads nothing
        const int b1 = quads_end(e1);
        for (int bw = (e0 >> 2) + (threadIdx.x & ~63); bw < b1; bw += kBinThreads) {
            const int b = bw + lane;
            const bool in = b < b1;
            f4 v = {0.f, 0.f, 0.f, 0.f};
            u4 k = {0, 0, 0, 0};
            if (in) {
                v = __builtin_nontemporal_load(m4 + b);
                if (TIDX) k = i4[b];
                else k = __builtin_nontemporal_load(i4 + b);
            }
            add_quad<RUNS, FX>(v, k, b << 2, e0, e1, in, acc, fxs);
        }
    } else {
        for (int e = e0 + threadIdx.x; e < e1; e += kBinThreads)
            unsafeAtomicAdd(&acc[idx[e] & kLocalMask], (acc_t)__builtin_nontemporal_load(msg + e));
    }
}

// Write the messages of one workgroup's tiles.  Wave w takes tiles
// w, w + W, w + 2W, ... (W waves).  Lane i first loads the offsets of the
// wave's i-th tile of the next 64.  The wave then writes its tiles four at a
// time: every lane loads the local indices of its entries in all four tiles
// (up to two entries per tile) before any value is looked up and stored, so
// eight index loads per lane are in flight; entries of longer tiles follow in
// rounds of four 64-entry chunks, again with the loads issued first.
//   src_off[t], src_off[t + 1]   tile t in the read layout (index array idx)
//   dst_off[t]                   tile t in the written layout
// LONG: the local indices may carry kLongBit (link side of a problem with
// fixed-point long rows), which is masked off where the LDS value is read.
// (Masked right at the load, the compiler waits for each index load before
// issuing the next: 17% slower passes on the large workload.)
template <typename T, bool LONG = false>
__device__ __forceinline__ void emit_tiles(const int *__restrict__ src_off,
                                           const int *__restrict__ dst_off, int ntiles,
                                           const uint16_t *__restrict__ idx, const acc_t *vals,
                                           T *__restrict__ out)
{
    constexpr int W = kBinThreads / 64;
    constexpr int U = PMP_BIN_EMIT_U;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int mine = ntiles > wave ? (ntiles - wave + W - 1) / W : 0;   // tiles of this wave
    for (int base = 0; base < mine; base += 64) {
        const int t = wave + (base + lane) * W;
        int src = 0, cnt = 0, dst = 0;
        if (base + lane < mine) {
            src = src_off[t];
            cnt = src_off[t + 1] - src;
            dst = dst_off[t];
        }
        const int nt = min(64, mine - base);
        for (int i0 = 0; i0 < nt; i0 += U) {
            int s_u[U], c_u[U], d_u[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = min(i0 + u, nt - 1);
                s_u[u] = __shfl(src, i, 64);
                c_u[u] = i0 + u < nt ? __shfl(cnt, i, 64) : 0;
                d_u[u] = __shfl(dst, i, 64);
            }
            int id[U][2];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int k = lane + 64 * r;
                    id[u][r] = k < c_u[u] ? (int)idx[s_u[u] + k] : -1;
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    if (id[u][r] >= 0) out[d_u[u] + lane + 64 * r] = (T)vals[LONG ? id[u][r] & kLocalMask : id[u][r]];
            // long tiles: four chunks of 64 entries per round, loads first
#pragma unroll
            for (int u = 0; u < U; ++u)
                for (int k0 = lane + 128; k0 - lane < c_u[u]; k0 += 256) {
                    int it[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int k = k0 + 64 * r;
                        it[r] = k < c_u[u] ? (int)idx[s_u[u] + k] : -1;
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (it[r] >= 0) out[d_u[u] + k0 + 64 * r] = (T)vals[LONG ? it[r] & kLocalMask : it[r]];
                }
        }
    }
}

// Two workgroups of kBinThreads share a CU (the LDS sums fit twice): ask for
// the register budget of 8 waves per SIMD.
#ifndef PMP_BIN_WAVES
#define PMP_BIN_WAVES 8
#endif
#if PMP_BIN_WAVES > 0
#define PMP_BIN_KERNEL \
    __global__ __launch_bounds__(kBinThreads) __attribute__((amdgpu_waves_per_eu(PMP_BIN_WAVES)))
#else
#define PMP_BIN_KERNEL __global__ __launch_bounds__(kBinThreads)
#endif

template <typename T, int MODE, bool TIDX>
PMP_BIN_KERNEL void k_bin_stream(Dev<T> d)
{
    if (d.ctl->done) return;
    extern __shared__ acc_t S[];
    __shared__ double sred[kBinThreads / 64];
    const int q = stream_block(blockIdx.x, gridDim.x, d.SR);
    const int j0 = d.sbs[q];
    const int ns = d.sbs[q + 1] - j0;
    for (int i = threadIdx.x; i < ns; i += kBinThreads) S[i] = 0.0;
    __syncthreads();
    // TIDX (chosen at launch when the stream blocks take several dispatch
    // rounds): the local stream indices are loaded as ordinary (temporal)
    // data, since the emission below reads them again; on the large workload
    // that read then hits more often (stream pass 0.367 -> 0.359 ms).  With
    // every stream block resident at once (the paper shape) the same hint
    // costs 6%, and on the link side it slows the link pass: there the
    // indices stay non-temporal.
    accumulate<T, false, false, TIDX>(d.mv, d.six, d.ov[(long long)q * d.P], d.ov[(long long)(q + 1) * d.P], S);
    __syncthreads();
    // Of the two workgroups of a CU the one nearer its end goes first, so that
    // the next block's loads start early: large workload, an iteration 695 ->
    // 691 us (a higher priority for the rows alone: 700; for the adds: 693).
    __builtin_amdgcn_s_setprio(1);
    const double irho = d.ctl->irho;
    double part = 0.0;
    constexpr int G = PMP_BIN_EPI;
    // The per-stream vectors (route length, weight, a) go through
    // non-temporally: the next read of a comes a whole iteration later, far
    // beyond what the memory-side cache keeps, and leaving them out of it
    // keeps more of the message tiles and indices there (large workload:
    // stream pass 0.357 -> 0.348 ms; the link side's vectors, tried the same
    // way, slowed the link pass by 3%).
    for (int i0 = threadIdx.x; i0 < ns; i0 += G * kBinThreads) {
        int L[G];
        double a[G], w[G], xo[G];
        bool a2[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = i0 + g * kBinThreads;
            if (i < ns) {
                const int j = j0 + i;
                L[g] = d.rlen ? (int)__builtin_nontemporal_load(d.rlen + j)
                              : d.col_ptr[j + 1] - d.col_ptr[j];
                a[g] = (double)__builtin_nontemporal_load(d.a + j);
                w[g] = (double)__builtin_nontemporal_load(d.wsig + j);
                a2[g] = is_alpha2(d, j);
                xo[g] = MODE == kCheck ? (double)d.x[j] : 0.0;
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = i0 + g * kBinThreads;
            if (i < ns) {
                const int j = j0 + i;
                T xt, at;
                stream_core<T>(a[g], w[g], L[g], (double)S[i], irho, d.lo, d.hi, d.alpha, a2[g], xt, at);
                const double xn = (double)xt;
                if (MODE == kCheck) {          // dual residual: sum_j L_j (dx_j)^2
                    const double dx = xn - xo[g];
                    part += screen((double)L[g] * dx * dx, (double)at);
                }
                if (MODE != kPlain) d.x[j] = xt;   // otherwise x travels only in the messages
                __builtin_nontemporal_store(at, d.a + j);
                S[i] = (acc_t)xn;
            }
        }
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(2);
    // tile (q, p) of the v messages and tile (p, q) of the x messages list the
    // same nonzeros in the same order
    emit_tiles<T>(d.ov + (long long)q * d.P, d.oxq + (long long)q * d.P, d.P, d.six, S, d.mx);
    if (MODE == kCheck) {
        part = block_sum_n<kBinThreads>(part, sred);
        if (threadIdx.x == 0) d.spart[q] = part;
    }
}

template <typename T, int MODE>
PMP_BIN_KERNEL void k_bin_link(Dev<T> d)
{
    if (d.ctl->done) return;
    extern __shared__ acc_t Y[];
    __shared__ double sred[kBinThreads / 64];
    const int p = xcd_block(blockIdx.x, gridDim.x);
    const int l0 = d.lbs[p];
    const int nl = d.lbs[p + 1] - l0;
    for (int i = threadIdx.x; i < nl; i += kBinThreads) Y[i] = 0.0;
    __syncthreads();
    const int e0 = d.ox[(long long)p * d.Q], e1 = d.ox[(long long)(p + 1) * d.Q];
    if (sizeof(T) == 4 && d.fx_shift) accumulate<T, PMP_BIN_RUNS, true>(d.mx, d.lix, e0, e1, Y, d.fx_scale);
    else accumulate<T, PMP_BIN_RUNS>(d.mx, d.lix, e0, e1, Y);
    __syncthreads();
    __builtin_amdgcn_s_setprio(1);
    double r2 = 0.0, s2 = 0.0;
    constexpr int G = MODE == kCheck ? 1 : PMP_BIN_EPI;   // a check carries more inputs
    for (int i0 = threadIdx.x; i0 < nl; i0 += G * kBinThreads) {
        int deg[G];
        LinkIn in[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = i0 + g * kBinThreads;
            if (i < nl) {
                const int l = l0 + i;
                deg[g] = d.dlen ? (int)d.dlen[l] : d.row_ptr[l + 1] - d.row_ptr[l];
                in[g] = link_load<T, MODE>(d, l);
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = i0 + g * kBinThreads;
            if (i < nl) {
                const int l = l0 + i;
                // v goes out in the messages; a check also stores it
                double y = (double)Y[i];
                if (d.fx_shift && deg[g] > kCap) y = (double)__double_as_longlong(Y[i]) * d.fx_inv;
                Y[i] = (acc_t)(MODE == kCheck
                                   ? link_update_in<T, MODE, true>(d, l, deg[g], y, in[g], r2, s2)
                                   : link_update_in<T, MODE, false>(d, l, deg[g], y, in[g], r2, s2));
            }
        }
    }
    if (MODE == kCheck) {
        r2 = block_sum_n<kBinThreads>(r2, sred);
        s2 = block_sum_n<kBinThreads>(s2, sred);
        if (threadIdx.x == 0) {
            d.lpart[2 * p] = r2;
            d.lpart[2 * p + 1] = s2;
        }
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(2);
    if (d.fx_shift) emit_tiles<T, true>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, d.mv);
    else emit_tiles<T>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, d.mv);
}

// Passes of workgroups that each have a CU to themselves (at most one block
// per CU on this side).  The memory system bounds them, but in phases: every
// workgroup loads messages, adds, loads rows and writes messages at the same
// time, and the kernels above also wait for a round of loads per four entries
// of a lane, for each row's stores, and for the indices a second time.  Here a
// lane issues its first kOneQuads groups of four entries at once (16 waves may
// use 128 registers each), the tiles' offsets with them, and the rows' vectors
// before the barrier that ends the LDS adds; the local indices stay in LDS for
// the emission.  One iteration, before -> after: 1e6 links x 5e5 streams,
// nnz = 5e6: 43.5 -> 37.8 us; 1e6 x 8e5, 8e6: 60.3 -> 47.7; 3e5 x 3e5, 3e6: 30.7
// -> 25.4; 4e5 x 4e5, 4e6: 29.2; in FP64, 5e6: 65 -> 49.4.  Within a pass at 5e6:
// (device clocks, mean over the blocks): 4.8 us until the messages are there, 4.1
// until every wave has added its own, 1.6 rows, 4.1 messages out, 3.7 to the next
// kernel's start.  Eight groups in place of five: 38.9 us; the rows'
// vectors issued with the messages: 40.6.
constexpr int kOneQuads = 5, kOneStreams = 2, kOneLinks = 4;   // groups of entries, rows a lane
constexpr size_t kOneLds = 158 * 1024;                          // (160 KiB, less the block sums)
#define PMP_BIN_ONE_KERNEL __global__ __launch_bounds__(kBinThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))

// The offsets of a wave's tiles, lane i: tile wave + i W (ntiles <= 64 W).
struct OneTiles {
    int src, end, dst, mine;
    __device__ __forceinline__ void load(const int *src_off, const int *dst_off, int ntiles)
    {
        constexpr int W = kBinThreads / 64;
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, t = wave + lane * W;
        mine = ntiles > wave ? (ntiles - wave + W - 1) / W : 0;
        const int tc = min(t, ntiles - 1);
        src = src_off[tc];
        end = src_off[tc + 1];
        dst = dst_off[tc];
    }
};

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int kRawBuffer = 0x00027000;      // resource word 3: 32-bit data, bounds in bytes

// Adds the entries [e0, e1) as accumulate does.  The indices go to cache,
// from entry e0 & ~3 on, where cache is given.
template <typename T, bool RUNS, bool FX>
struct OneEntries {
    static constexpr int K = sizeof(T) == 4 ? kOneQuads : 4;
    typedef T v4 __attribute__((ext_vector_type(4)));
    typedef unsigned short u4 __attribute__((ext_vector_type(4)));
    v4 v[K];
    u4 k[K];
    // (buffer loads, whose lanes past the end read nothing: with a branch
    // around a load the compiler waits for all of them before it uses the first)
    __device__ __forceinline__ void load(const T *msg, const uint16_t *idx, int e0, int e1)
    {
        constexpr int kNt = 2;                             // non-temporal
        const int q0 = e0 >> 2, nq = min(quads_end(e1) - q0, K * kBinThreads);
        auto m = __builtin_amdgcn_make_buffer_rsrc((void *)((const v4 *)msg + q0), 0, nq * (int)sizeof(v4), kRawBuffer);
        auto x = __builtin_amdgcn_make_buffer_rsrc((void *)((const u4 *)idx + q0), 0, nq * (int)sizeof(u4), kRawBuffer);
#pragma unroll
        for (int g = 0; g < K; ++g) {
            const int b = threadIdx.x + g * kBinThreads;
            if constexpr (sizeof(T) == 4) {
                v[g] = __builtin_bit_cast(v4, __builtin_amdgcn_raw_buffer_load_b128(m, b * 16, 0, kNt));
            } else {
                struct { u32x4 lo, hi; } t = {__builtin_amdgcn_raw_buffer_load_b128(m, b * 32, 0, kNt),
                                              __builtin_amdgcn_raw_buffer_load_b128(m, b * 32 + 16, 0, kNt)};
                v[g] = __builtin_bit_cast(v4, t);
            }
            k[g] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b64(x, b * 8, 0, kNt));
        }
    }
    __device__ __forceinline__ void add(const T *msg, const uint16_t *idx, int e0, int e1, acc_t *acc, u4 *cache,
                                        double fxs)
    {
        const int lane = threadIdx.x & 63, q0 = e0 >> 2, b1 = quads_end(e1);
        int w = q0 + (threadIdx.x & ~63);
#pragma unroll
        for (int g = 0; g < K; ++g, w += kBinThreads)
            if (w < b1) {                                  // the whole wave
                const int b = w + lane;
                if (cache && b < b1) cache[b - q0] = k[g];
                add_quad<RUNS, FX>(v[g], k[g], b << 2, e0, e1, b < b1, acc, fxs);
            }
        for (; w < b1; w += kBinThreads) {
            const int b = w + lane, bc = min(b, b1 - 1);
            const v4 x = __builtin_nontemporal_load((const v4 *)msg + bc);
            const u4 y = __builtin_nontemporal_load((const u4 *)idx + bc);
            if (cache && b < b1) cache[b - q0] = y;
            add_quad<RUNS, FX>(x, y, b << 2, e0, e1, b < b1, acc, fxs);
        }
    }
};

// emit_tiles with the offsets in registers and the indices read through at(e).
template <typename T, bool LONG, bool NT, typename At>
__device__ __forceinline__ void one_emit(const OneTiles &o, const acc_t *vals, T *__restrict__ out, At at)
{
    constexpr int U = PMP_BIN_EMIT_U;
    auto put = [&](int at, int i) {
        const T x = (T)vals[LONG ? i & kLocalMask : i];
        if (NT) __builtin_nontemporal_store(x, out + at);
        else out[at] = x;
    };
    const int lane = threadIdx.x & 63;
    for (int i0 = 0; i0 < o.mine; i0 += U) {
        int s_u[U], c_u[U], d_u[U], id[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u, o.mine - 1);
            s_u[u] = __builtin_amdgcn_readlane(o.src, i);
            c_u[u] = i0 + u < o.mine ? __builtin_amdgcn_readlane(o.end, i) - s_u[u] : 0;
            d_u[u] = __builtin_amdgcn_readlane(o.dst, i);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int k = lane + 64 * r;
                id[u][r] = k < c_u[u] ? (int)at(s_u[u] + k) : -1;
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 2; ++r)
                if (id[u][r] >= 0) put(d_u[u] + lane + 64 * r, id[u][r]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            for (int k = lane + 128; k < c_u[u]; k += 64) put(d_u[u] + k, (int)at(s_u[u] + k));
    }
}

// All loads issued so far.  Without it the compiler waits at each row's first
// use and, not knowing whether the row before it stored, for that row's stores
// too: loads and stores share a counter.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt(0) alone

// The vectors of rows r0 + threadIdx.x + g kBinThreads below r1 (or of the
// last row), in registers.
template <typename T, int MODE, int G>
struct OneStreams {
    int L0[G], L1[G];
    T a[G], w[G], xo[G];
    uint8_t ut[G];
    __device__ __forceinline__ void load(const Dev<T> &d, int r0, int r1)
    {
        auto row = [&](int g) { return min(r0 + g * kBinThreads + (int)threadIdx.x, r1 - 1); };
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int j = row(g);
            a[g] = __builtin_nontemporal_load(d.a + j);
            w[g] = __builtin_nontemporal_load(d.wsig + j);
            if (MODE == kCheck) xo[g] = d.x[j];
        }
        if (d.rlen) {
#pragma unroll
            for (int g = 0; g < G; ++g) L0[g] = 0, L1[g] = __builtin_nontemporal_load(d.rlen + row(g));
        } else {
#pragma unroll
            for (int g = 0; g < G; ++g) L0[g] = d.col_ptr[row(g)], L1[g] = d.col_ptr[row(g) + 1];
        }
        if (d.util) {
#pragma unroll
            for (int g = 0; g < G; ++g) ut[g] = d.util[row(g)];
        }
    }
};
template <typename T, int MODE, int G>
struct OneLinks {
    int g0[G], g1[G];
    T c[G], u[G], b[G], zs[G];
    double yp[G], pp[G];
    __device__ __forceinline__ void load(const Dev<T> &d, int r0, int r1)
    {
        auto row = [&](int g) { return min(r0 + g * kBinThreads + (int)threadIdx.x, r1 - 1); };
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int l = row(g);
            c[g] = d.c[l];
            u[g] = d.u[l];
            b[g] = d.b[l];
            zs[g] = d.zs[l];
            if (MODE == kCheck) {
                yp[g] = d.y_prev[l];
                pp[g] = d.ps_prev[l];
            }
        }
        if (d.dlen) {
#pragma unroll
            for (int g = 0; g < G; ++g) g0[g] = 0, g1[g] = d.dlen[row(g)];
        } else {
#pragma unroll
            for (int g = 0; g < G; ++g) g0[g] = d.row_ptr[row(g)], g1[g] = d.row_ptr[row(g) + 1];
        }
    }
};

template <typename T, int MODE>
PMP_BIN_ONE_KERNEL void k_bin_stream_one(Dev<T> d, int cap, int nt)
{
    typedef unsigned short u4 __attribute__((ext_vector_type(4)));
    extern __shared__ acc_t S[];
    __shared__ double sred[kBinThreads / 64];
    const int q = stream_block(blockIdx.x, gridDim.x, d.SR);
    const int *ov = d.ov + (long long)q * d.P;
    const int j0 = d.sbs[q], j1 = d.sbs[q + 1], e0 = ov[0], e1 = ov[d.P];
    const double irho = d.ctl->irho;
    if (d.ctl->done) return;
    if (j0 >= j1) {
        if (MODE == kCheck && threadIdx.x == 0) d.spart[q] = 0.0;
        return;
    }
    uint16_t *kept = (uint16_t *)(S + d.SB);
    const bool fits = quads_end(e1) - (e0 >> 2) <= cap / 4;
    constexpr int G = kOneStreams;
    OneEntries<T, false, false> en;
    OneStreams<T, MODE, G> rows;
    OneTiles tl;
    en.load(d.mv, d.six, e0, e1);
    tl.load(ov, d.oxq + (long long)q * d.P, d.P);
    for (int i = threadIdx.x; i < j1 - j0; i += kBinThreads) S[i] = 0.0;
    __syncthreads();
    en.add(d.mv, d.six, e0, e1, S, fits ? (u4 *)kept : nullptr, 0.0);
    rows.load(d, j0, j1);
    __syncthreads();
    double part = 0.0;
    for (int r0 = j0; r0 < j1; r0 += G * kBinThreads) {
        if (r0 > j0) rows.load(d, r0, j1);
        wait_loads();
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int j = r0 + g * kBinThreads + (int)threadIdx.x;
            if (j < j1) {
                const int L = rows.L1[g] - rows.L0[g];
                T xt, at;
                stream_core<T>((double)rows.a[g], (double)rows.w[g], L, (double)S[j - j0], irho, d.lo, d.hi, d.alpha,
                               d.util && rows.ut[g] == PMP_UTIL_ALPHA2, xt, at);
                const double xn = (double)xt;
                if (MODE == kCheck) {          // dual residual: sum_j L_j (dx_j)^2
                    const double dx = xn - (double)rows.xo[g];
                    part += screen((double)L * dx * dx, (double)at);
                }
                if (MODE != kPlain) d.x[j] = xt;
                __builtin_nontemporal_store(at, d.a + j);
                S[j - j0] = (acc_t)xn;
            }
        }
    }
    __syncthreads();
    auto at = [&](int e) { return kept[e - (e0 & ~3)]; };
    if (!fits) one_emit<T, false, false>(tl, S, d.mx, [&](int e) { return d.six[e]; });
    else if (nt) one_emit<T, false, true>(tl, S, d.mx, at);
    else one_emit<T, false, false>(tl, S, d.mx, at);
    if (MODE == kCheck) {
        part = block_sum_n<kBinThreads>(part, sred);
        if (threadIdx.x == 0) d.spart[q] = part;
    }
}

template <typename T, int MODE, bool FX>
PMP_BIN_ONE_KERNEL void k_bin_link_one(Dev<T> d, int cap, int nt)
{
    typedef unsigned short u4 __attribute__((ext_vector_type(4)));
    extern __shared__ acc_t Y[];
    __shared__ double sred[kBinThreads / 64];
    const int p = xcd_block(blockIdx.x, gridDim.x);
    const int *ox = d.ox + (long long)p * d.Q;
    const int l0 = d.lbs[p], l1 = d.lbs[p + 1], e0 = ox[0], e1 = ox[d.Q];
    if (d.ctl->done) return;
    if (l0 >= l1) {
        if (MODE == kCheck && threadIdx.x == 0) d.lpart[2 * p] = d.lpart[2 * p + 1] = 0.0;
        return;
    }
    uint16_t *kept = (uint16_t *)(Y + d.LB);
    const bool fits = quads_end(e1) - (e0 >> 2) <= cap / 4;
    constexpr int G = MODE == kCheck || sizeof(T) == 8 ? 2 : kOneLinks;   // a check carries more inputs
    OneEntries<T, sizeof(T) == 4 && PMP_BIN_RUNS, FX> en;
    OneLinks<T, MODE, G> rows;
    OneTiles tl;
    en.load(d.mx, d.lix, e0, e1);
    tl.load(ox, d.ovp + (long long)p * d.Q, d.Q);
    for (int i = threadIdx.x; i < l1 - l0; i += kBinThreads) Y[i] = 0.0;
    __syncthreads();
    en.add(d.mx, d.lix, e0, e1, Y, fits ? (u4 *)kept : nullptr, d.fx_scale);
    rows.load(d, l0, l1);
    __syncthreads();
    double r2 = 0.0, s2 = 0.0;
    for (int r0 = l0; r0 < l1; r0 += G * kBinThreads) {
        if (r0 > l0) rows.load(d, r0, l1);
        wait_loads();
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int l = r0 + g * kBinThreads + (int)threadIdx.x;
            if (l < l1) {
                const int deg = rows.g1[g] - rows.g0[g];
                const LinkIn in{(double)rows.c[g], (double)rows.u[g], (double)rows.b[g], (double)rows.zs[g],
                                MODE == kCheck ? rows.yp[g] : 0.0, MODE == kCheck ? rows.pp[g] : 0.0};
                double y = (double)Y[l - l0];
                if (FX && deg > kCap) y = (double)__double_as_longlong(Y[l - l0]) * d.fx_inv;
                // v goes out in the messages; a check also stores it
                Y[l - l0] = (acc_t)link_update_in<T, MODE, MODE == kCheck>(d, l, deg, y, in, r2, s2);
            }
        }
    }
    if (MODE == kCheck) {
        r2 = block_sum_n<kBinThreads>(r2, sred);
        s2 = block_sum_n<kBinThreads>(s2, sred);
        if (threadIdx.x == 0) {
            d.lpart[2 * p] = r2;
            d.lpart[2 * p + 1] = s2;
        }
    }
    __syncthreads();
    auto at = [&](int e) { return kept[e - (e0 & ~3)]; };
    if (!fits) one_emit<T, FX, false>(tl, Y, d.mv, [&](int e) { return d.lix[e]; });
    else if (nt) one_emit<T, FX, true>(tl, Y, d.mv, at);
    else one_emit<T, FX, false>(tl, Y, d.mv, at);
}

// After a check (apply = 1): apply a pending u rescale (eq. (18)), refresh
// v = b - u and rewrite the link messages; without a pending rescale the
// check's link pass has written them already and nothing is done.  With
// apply = 0 the messages are rewritten from v.
template <typename T>
PMP_BIN_KERNEL void k_bin_emit(Dev<T> d, int apply)
{
    if (apply && d.ctl->ratio == 1.0) return;
    extern __shared__ acc_t Y[];
    const int p = xcd_block(blockIdx.x, gridDim.x);
    const int l0 = d.lbs[p];
    const int nl = d.lbs[p + 1] - l0;
    const double ratio = apply ? d.ctl->ratio : 1.0;
    for (int i = threadIdx.x; i < nl; i += kBinThreads) {
        const int l = l0 + i;
        T vt = d.v[l];
        if (ratio != 1.0) {
            T ut = d.u[l];
            vt = link_rescale<T>(d.b[l], ut, ratio);
            d.u[l] = ut;
            d.v[l] = vt;
        }
        Y[i] = (acc_t)vt;
    }
    __syncthreads();
    if (d.fx_shift) emit_tiles<T, true>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, d.mv);
    else emit_tiles<T>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, d.mv);
}

// Reverse mode in the binned layout: the two sums of a reversed iteration,
// R^T ybar (per stream) and R Sbar (per link), move as messages in the
// problem's precision through the same tiles as the forward messages (ybar in
// the v layout, Sbar in the x layout) and are summed in FP64 as there.  The
// FP64 values of ybar and Sbar are rounded to the message precision, so in
// FP32 these sums match the gather layout's FP64 gathers to FP32 rounding
// (a gradient of the adjoint workload: 0.0857 s, against 0.0928 s with FP64
// messages).
template <typename T>
PMP_BIN_KERNEL void k_bin_adj_stream(Dev<T> d, AdjDev a, const T *xt, int last,
                                     const T *my, T *ms)
{
    extern __shared__ acc_t S[];
    const int q = xcd_block(blockIdx.x, gridDim.x);
    const int j0 = d.sbs[q];
    const int ns = d.sbs[q + 1] - j0;
    for (int i = threadIdx.x; i < ns; i += kBinThreads) S[i] = 0.0;
    __syncthreads();
    accumulate<T, false>(my, d.six, d.ov[(long long)q * d.P], d.ov[(long long)(q + 1) * d.P], S);
    __syncthreads();
    const double rho = d.ctl->rho;
    for (int i = threadIdx.x; i < ns; i += kBinThreads) {
        const int j = j0 + i;
        const int L = d.rlen ? (int)d.rlen[j] : d.col_ptr[j + 1] - d.col_ptr[j];
        AdjStreamIn<T> in;
        in.load(d, a, xt, j, last);
        S[i] = adj_stream_step<T>(d, a, in, j, L, (double)S[i], rho);
    }
    __syncthreads();
    emit_tiles<T>(d.ov + (long long)q * d.P, d.oxq + (long long)q * d.P, d.P, d.six, S, ms);
}

// R Sbar per link, then (mu_prev given) the link step of the iteration
// before, whose ybar goes out as messages for the next stream step.
template <typename T>
PMP_BIN_KERNEL void k_bin_adj_link(Dev<T> d, AdjDev a, const uint8_t *mu_prev, const T *ms,
                                   T *my)
{
    extern __shared__ acc_t Y[];
    const int p = xcd_block(blockIdx.x, gridDim.x);
    const int l0 = d.lbs[p];
    const int nl = d.lbs[p + 1] - l0;
    for (int i = threadIdx.x; i < nl; i += kBinThreads) Y[i] = 0.0;
    __syncthreads();
    accumulate<T, false>(ms, d.lix, d.ox[(long long)p * d.Q], d.ox[(long long)(p + 1) * d.Q], Y);
    __syncthreads();
    for (int i = threadIdx.x; i < nl; i += kBinThreads) {
        const int l = l0 + i;
        const double vbar = (double)Y[i];
        AdjLinkIn in;
        in.load(a, l, mu_prev);
        in.B += vbar;
        in.U -= vbar;
        if (mu_prev) {
            const int deg = d.dlen ? (int)d.dlen[l] : d.row_ptr[l + 1] - d.row_ptr[l];
            Y[i] = adj_link_step(a, l, deg, d.alpha, in);
        } else {
            a.B[l] = in.B;
            a.U[l] = in.U;
        }
    }
    if (!mu_prev) return;   // ybar unchanged: its messages still hold
    __syncthreads();
    if (d.fx_shift) emit_tiles<T, true>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, my);
    else emit_tiles<T>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, my);
}

// ybar messages from a.ybar (after it changed outside k_bin_adj_link).
template <typename T>
PMP_BIN_KERNEL void k_bin_adj_emit(Dev<T> d, AdjDev a, T *my)
{
    extern __shared__ acc_t Y[];
    const int p = xcd_block(blockIdx.x, gridDim.x);
    const int l0 = d.lbs[p];
    const int nl = d.lbs[p + 1] - l0;
    for (int i = threadIdx.x; i < nl; i += kBinThreads) Y[i] = a.ybar[l0 + i];
    __syncthreads();
    if (d.fx_shift) emit_tiles<T, true>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, my);
    else emit_tiles<T>(d.ox + (long long)p * d.Q, d.ovp + (long long)p * d.Q, d.Q, d.lix, Y, my);
}

}  // namespace

void binned_configure()
{
    const int bytes = kBinMaxBlock * (int)sizeof(acc_t);
#define PMP_BIN_ATTR(K) (void)hipFuncSetAttribute((const void *)(K), hipFuncAttributeMaxDynamicSharedMemorySize, bytes)
    PMP_BIN_ATTR((k_bin_stream<float, kPlain, false>));
    PMP_BIN_ATTR((k_bin_stream<float, kSave, false>));
    PMP_BIN_ATTR((k_bin_stream<float, kCheck, false>));
    PMP_BIN_ATTR((k_bin_stream<double, kPlain, false>));
    PMP_BIN_ATTR((k_bin_stream<double, kSave, false>));
    PMP_BIN_ATTR((k_bin_stream<double, kCheck, false>));
    PMP_BIN_ATTR((k_bin_stream<float, kPlain, true>));
    PMP_BIN_ATTR((k_bin_stream<float, kSave, true>));
    PMP_BIN_ATTR((k_bin_stream<float, kCheck, true>));
    PMP_BIN_ATTR((k_bin_stream<double, kPlain, true>));
    PMP_BIN_ATTR((k_bin_stream<double, kSave, true>));
    PMP_BIN_ATTR((k_bin_stream<double, kCheck, true>));
    PMP_BIN_ATTR((k_bin_link<float, kPlain>));
    PMP_BIN_ATTR((k_bin_link<float, kSave>));
    PMP_BIN_ATTR((k_bin_link<float, kCheck>));
    PMP_BIN_ATTR((k_bin_link<double, kPlain>));
    PMP_BIN_ATTR((k_bin_link<double, kSave>));
    PMP_BIN_ATTR((k_bin_link<double, kCheck>));
    PMP_BIN_ATTR((k_bin_emit<float>));
    PMP_BIN_ATTR((k_bin_emit<double>));
    PMP_BIN_ATTR((k_bin_adj_stream<float>));
    PMP_BIN_ATTR((k_bin_adj_stream<double>));
    PMP_BIN_ATTR((k_bin_adj_link<float>));
    PMP_BIN_ATTR((k_bin_adj_link<double>));
    PMP_BIN_ATTR((k_bin_adj_emit<float>));
    PMP_BIN_ATTR((k_bin_adj_emit<double>));
    auto one = [&](const void *f) { (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOneLds); };
#define PMP_BIN_ONE_ATTR(T, MODE)                        \
    one((const void *)(k_bin_stream_one<T, MODE>));      \
    one((const void *)(k_bin_link_one<T, MODE, false>)); \
    one((const void *)(k_bin_link_one<T, MODE, sizeof(T) == 4>));
    PMP_BIN_ONE_ATTR(float, kPlain)
    PMP_BIN_ONE_ATTR(float, kSave)
    PMP_BIN_ONE_ATTR(float, kCheck)
    PMP_BIN_ONE_ATTR(double, kPlain)
    PMP_BIN_ONE_ATTR(double, kSave)
    PMP_BIN_ONE_ATTR(double, kCheck)
#undef PMP_BIN_ONE_ATTR
#undef PMP_BIN_ATTR
}

// A side whose blocks all have a CU of their own takes the passes above, but not
// a link side whose fullest block (long rows) has more entries than are loaded at
// once and one and a half times the mean: the rest come a round at a time.
// 1e5 links x 5e5 streams, 30 links on 50,000 streams each, nnz = 6.5e6 (fullest
// 2.5 times the mean): 95.7 us an iteration against 86.2, in FP64 130 against 119;
// 1e6 x 5e5, 500 links on 5,000 each, 7.5e6 (1.2 times): 60.0 against 66.5.  The
// indices of cap entries stay in LDS (a quarter more than the mean, in what one
// workgroup may have).  With several blocks a CU, two resident workgroups
// overlap their phases instead: 2e7 nonzeros 106 us against 111, 4e7 210
// against 254.  nt: the messages go out non-temporally while the tiles hold
// fewer than 64 entries: an iteration at nnz = 2.8e6 24.8 us against 31.1, at
// 4e6 29.2 against 33.4, at 5e6 37.9 against 37.8, at 8e6 53.5 against 47.7.
template <typename T>
bool one_block(const Dev<T> &d, int blocks, int other, int rows, int &cap, int &nt, size_t &lds)
{
    if (blocks > d.CUs || other > kBinThreads) return false;
    const size_t sums = (size_t)rows * sizeof(acc_t);
    const long long mean = d.nnz / std::max(1, blocks);
    cap = (int)std::min<long long>((mean + mean / 4 + 8) & ~3LL, ((long long)(kOneLds - sums) / 2) & ~3LL);
    lds = sums + (size_t)cap * 2;
    nt = d.nnz < 64LL * blocks * other;
    return true;
}

template <typename T>
void launch_bin_stream(const Dev<T> &d, int mode, hipStream_t s)
{
    size_t lds = (size_t)d.SB * sizeof(acc_t);
    const dim3 g(d.Q), b(kBinThreads);
    int cap, nt;
    if (one_block(d, d.Q, d.P, d.SB, cap, nt, lds)) {
        if (mode == kPlain) hipLaunchKernelGGL((k_bin_stream_one<T, kPlain>), g, b, lds, s, d, cap, nt);
        else if (mode == kSave) hipLaunchKernelGGL((k_bin_stream_one<T, kSave>), g, b, lds, s, d, cap, nt);
        else hipLaunchKernelGGL((k_bin_stream_one<T, kCheck>), g, b, lds, s, d, cap, nt);
        return;
    }
    const bool rounds = d.SR < d.Q;   // several dispatch rounds: temporal index loads
    switch (mode) {
    case kPlain:
        if (rounds) hipLaunchKernelGGL((k_bin_stream<T, kPlain, true>), g, b, lds, s, d);
        else hipLaunchKernelGGL((k_bin_stream<T, kPlain, false>), g, b, lds, s, d);
        break;
    case kSave:
        if (rounds) hipLaunchKernelGGL((k_bin_stream<T, kSave, true>), g, b, lds, s, d);
        else hipLaunchKernelGGL((k_bin_stream<T, kSave, false>), g, b, lds, s, d);
        break;
    default:
        if (rounds) hipLaunchKernelGGL((k_bin_stream<T, kCheck, true>), g, b, lds, s, d);
        else hipLaunchKernelGGL((k_bin_stream<T, kCheck, false>), g, b, lds, s, d);
        break;
    }
}

template <typename T, bool FX>
void launch_bin_link_one(const Dev<T> &d, int mode, int cap, int nt, size_t lds, hipStream_t s)
{
    const dim3 g(d.P), b(kBinThreads);
    if (mode == kPlain) hipLaunchKernelGGL((k_bin_link_one<T, kPlain, FX>), g, b, lds, s, d, cap, nt);
    else if (mode == kSave) hipLaunchKernelGGL((k_bin_link_one<T, kSave, FX>), g, b, lds, s, d, cap, nt);
    else hipLaunchKernelGGL((k_bin_link_one<T, kCheck, FX>), g, b, lds, s, d, cap, nt);
}

template <typename T>
void launch_bin_link(const Dev<T> &d, int mode, hipStream_t s)
{
    size_t lds = (size_t)d.LB * sizeof(acc_t);
    int cap, nt;
    const bool even = d.fullest <= 4 * kOneQuads * kBinThreads || 2 * (long long)d.fullest * d.P <= 3 * d.nnz;
    if (even && one_block(d, d.P, d.Q, d.LB, cap, nt, lds)) {
        if (sizeof(T) == 4 && d.fx_shift) launch_bin_link_one<T, sizeof(T) == 4>(d, mode, cap, nt, lds, s);
        else launch_bin_link_one<T, false>(d, mode, cap, nt, lds, s);
        return;
    }
    switch (mode) {
    case kPlain:
        hipLaunchKernelGGL((k_bin_link<T, kPlain>), dim3(d.P), dim3(kBinThreads), lds, s, d);
        break;
    case kSave:
        hipLaunchKernelGGL((k_bin_link<T, kSave>), dim3(d.P), dim3(kBinThreads), lds, s, d);
        break;
    default:
        hipLaunchKernelGGL((k_bin_link<T, kCheck>), dim3(d.P), dim3(kBinThreads), lds, s, d);
        break;
    }
}

template <typename T>
void launch_bin_emit(const Dev<T> &d, int apply, hipStream_t s)
{
    hipLaunchKernelGGL((k_bin_emit<T>), dim3(d.P), dim3(kBinThreads), (size_t)d.LB * sizeof(acc_t),
                       s, d, apply);
}

template <typename T>
void launch_bin_adj_stream(const Dev<T> &d, const AdjDev &a, const T *xt, int last,
                           const T *my, T *ms, hipStream_t s)
{
    hipLaunchKernelGGL((k_bin_adj_stream<T>), dim3(d.Q), dim3(kBinThreads),
                       ((size_t)d.SB) * sizeof(acc_t), s, d, a, xt, last, my, ms);
}

template <typename T>
void launch_bin_adj_link(const Dev<T> &d, const AdjDev &a, const uint8_t *mu_prev,
                         const T *ms, T *my, hipStream_t s)
{
    hipLaunchKernelGGL((k_bin_adj_link<T>), dim3(d.P), dim3(kBinThreads),
                       ((size_t)d.LB) * sizeof(acc_t), s, d, a, mu_prev, ms, my);
}

template <typename T>
void launch_bin_adj_emit(const Dev<T> &d, const AdjDev &a, T *my, hipStream_t s)
{
    hipLaunchKernelGGL((k_bin_adj_emit<T>), dim3(d.P), dim3(kBinThreads),
                       ((size_t)d.LB) * sizeof(acc_t), s, d, a, my);
}

template void launch_bin_stream<float>(const Dev<float> &, int, hipStream_t);
template void launch_bin_stream<double>(const Dev<double> &, int, hipStream_t);
template void launch_bin_link<float>(const Dev<float> &, int, hipStream_t);
template void launch_bin_link<double>(const Dev<double> &, int, hipStream_t);
template void launch_bin_emit<float>(const Dev<float> &, int, hipStream_t);
template void launch_bin_emit<double>(const Dev<double> &, int, hipStream_t);
template void launch_bin_adj_stream<float>(const Dev<float> &, const AdjDev &, const float *, int,
                                           const float *, float *, hipStream_t);
template void launch_bin_adj_stream<double>(const Dev<double> &, const AdjDev &, const double *,
                                            int, const double *, double *, hipStream_t);
template void launch_bin_adj_link<float>(const Dev<float> &, const AdjDev &, const uint8_t *,
                                         const float *, float *, hipStream_t);
template void launch_bin_adj_link<double>(const Dev<double> &, const AdjDev &, const uint8_t *,
                                          const double *, double *, hipStream_t);
template void launch_bin_adj_emit<float>(const Dev<float> &, const AdjDev &, float *, hipStream_t);
template void launch_bin_adj_emit<double>(const Dev<double> &, const AdjDev &, double *, hipStream_t);

}  // namespace pmp
