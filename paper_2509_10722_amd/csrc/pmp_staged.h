// Passes that gather from LDS: the PMP iteration of mid-sized instances.
//
// A random 4- or 8-byte gather from the L2 moves a whole 128-byte line to the
// CU, which caps the gather layout at about 2.2e11 nonzeros/s; the binned
// layout moves every nonzero's message through memory and back (12 bytes a
// nonzero and pass).  While the gathered vector itself is small (v of 1e5
// links: 400 KB), it is cheaper to let every CU stream all of it through its
// LDS, chunk by chunk, and gather there: one workgroup per CU owns a block of
// rows (streams or links), and its entries are 16-bit indices into the chunk.
//
//   stream pass  S = 1: a workgroup sums its streams over all chunks of v and
//                runs the stream update itself.
//   link pass    x is larger: S workgroups share a block of links, each
//                streaming 1 / S of x, and leave partial sums; a second kernel
//                adds the S of them in order and runs the link update.
//
// The next chunk and its indices are on their way, in registers, while the
// present one is summed.  Indices: in every chunk the block's rows are
// sorted by how many words of two entries they have there; 64 of them (a
// wave's lanes) form a slice, whose length is that of its first row, so there
// is next to no padding (the index of a zero behind the chunk).  A lane adds
// its row's entries to the row's FP64 sum in LDS.  A row belongs to one lane
// in a chunk and the chunks follow each other, so the order of every sum is
// fixed by the tables' chunks and the column order: runs repeat bit for bit.
//
// What bounds it: the CU's L2 read path while staging (about 40 bytes a clock
// and CU), then LDS gathers (5-6 clocks a wave and step), then launch latency.
// Measured rates and where the line to the other layouts lies: staged_plan.
//
// Part of pmp_kernels.hip, which includes it.
#pragma once

#include "pmp_device.h"

#include <algorithm>

namespace pmp {

namespace {

constexpr int kST = 1024;                  // lanes of a workgroup
constexpr int kSW = kST / 64;
constexpr int kStLds = 158 * 1024;         // dynamic LDS of a workgroup
constexpr int kStK = 4;                    // most slices per wave
constexpr int kStWords = 8;                // index words whose gathers are in flight together
constexpr int kStSteps = 9;                // 16-byte loads of a lane per chunk (at most 144 KB)

// A chunk on its way to LDS: 16 bytes a lane and step, held in registers until
// the chunk before it is used up.  Up to 15 bytes past the end are read (the
// workspace pads every vector to 256 bytes).
typedef unsigned quad_t __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ void chunk_load(quad_t (&v)[kStSteps], const T *src, int cnt)
{
    const int quads = cnt > 0 ? (cnt * (int)sizeof(T) + 15) / 16 : 0;
    const quad_t *s4 = (const quad_t *)src;
#pragma unroll
    for (int k = 0; k < kStSteps; ++k)
        if (k * kST < quads) v[k] = s4[min(k * kST + (int)threadIdx.x, quads - 1)];
}
template <typename T>
__device__ __forceinline__ void chunk_store(const quad_t (&v)[kStSteps], T *dst, int cnt)
{
    const int quads = cnt > 0 ? (cnt * (int)sizeof(T) + 15) / 16 : 0;
#pragma unroll
    for (int k = 0; k < kStSteps; ++k) {
        const int i = k * kST + (int)threadIdx.x;
        if (k * kST < quads && i < quads) ((quad_t *)dst)[i] = v[k];
    }
}

// Row sums of block r over the chunks [c0, c1): returns the block's sums in
// LDS, in row order.
template <typename T>
__device__ __forceinline__ double *staged_rows(const StagedSide &sd, const T *src, int r, int c0, int c1,
                                               unsigned char *lds)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *acc = (double *)lds;                          // [RB]
    T *buf = (T *)(lds + (size_t)sd.RB * 8);              // the chunk, with a zero behind it
    for (int i = tid; i < sd.RB; i += kST) acc[i] = 0.0;
    if (tid == 0) buf[sd.CH] = T(0);                      // (chunks are whole 16-byte steps: it stays)
    // lane i holds the descriptor of the i-th chunk, so that none is waited for
    // between chunks
    uint4 mine = make_uint4(0, 0, 0, 0);
    if (lane < c1 - c0) mine = sd.desc[((size_t)r * sd.C + c0 + lane) * kSW + wave];
    auto desc = [&](int c) {
        const int i = min(c - c0, 63);
        return make_uint4((unsigned)__builtin_amdgcn_readlane((int)mine.x, i),
                          (unsigned)__builtin_amdgcn_readlane((int)mine.y, i),
                          (unsigned)__builtin_amdgcn_readlane((int)mine.z, i),
                          (unsigned)__builtin_amdgcn_readlane((int)mine.w, i));
    };
    quad_t next[kStSteps];
#pragma unroll
    for (int k = 0; k < kStSteps; ++k) next[k] = quad_t(0u);
    const unsigned none = (unsigned)sd.CH | (unsigned)sd.CH << 16;
    // index words and rows of a chunk, asked for a chunk ahead
    constexpr int kAhead = sizeof(T) == 4 ? 2 * kStWords : kStWords;
    unsigned q[kAhead], qn[kAhead];
    unsigned long long pm, pmn;                           // the lane's row in each slice, 16 bits each
    auto ask = [&](int c, const uint4 &ds, unsigned *qq, unsigned long long &pp) {
        const unsigned *p = sd.idx + (size_t)ds.x * 64 + lane;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) qq[u] = u < (int)ds.y ? p[u * 64] : none;
        pp = ((const unsigned long long *)sd.perm)[(((size_t)r * sd.C + c) * kSW + wave) * 64 + lane];
    };
    const uint4 first = desc(c0);
    chunk_load<T>(next, src + (size_t)c0 * sd.CH, min(sd.src - c0 * sd.CH, sd.CH));
    ask(c0, first, qn, pmn);
    for (int c = c0; c < c1; ++c) {
        if (c > c0) __syncthreads();                      // the chunk before is used up
        chunk_store<T>(next, buf, min(sd.src - c * sd.CH, sd.CH));
#pragma unroll
        for (int u = 0; u < kAhead; ++u) q[u] = qn[u];
        pm = pmn;
        __syncthreads();
        const uint4 ds = desc(c);
        if (c + 1 < c1) {
            chunk_load<T>(next, src + (size_t)(c + 1) * sd.CH, min(sd.src - (c + 1) * sd.CH, sd.CH));
            ask(c + 1, desc(c + 1), qn, pmn);
        }
        const T *bc = buf;
        const int total = (int)ds.y;
        const unsigned long long ends = (unsigned long long)ds.w << 32 | ds.z;   // last words of slices
        int k = 0;
        double s0 = 0.0, s1 = 0.0;
        // eight words: all their gathers in flight, then the sums
        auto eight = [&](const unsigned *w, int i) {
            T v[2 * kStWords];
#pragma unroll
            for (int u = 0; u < kStWords; ++u) {
                v[2 * u] = bc[w[u] & 0xffffu];
                v[2 * u + 1] = bc[w[u] >> 16];
            }
#pragma unroll
            for (int u = 0; u < kStWords; ++u) {
                s0 += (double)v[2 * u];
                s1 += (double)v[2 * u + 1];
                if (ends >> (i + u) & 1) {                // uniform in the wave
                    const unsigned row = (unsigned)(pm >> (16 * k)) & 0xffffu;
                    if (row != 0xffffu) acc[row] += s0 + s1;
                    s0 = s1 = 0.0;
                    ++k;
                }
            }
        };
#pragma unroll
        for (int i = 0; i < kAhead; i += kStWords)
            if (i < total) eight(q + i, i);
        for (int i = kAhead; i < total; i += kStWords) {    // (these wait behind the next chunk's loads)
            const unsigned *p = sd.idx + (size_t)ds.x * 64 + lane;
            unsigned w[kStWords];
#pragma unroll
            for (int u = 0; u < kStWords; ++u) w[u] = i + u < total ? p[(i + u) * 64] : none;
            eight(w, i);
        }
    }
    __syncthreads();
    return acc;
}

template <typename T, bool CHECK>
__global__ __launch_bounds__(kST) void k_staged_stream(Dev<T> d)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ double sred[kSW];
    const StagedSide &sd = d.ss;
    const double irho = d.ctl->irho;
    if (d.ctl->done) return;
    const int r = blockIdx.x;
    // the state of a lane's first two streams is asked for before the sums
    constexpr int G = 2;
    const int j0 = r * sd.RB, nr = min(sd.RB, d.n - j0);
    int L[G];
    double a[G], w[G], xo[G];
    bool a2[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int i = threadIdx.x + g * kST, j = j0 + i;
        L[g] = 0;
        if (i < nr) {
            L[g] = d.col_ptr[j + 1] - d.col_ptr[j];
            a[g] = (double)d.a[j];
            w[g] = (double)d.wsig[j];
            a2[g] = is_alpha2(d, j);
            xo[g] = CHECK ? (double)d.x[j] : 0.0;
        }
    }
    const double *nat = staged_rows<T>(sd, d.v, r, 0, sd.C, lds);
    double part = 0.0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int i = threadIdx.x + g * kST, j = j0 + i;
        if (i < nr) {
            T xt, at;
            stream_core<T>(a[g], w[g], L[g], nat[i], irho, d.lo, d.hi, d.alpha, a2[g], xt, at);
            if (CHECK) {
                const double dx = (double)xt - xo[g];
                part += screen((double)L[g] * dx * dx, (double)at);
            }
            d.x[j] = xt;
            d.a[j] = at;
        }
    }
    for (int i = threadIdx.x + G * kST; i < nr; i += kST) {
        const int j = j0 + i;
        part += stream_update<T, CHECK>(d, j, d.col_ptr[j + 1] - d.col_ptr[j], nat[i], irho);
    }
    if (CHECK) {
        part = block_sum_n<kST>(part, sred);
        if (threadIdx.x == 0) d.spart[r] = part;
    }
}

// Partial link sums: workgroup (r, s) sums the links of block r over its
// share of the chunks of src.
template <typename T>
__global__ __launch_bounds__(kST) void k_staged_part(StagedSide sd, const T *src, double *part, int rows,
                                                     const Ctl *ctl)
{
    extern __shared__ __align__(16) unsigned char lds[];
    if (ctl && ctl->done) return;
    const int s = blockIdx.x % sd.S, r = blockIdx.x / sd.S;
    const double *nat = staged_rows<T>(sd, src, r, s * sd.CPS, (s + 1) * sd.CPS, lds);
    const int l0 = r * sd.RB, nr = min(sd.RB, rows - l0);
    for (int i = threadIdx.x; i < nr; i += kST) part[(size_t)s * rows + l0 + i] = nat[i];
}

template <typename T, int MODE>
__global__ __launch_bounds__(kBlock) void k_staged_link(Dev<T> d)
{
    __shared__ double sred[kBlock / 64];
    const int l = blockIdx.x * kBlock + threadIdx.x;
    const bool in = l < d.m;
    double y = 0.0, r2 = 0.0, s2 = 0.0;
    LinkIn li{1.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int deg = 0;
    if (in) {
        li = link_load<T, MODE>(d, l);
        deg = d.row_ptr[l + 1] - d.row_ptr[l];
#pragma unroll 8
        for (int s = 0; s < d.sl.S; ++s) y += d.lsum[(size_t)s * d.m + l];
    }
    if (d.ctl->done) return;
    if (in) link_update_in<T, MODE>(d, l, deg, y, li, r2, s2);
    if (MODE == kCheck) {
        r2 = block_sum(r2, sred);
        s2 = block_sum(s2, sred);
        if (threadIdx.x == 0) {
            d.lpart[2 * blockIdx.x] = r2;
            d.lpart[2 * blockIdx.x + 1] = s2;
        }
    }
}

// Reverse mode: R^T ybar and R Sbar in the same tables.  ybar and Sbar are
// staged in the problem's precision (yt, st), as the binned messages are: for
// FP64 problems, and FP32 ones that would otherwise be binned (Dev::staged_adj).
template <typename T>
__global__ __launch_bounds__(kST) void k_staged_adj_stream(Dev<T> d, AdjDev a, const T *xt, int last,
                                                           const T *yt, T *st)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const StagedSide &sd = d.ss;
    const double rho = d.ctl->rho;
    const int r = blockIdx.x;
    const double *nat = staged_rows<T>(sd, yt, r, 0, sd.C, lds);
    const int j0 = r * sd.RB, nr = min(sd.RB, d.n - j0);
    for (int i = threadIdx.x; i < nr; i += kST) {
        const int j = j0 + i;
        AdjStreamIn<T> in;
        in.load(d, a, xt, j, last);
        st[j] = (T)adj_stream_step<T>(d, a, in, j, d.col_ptr[j + 1] - d.col_ptr[j], nat[i], rho);
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_staged_adj_link(Dev<T> d, AdjDev a, const uint8_t *mu_prev, T *yt)
{
    const int l = blockIdx.x * kBlock + threadIdx.x;
    if (l >= d.m) return;
    AdjLinkIn in;
    in.load(a, l, mu_prev);
    double vbar = 0.0;
#pragma unroll 8
    for (int s = 0; s < d.sl.S; ++s) vbar += d.lsum[(size_t)s * d.m + l];
    in.B += vbar;
    in.U -= vbar;
    if (mu_prev) {
        yt[l] = (T)adj_link_step(a, l, d.row_ptr[l + 1] - d.row_ptr[l], d.alpha, in);
    } else {
        a.B[l] = in.B;
        a.U[l] = in.U;
    }
}

template <typename T>
__global__ void k_staged_adj_cast(const double *y, int m, T *yt)
{
    for (int l = blockIdx.x * blockDim.x + threadIdx.x; l < m; l += gridDim.x * blockDim.x) yt[l] = (T)y[l];
}

// ---- tables ------------------------------------------------------------------

// First entry of [b, e) whose index is not below v (indices ascending).  Entry
// numbers go up to 2^31 - 1, so the middle is formed from the distance.
template <typename I>
__host__ __device__ __forceinline__ int lower_entry(const I &idx, int b, int e, long long v)
{
    while (b < e) {
        const int mid = b + (e - b) / 2;
        if (idx[mid] < v) b = mid + 1;
        else e = mid;
    }
    return b;
}

// First and last + 1 entry of row [b, e) in [lo, hi).
__device__ __forceinline__ void chunk_range(const int *idx, int b, int e, long long lo, long long hi, int &p,
                                            int &q)
{
    p = lower_entry(idx, b, e, lo);
    q = lower_entry(idx, b, e, hi);
}

// Tile (r, c): its rows sorted by their words there, most first, in slots
// (slice k of a wave: the slices go round the waves forth and back), every
// wave's words and the mask of those that end a slice.  A wave of more than 64
// words sets *fail.
__global__ __launch_bounds__(kST) void k_staged_sort(StagedSide sd, const int *ptr, const int *idx, int rows,
                                                     uint16_t *perm, uint4 *desc, int *total, int *fail)
{
    __shared__ int hist[256];
    __shared__ unsigned char width[kStK * kSW], words[kStK * kST];
    const int c = blockIdx.x % sd.C, r = blockIdx.x / sd.C;
    const int r0 = r * sd.RB, nr = min(sd.RB, rows - r0), tid = threadIdx.x;
    const size_t t = (size_t)blockIdx.x;
    uint16_t *out = perm + t * kStK * kST;                // [wave][lane][slice]
    for (int i = tid; i < 256; i += kST) hist[i] = 0;
    for (int i = tid; i < kStK * kSW; i += kST) width[i] = 0;
    for (int i = tid; i < kStK * kST; i += kST) out[i] = 0xffff;
    __syncthreads();
    for (int i = tid; i < nr; i += kST) {
        int p, q;
        chunk_range(idx, ptr[r0 + i], ptr[r0 + i + 1], (long long)c * sd.CH, (long long)(c + 1) * sd.CH, p, q);
        const int w = min((q - p + 1) / 2, 255);          // (255 is refused below)
        words[i] = (unsigned char)w;
        if (w > 0) atomicAdd(&hist[255 - w], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int s = 0;
        for (int i = 0; i < 256; ++i) {
            const int n = hist[i];
            hist[i] = s;
            s += n;
        }
    }
    __syncthreads();
    for (int i = tid; i < nr; i += kST) {
        const int w = words[i];
        if (w == 0) continue;
        const int at = atomicAdd(&hist[255 - w], 1), sl = at / 64, k = sl / kSW;
        const int wave = k & 1 ? kSW - 1 - sl % kSW : sl % kSW;
        out[(wave * 64 + at % 64) * kStK + k] = (uint16_t)i;
        if (at % 64 == 0) width[k * kSW + wave] = (unsigned char)w;
    }
    __syncthreads();
    if (tid < kSW) {
        unsigned long long ends = 0;
        int sum = 0;
        for (int k = 0; k < kStK; ++k) {
            sum += width[k * kSW + tid];
            if (sum > 64) {
                atomicOr(fail, 1);
                sum = 64;
            }
            if (width[k * kSW + tid]) ends |= 1ull << (sum - 1);
        }
        desc[t * kSW + tid] = make_uint4(0u, (unsigned)sum, (unsigned)ends, (unsigned)(ends >> 32));
        total[t * kSW + tid] = sum;
    }
}

// The descriptors' first words and the index words of tile (r, c).
__global__ __launch_bounds__(kST) void k_staged_fill(StagedSide sd, const int *ptr, const int *idx,
                                                     const uint16_t *perm, uint4 *desc, const int *start,
                                                     unsigned *words)
{
    const int c = blockIdx.x % sd.C, r = blockIdx.x / sd.C, r0 = r * sd.RB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t t = (size_t)blockIdx.x;
    const uint4 ds = desc[t * kSW + wave];
    const unsigned long long ends = (unsigned long long)ds.w << 32 | ds.z;
    const unsigned at = (unsigned)start[t * kSW + wave];
    unsigned *out = words + (size_t)at * 64 + lane;
    int k = -1, p = 0, q = 0;
    for (int i = 0; i < (int)ds.y; ++i) {
        if (i == 0 || (ends >> (i - 1) & 1)) {            // the next slice's row
            const int row = perm[((t * kSW + wave) * 64 + lane) * kStK + ++k];
            p = q = 0;
            if (row != 0xffff)
                chunk_range(idx, ptr[r0 + row], ptr[r0 + row + 1], (long long)c * sd.CH,
                            (long long)(c + 1) * sd.CH, p, q);
        }
        const unsigned lo = p < q ? (unsigned)(idx[p] - c * sd.CH) : (unsigned)sd.CH;
        const unsigned hi = q - p > 1 ? (unsigned)(idx[p + 1] - c * sd.CH) : (unsigned)sd.CH;
        out[(size_t)i * 64] = lo | hi << 16;
        p += min(2, q - p);
    }
    if (lane == 0) desc[t * kSW + wave].x = at;
}

// One side's shape: S workgroups a block of rows, about kSmallBlocks in all.
bool staged_side(int rows, int src, size_t sz, int S, StagedSide &sd)
{
    const int R = std::max(1, kSmallBlocks / S);
    const int per = (rows + R - 1) / R;
    sd.RB = std::min(kStK * kST, std::max(64, (per + 63) / 64 * 64));
    sd.R = (rows + sd.RB - 1) / sd.RB;
    const long long bytes = std::min<long long>(kStLds - (long long)sd.RB * 8 - 64, kStSteps * kST * 16);
    const long long room = bytes / (long long)sz / 8 * 8;
    const long long most = std::min<long long>(room, 65528);
    if (most < 1024) return false;
    const long long chunks = (src + most - 1) / most;
    sd.CPS = (int)std::max<long long>(1, (chunks + S - 1) / S);
    if (sd.CPS > 63) return false;          // a lane of a wave for every chunk's descriptor
    sd.S = S;
    sd.C = S * sd.CPS;
    sd.CH = (int)(((src + sd.C - 1) / sd.C + 7) / 8 * 8);
    sd.src = src;
    sd.perm = nullptr;
    sd.desc = nullptr;
    sd.idx = nullptr;
    return true;
}

// A wave holds at most 64 words of two entries a lane in a chunk, so a tile at
// most 128 entries a lane and a row at most 128.  Above that on average some
// wave is too full for certain: such tables are not begun (their set-up walks
// every row of every tile).
bool staged_room(const StagedSide &sd, int rows, long long nnz)
{
    return nnz <= 128LL * sd.C * std::min<long long>(rows, (long long)sd.R * kST);
}

size_t staged_lds(const StagedSide &sd, size_t sz) { return (size_t)sd.RB * 8 + ((size_t)sd.CH + 8) * sz; }

}  // namespace

bool staged_plan(int m, int n, long long nnz, size_t sz, StagedSide &ss, StagedSide &sl)
{
    if (m < 1024 || n < 1024) return false;
    // Up to there the gather passes have blocks for every CU and need two
    // launches, not three: 1e4 links x 1e5 streams, nnz = 7.5e5, an iteration
    // 14.1 us against 16.1 (FP64), 12.8 against 13.0 (FP32).
    if (small_blocks(nnz)) return false;
    if (!staged_side(n, m, sz, 1, ss) || ss.R > kSmallBlocks || !staged_room(ss, n, nnz)) return false;
    // Times of an iteration in us, fitted to MI355X runs.  A chunk costs its
    // bytes at 62 KB/us (load path, then LDS writes) and 0.8 for the two
    // barriers and the sums between them.  Measured, against the layout taken
    // otherwise: 1e5 links x 5e5 streams, nnz = 5e6: 29.8 against 36.3 binned
    // (FP32), 43.9 against 64.2 gathered (FP64); 1e5 x 1e6, nnz = 7.5e6: 39.3
    // against 44.6 binned; 2e4 x 3e5, nnz = 2.4e6: 18 and 22 against 24 and 36;
    // 1e5 x 1e6 in FP64: 56 against 119.  On the other side of the line: 2e5 x
    // 5e5: 51 against 36.5 binned, 75 against 65 gathered; 1e5 x 3e5, nnz = 3e6:
    // 25.6 against 25.0 binned; 1e5 x 1e5, nnz = 8e5: 21 against 16 gathered.
    const double mil = nnz * 1e-6;
    auto chunks = [&](const StagedSide &sd) { return sd.CPS * (0.8 + (double)sd.CH * sz / 62e3); };
    double best = 1e30;
    for (int S = 1; S <= 32; ++S) {
        StagedSide t;
        if (!staged_side(m, n, sz, S, t) || t.R * t.S > kSmallBlocks) continue;
        const double us = chunks(t) + t.RB * 8.0 / 60e3 + (double)m * 8.0 * S / 4e6;
        if (us < best) {
            best = us;
            sl = t;
        }
    }
    if (best > 1e29 || !staged_room(sl, m, nnz)) return false;
    const double staged = 3.5 + chunks(ss) + 3.0 + best + 4.5 + 0.5 * mil;
    // the other layouts: gathers from L2 (or past it), binned messages
    const bool binned = sz == 4 && nnz >= (1LL << 21);
    auto gather = [&](double bytes) {
        return 4.5 + mil * (bytes > 4.2e6 ? 9.0 : sz == 8 ? 4.9 : 4.1);
    };
    auto messages = [&]() { return mil < 4.19 ? 13.7 + 3.7 * mil : mil < 13.1 ? 20.0 + 3.3 * mil : 12.0 + 5.9 * mil; };
    const double other = binned ? messages() : gather((double)m * sz) + gather((double)n * sz);
    return staged < 0.95 * other;
}

size_t staged_tiles(const StagedSide &sd) { return (size_t)sd.R * sd.C * kSW; }
size_t staged_slots(const StagedSide &sd) { return (size_t)sd.R * sd.C * kStK * kST; }
// Index words a side may take.  A tile needs at most a word an entry, and a slice
// of its widest row (64 lanes, at most 64 words): every other slice is no wider
// than the rows of the one before it.
size_t staged_words_cap(const StagedSide &sd, long long nnz)
{
    return std::min(2 * (size_t)nnz + 65536, (size_t)nnz + (size_t)sd.R * sd.C * 64 * 64);
}
size_t staged_scratch_ints(const StagedSide &sd)
{
    return 2 * staged_tiles(sd) + 2 + scan_scratch_ints((int)staged_tiles(sd));
}

hipError_t staged_build(StagedSide &ss, const StagedTables &ts, StagedSide &sl, const StagedTables &tl, long long nnz,
                        int *scratch, bool *ok, hipStream_t s)
{
    StagedSide *sd[2] = {&ss, &sl};
    const StagedTables *tb[2] = {&ts, &tl};
    int *start[2], *fail[2], h[2][2] = {};
    hipError_t e = hipSuccess;
    for (int k = 0; k < 2; ++k) {
        const int tiles = (int)staged_tiles(*sd[k]);
        int *total = scratch, *bsum = total + 2 * tiles + 2;
        start[k] = total + tiles;
        fail[k] = total + 2 * tiles + 1;                  // right behind the last start
        scratch += staged_scratch_ints(*sd[k]);
        launch_fill_int(fail[k], 0, 1, s);
        hipLaunchKernelGGL(k_staged_sort, dim3(sd[k]->R * sd[k]->C), dim3(kST), 0, s, *sd[k], tb[k]->ptr, tb[k]->idx,
                           tb[k]->rows, tb[k]->perm, tb[k]->desc, total, fail[k]);
        launch_scan_int(total, tiles, start[k], bsum, s);
        if (e == hipSuccess) e = hipMemcpyAsync(h[k], start[k] + tiles, 8, hipMemcpyDeviceToHost, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    *ok = true;
    for (int k = 0; k < 2; ++k) *ok = *ok && h[k][1] == 0 && h[k][0] >= 0 && (size_t)h[k][0] * 64 <= staged_words_cap(*sd[k], nnz);
    if (!*ok) return hipSuccess;
    for (int k = 0; k < 2; ++k) {
        hipLaunchKernelGGL(k_staged_fill, dim3(sd[k]->R * sd[k]->C), dim3(kST), 0, s, *sd[k], tb[k]->ptr, tb[k]->idx,
                           tb[k]->perm, tb[k]->desc, start[k], tb[k]->words);
        sd[k]->perm = tb[k]->perm;
        sd[k]->desc = tb[k]->desc;
        sd[k]->idx = tb[k]->words;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t staged_configure()
{
    hipError_t e = hipSuccess;
    for (const void *f : {(const void *)k_staged_stream<T, false>, (const void *)k_staged_stream<T, true>,
                          (const void *)k_staged_part<T>, (const void *)k_staged_adj_stream<T>})
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kStLds);
    return e;
}

template <typename T>
void launch_staged_stream(const Dev<T> &d, bool check, hipStream_t s)
{
    const size_t lds = staged_lds(d.ss, sizeof(T));
    if (check) hipLaunchKernelGGL((k_staged_stream<T, true>), dim3(d.ss.R), dim3(kST), lds, s, d);
    else hipLaunchKernelGGL((k_staged_stream<T, false>), dim3(d.ss.R), dim3(kST), lds, s, d);
}

template <typename T>
void launch_staged_link(const Dev<T> &d, int mode, hipStream_t s)
{
    hipLaunchKernelGGL((k_staged_part<T>), dim3(d.sl.R * d.sl.S), dim3(kST), staged_lds(d.sl, sizeof(T)), s,
                       d.sl, d.x, d.lsum, d.m, d.ctl);
    const dim3 g((d.m + kBlock - 1) / kBlock);
    if (mode == kPlain) hipLaunchKernelGGL((k_staged_link<T, kPlain>), g, dim3(kBlock), 0, s, d);
    else if (mode == kSave) hipLaunchKernelGGL((k_staged_link<T, kSave>), g, dim3(kBlock), 0, s, d);
    else hipLaunchKernelGGL((k_staged_link<T, kCheck>), g, dim3(kBlock), 0, s, d);
}

template <typename T>
void launch_staged_adj_stream(const Dev<T> &d, const AdjDev &a, const T *xt, int last, const T *yt, T *st,
                              hipStream_t s)
{
    hipLaunchKernelGGL((k_staged_adj_stream<T>), dim3(d.ss.R), dim3(kST), staged_lds(d.ss, sizeof(T)), s, d, a,
                       xt, last, yt, st);
}

template <typename T>
void launch_staged_adj_link(const Dev<T> &d, const AdjDev &a, const uint8_t *mu_prev, const T *st, T *yt,
                            hipStream_t s)
{
    hipLaunchKernelGGL((k_staged_part<T>), dim3(d.sl.R * d.sl.S), dim3(kST), staged_lds(d.sl, sizeof(T)), s,
                       d.sl, st, d.lsum, d.m, (const Ctl *)nullptr);
    hipLaunchKernelGGL((k_staged_adj_link<T>), dim3((d.m + kBlock - 1) / kBlock), dim3(kBlock), 0, s, d, a,
                       mu_prev, yt);
}

template <typename T>
void launch_staged_adj_cast(const Dev<T> &d, const AdjDev &a, T *yt, hipStream_t s)
{
    hipLaunchKernelGGL((k_staged_adj_cast<T>), dim3(std::min(1024, (d.m + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                       s, a.ybar, d.m, yt);
}

int staged_link_parts(int m) { return (m + kBlock - 1) / kBlock; }

#define PMP_STAGED_INSTANTIATE(T)                                                              \
    template hipError_t staged_configure<T>();                                                 \
    template void launch_staged_stream<T>(const Dev<T> &, bool, hipStream_t);                  \
    template void launch_staged_link<T>(const Dev<T> &, int, hipStream_t);                     \
    template void launch_staged_adj_stream<T>(const Dev<T> &, const AdjDev &, const T *, int,  \
                                              const T *, T *, hipStream_t);                    \
    template void launch_staged_adj_link<T>(const Dev<T> &, const AdjDev &, const uint8_t *,   \
                                            const T *, T *, hipStream_t);                      \
    template void launch_staged_adj_cast<T>(const Dev<T> &, const AdjDev &, T *, hipStream_t);
PMP_STAGED_INSTANTIATE(float)
PMP_STAGED_INSTANTIATE(double)
#undef PMP_STAGED_INSTANTIATE

}  // namespace pmp
