// Index arithmetic and planning rules of the HIP library at sizes that no test
// runs on a GPU, under AddressSanitizer and UndefinedBehaviorSanitizer (host
// code only; no GPU call is made).  The translation unit includes the source
// whose helpers have internal linkage; the other sources are linked as usual.
#include "pmp_kernels.hip"

#include <cstdio>
#include <cstdlib>
#include <vector>

using namespace pmp;

#define REQUIRE(cond)                                                          \
    do {                                                                       \
        if (!(cond)) {                                                         \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                      \
        }                                                                      \
    } while (0)

// Entries [b, e) of a pattern of up to 2^31 - 1 nonzeros without their memory:
// entry k holds 3 (k - b); a read outside the row ends the program.
struct RowOf {
    int b, e;
    int operator[](int k) const
    {
        REQUIRE(k >= b && k < e);
        return 3 * (k - b);
    }
};

static void check_lower_entry()
{
    const int rows[][2] = {{0, 0},
                           {0, 1},
                           {5, 4000},
                           {(1 << 30) - 7, (1 << 30) + 9},
                           {1079990000, 1080000000},
                           {2147483647 - 5000, 2147483647}};
    for (auto &r : rows) {
        const RowOf row{r[0], r[1]};
        for (long long v : {-1LL, 0LL, 1LL, 2999LL, 3000LL, 14997LL, 1LL << 31}) {
            const long long k = r[0] + (v <= 0 ? 0 : (v + 2) / 3);
            REQUIRE(lower_entry(row, r[0], r[1], v) == (int)std::min<long long>(k, r[1]));
        }
    }
}

// Tables that a pattern of these sizes cannot fit are not planned; the shapes
// that run staged still are.
static void check_staged_plan()
{
    StagedSide ss, sl;
    for (size_t sz : {(size_t)4, (size_t)8}) {
        REQUIRE(!staged_plan(300000, 1040000, 1080000000LL, sz, ss, sl));
        REQUIRE(staged_plan(100000, 500000, 5000000LL, sz, ss, sl));
        REQUIRE(staged_plan(20003, 200007, 1600000LL, sz, ss, sl));
    }
    const int sizes[][2] = {{5000, 150000}, {20000, 200000}, {100000, 1000000}, {300000, 1040000}, {2000000, 1040000}};
    for (auto &z : sizes)
        for (long long nnz = 1 << 20; nnz < (1LL << 31); nnz += nnz / 3)
            for (size_t sz : {(size_t)4, (size_t)8}) {
                if (!staged_plan(z[0], z[1], nnz, sz, ss, sl)) continue;
                const StagedSide *side[2] = {&ss, &sl};
                for (int k = 0; k < 2; ++k) {
                    const StagedSide &sd = *side[k];
                    const int rows = k ? z[0] : z[1];
                    // a tile's mean is within what its 16 waves hold
                    REQUIRE(nnz / ((long long)sd.R * sd.C) <= 16LL * 64 * 64 * 2);
                    REQUIRE(nnz / ((long long)rows * sd.C) <= 128);
                    REQUIRE(sd.C <= 32 * 63 && (long long)sd.CH * sd.C >= sd.src);
                }
            }
}

// Walks over entries that end at 2^31 - 1: every entry once, nothing beyond.
static void check_walks()
{
    const unsigned counts[] = {0u, 1u, 255u, 256u, 2047u, 2048u, 2049u, 5000u, 2147483647u - 1792u, 2147483647u};
    for (unsigned cnt : counts)
        for (unsigned lane : {0u, 1u, 254u, 255u}) {
            unsigned next = lane;
            bool ended = false;
            strided_rounds(cnt, lane,
                           [&](unsigned k) {
                               REQUIRE(!ended && k == next && (unsigned long long)k + 7 * kBlock < cnt);
                               next = k + 8 * kBlock;
                           },
                           [&](unsigned k) {
                               REQUIRE(!ended && k == next && k < cnt);
                               ended = true;
                               for (int r = 0; r < 8; ++r) next = (unsigned long long)k + r * kBlock < cnt ? k + (r + 1) * kBlock : next;
                           });
            REQUIRE(next >= cnt && (lane >= cnt || next - cnt < (unsigned)kBlock));
        }
    const int rows[][2] = {{0, 4097}, {7, 7 + 8192}, {7, 7 + 8193}, {2147483647 - 50000, 2147483647}};
    for (auto &r : rows) {
        int at = r[0], chunks = 0;
        for_chunks(r[0], r[1], [&](int b, int e) {
            REQUIRE(b == at && e > b && e - b <= kLongChunk && e <= r[1]);
            at = e;
            ++chunks;
        });
        REQUIRE(at == r[1] && chunks == (r[1] - r[0] + kLongChunk - 1) / kLongChunk);
    }
    for (long long e : {0LL, 1LL, 3LL, 4LL, 5LL, 2147483644LL, 2147483645LL, 2147483647LL})
        REQUIRE(quads_end((int)e) == (int)((e + 3) / 4));
}

// Link blocks from sampled row pointers, at the sizes of the large networks:
// taken, within the plan's bounds (the block starts' array ends there), every
// row once, and no block much heavier than its share.
static void check_sampled(int m, int n, long long nnz, int kind, bool taken)
{
    std::vector<int> ptr((size_t)m + 1, 0);
    unsigned long long state = 7;
    for (int l = 0; l < m; ++l) {
        state = state * 6364136223846793005ull + 1442695040888963407ull;
        const long long mean = nnz / m;
        long long d = 0;
        if (kind == 0) d = (long long)(state >> 33) % (2 * mean + 1);          // about the mean
        else if (kind == 1) d = l < m / 2 ? 0 : 2 * mean;                      // half the links unused
        else d = l % 5000 == 0 ? 4000 : l % 3 == 0 ? mean : 0;                 // hubs among short rows
        ptr[(size_t)l + 1] = (int)std::min<long long>(nnz, ptr[(size_t)l] + d);
    }
    const long long have = ptr[(size_t)m];
    long long most = 0, longest = 0;
    for (int l = 0; l < m; ++l) longest = std::max<long long>(longest, ptr[(size_t)l + 1] - ptr[(size_t)l]);
    const int step = binned_sample_step(m, n, have);
    REQUIRE(step > 1 && 256LL * step <= m / 256);
    std::vector<int> samples;
    for (long long k = 0; k < m; k += step) samples.push_back(ptr[(size_t)k]);
    samples.push_back((int)have);
    const BinnedPlan bound = binned_plan(m, n, have);
    BinnedPlan bp = bound;
    std::vector<int> lbs((size_t)bound.P + 1), sbs((size_t)bound.Q + 1);
    const bool ok = binned_blocks_sampled(samples.data(), (int)samples.size(), step, (int)longest, m, n, have, bp,
                                          lbs.data(), sbs.data());
    REQUIRE(ok || !taken);
    if (!ok) return;
    REQUIRE(bp.P >= 1 && bp.P <= bound.P && bp.LB <= bound.LB && bp.Q == bound.Q);
    REQUIRE(lbs[0] == 0 && lbs[(size_t)bp.P] == m);
    for (int p = 0; p < bp.P; ++p) {
        REQUIRE(lbs[(size_t)p + 1] > lbs[(size_t)p] && lbs[(size_t)p + 1] - lbs[(size_t)p] <= bp.LB);
        most = std::max<long long>(most, ptr[(size_t)lbs[(size_t)p + 1]] - ptr[(size_t)lbs[(size_t)p]]);
    }
    // at most the longest row and a step and a half of mean rows past the quota,
    // which is an eighth above the share at most
    const int blocks0 = bound.P - (m + bound.LB - 1) / bound.LB - 1;
    const long long quota = (have + blocks0 - 1) / blocks0;
    REQUIRE(bp.fullest == most && most <= quota + quota / 8 + longest + 3 * (have * step / (2LL * m)));
    // even rows: the blocks that the CUs hold at once, or up to a hundredth fewer
    if (kind == 0 && blocks0 <= 512) REQUIRE(bp.P <= blocks0 && bp.P >= blocks0 - blocks0 / 100);
}

// Workgroups of the gather passes over small problems: never so few segments
// that there are more of them than the chip takes at once for nothing.
static void check_small_blocks()
{
    for (long long nnz : {1000LL, 330000LL, 750000LL, (1LL << 20) - 1, 1LL << 20, 1LL << 30})
        for (int count : {1, 1000, 19800, 60000, 200000, 1000000, 2000000000}) {
            const int segs = block_segments(count, nnz), cap = block_nonzeros(nnz);
            REQUIRE(segs >= 128 && segs <= kBlock && segs % 64 == 0 && cap >= 1024 && cap <= kCap);
            if (!small_blocks(nnz)) REQUIRE(segs == kBlock && cap == kCap);
        }
}

// Up to 200 nonzeros a tile of 256 x 256 blocks, neither side of a problem has
// more (bp.Q is the stream blocks; bp.P bounds the link blocks from above).
static void check_block_counts()
{
    const long long line = 200LL * 256 * 256;
    const int sizes[][2] = {{1000000, 800000}, {1800000, 900000}, {300000, 1000000}, {100000, 500000}};
    for (auto &z : sizes)
        for (long long nnz : {2200000LL, 5000000LL, 8400000LL, 9000000LL, 12000000LL, line - 300000, line + 300000, 3 * line}) {
            const BinnedPlan bp = binned_plan(z[0], z[1], nnz);
            const int blocks0 = bp.P - (z[0] + bp.LB - 1) / bp.LB - 1;
            const bool one = nnz < line - 200000;        // (a few blocks less than 256 by rounding)
            REQUIRE(one ? bp.Q <= 256 && blocks0 <= 256 : blocks0 > 256);
        }
}

// Every row pointer: rows of which some are empty for a stretch, or much longer
// than the rest, come to no more blocks than CUs where a little more per block
// avoids it.
static void check_even_cut()
{
    for (int kind = 0; kind < 3; ++kind) {
        const int m = 60000, n = 500000;
        std::vector<int> ptr((size_t)m + 1, 0);
        for (int l = 0; l < m; ++l) {
            const int d = kind == 0 ? 60 : kind == 1 ? (l > 29000 && l < 29400 ? 0 : 60) : (l % 1000 == 0 ? 1500 : 50 + l % 7);
            ptr[(size_t)l + 1] = ptr[(size_t)l] + d;
        }
        const long long nnz = ptr[(size_t)m];
        const BinnedPlan bound = binned_plan(m, n, nnz);
        BinnedPlan bp = bound;
        std::vector<int> lbs((size_t)bound.P + 1), sbs((size_t)bound.Q + 1);
        binned_blocks(ptr.data(), m, n, nnz, bp, lbs.data(), sbs.data());
        REQUIRE(bp.P <= 256 && bp.P <= bound.P && bp.LB <= bound.LB);
        long long most = 0;
        for (int p = 0; p < bp.P; ++p) {
            REQUIRE(lbs[(size_t)p + 1] > lbs[(size_t)p] && lbs[(size_t)p + 1] - lbs[(size_t)p] <= bp.LB);
            most = std::max<long long>(most, ptr[(size_t)lbs[(size_t)p + 1]] - ptr[(size_t)lbs[(size_t)p]]);
        }
        REQUIRE(lbs[(size_t)bp.P] == m && bp.fullest == most);
    }
}

int main()
{
    check_even_cut();
    check_block_counts();
    REQUIRE(binned_sample_step(65536, 500000, 5000000) == 1 && binned_sample_step(2147483647, 500000, 2147483647) == 39);
    check_small_blocks();
    for (int kind = 0; kind < 3; ++kind) {
        check_sampled(1000000, 500000, 5000000LL, kind, kind == 0);
        check_sampled(3000000, 3000000, 30000000LL, kind, kind == 0);
        check_sampled(5000000, 20000000, 117000000LL, kind, kind == 0);
        check_sampled(10000000, 5000000, 50000000LL, kind, kind == 0);
    }
    check_walks();
    check_lower_entry();
    check_staged_plan();
    std::printf("host entries: all checks passed\n");
    return 0;
}
