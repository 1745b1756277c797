// Host-side planners: tile shape, K split and workspace layout of the FP8
// GEMM, and the workspace layout of the acceptance.  Plain C++ (no HIP), so
// the argument checks and plans can also be built and exercised on a host
// without a GPU.
#include <utility>

#include "kernels.hpp"
#include "plan.hpp"

namespace specfp8 {

namespace {

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Estimated time (us, up to a constant) of an M x N x K GEMM on a tile kind
// with K split some ways: the K-steps of the busiest compute unit
// (its workgroups share it, or follow each other where LDS holds no more), a
// fixed cost per workgroup batch and its epilogue, the operand and output
// bytes, and the split-K reduction.  The constants are a fit to timings of
// every kind and split (MI355X, cold weights, M from 1 to 4096).  What checks
// them: over 80 linears of random and of the layer's shapes its choice takes
// 0.3% longer than the fastest of all kinds and splits, 4.0% at most.  split_us and
// more_us correct two kinds whose splits the fit took for cheaper than they are: at
// 6144 x 4096, M = 80, the 80x64 tile split in 2 takes 13.0 us and the unsplit
// 64x64 tile 12.2; at 4096 x 3584, M = 160, 11.9 and 10.7; at 3000 x 9984, M =
// 144, the 160x64 tile split in 5 takes 18.7 and 64x128 in 3 17.7.
//
// Planning is on the host path of every call, so everything that depends on the
// kind alone is a constant of an unrolled instance (no division by a variable):
// 0.05-0.19 us a plan, 0.2-0.8 with a loop over the table.
struct Best {
    double us = -1.0;
    int kind = kFarKind, splits = 1;
};

struct Shape {
    int64_t M, N, ksteps;
    int need;           // kHas* of the epilogue
    bool may_split;
    double traffic;     // the terms without kind or split
    double out;
    int64_t steps[9];   // K-steps of a workgroup by split
};

// The kind's split with the smallest estimate, if that is below the best so
// far.  A split keeps at least 3 K-steps per workgroup and at most 640
// workgroups (beyond both, partial tiles outweigh the gain).
template <int KIND>
inline void consider(const Shape& x, Best& best) {
    constexpr TileShape t = kTiles[KIND];
    constexpr int bm = tile_bm(KIND), bn = tile_bn(KIND), resident = 160 / t.lds;
    constexpr double blocks = t.wtm * t.wtn;                           // 16x16 blocks per wave
    if ((t.has & x.need) != x.need) return;
    const int64_t tiles = ((x.M + bm - 1) / bm) * ((x.N + bn - 1) / bn);
    const int max_splits = (t.has & kHasSplit) != 0 && x.may_split ? 8 : 1;
    for (int s = 1; s <= max_splits; ++s) {
        if (s > 1 && (x.ksteps < 3 * s || tiles * s > 640)) break;
        const int64_t per_cu = (tiles * s + 255) / 256;                // workgroups of the busiest of 256 compute units
        const double batches = (double)((per_cu + resident - 1) / resident);
        double us = t.step_us * (double)per_cu * (double)x.steps[s] + batches * (1.61 + 0.102 * blocks) + x.traffic + x.out;
        if (s > 1) us += 0.7 + t.split_us + (s - 2) * t.more_us + s * (0.3 + 0.062 * blocks);
        if (best.us < 0.0 || us < best.us) best = {us, KIND, s};
    }
}

template <int... KIND>
inline void consider_all(const Shape& x, Best& best, std::integer_sequence<int, KIND...>) {
    (consider<KIND>(x, best), ...);
}

// The kind and split with the smallest estimate among those that have the
// epilogue.
GemmPlan best_plan(int64_t M, int64_t N, int64_t K, int epilogue, bool may_split) {
    Shape x{};
    x.M = M;
    x.N = N;
    x.ksteps = K / kGemmBK;
    x.need = epilogue == kEpiStats ? kHasStats : (epilogue == kEpiSilu ? kHasSilu : 0);
    x.may_split = may_split && epilogue == kEpiPlain;
    x.traffic = ((double)N * (double)K + (double)M * (double)K) / 10.1e6;
    x.out = 0.119e-6 * 2.0 * (double)M * (double)N;
    x.steps[1] = x.ksteps;
    if (x.may_split) {
        x.steps[2] = (x.ksteps + 1) / 2;
        x.steps[3] = (x.ksteps + 2) / 3;
        x.steps[4] = (x.ksteps + 3) / 4;
        x.steps[5] = (x.ksteps + 4) / 5;
        x.steps[6] = (x.ksteps + 5) / 6;
        x.steps[7] = (x.ksteps + 6) / 7;
        x.steps[8] = (x.ksteps + 7) / 8;
    }
    Best best;
    consider_all(x, best, std::make_integer_sequence<int, kTileKinds>{});
    return plan_gemm_as(M, N, K, best.kind, best.splits, epilogue);
}

// A staggered K start pays where few M-tiles read many N-tiles of weights in
// step: their row stride puts one K column of all rows on few memory channels
// (cold weights, in order -> staggered: N = 28672, K = 4096 M = 8 27.7 -> 24.5
// us, M = 80 33.7 -> 29.8, M = 160 39.0 -> 35.8; N = 12288 M = 80 18.6 -> 17.9;
// equal from N = 6144 down, where the tiles are few).
bool stagger_pays(const GemmPlan& p) { return p.splits == 1 && p.m_tiles <= 2 && p.n_tiles >= 192; }

// Whether the plain GEMM of plan p staggers: where it pays and every tile lies
// within one block of columns that share a start (plan.hpp), so that the order
// in which a column's products are summed depends on the column alone.
bool plain_staggers(const GemmPlan& p) { return stagger_pays(p) && kStaggerCols % tile_bn(p.kind) == 0; }

}  // namespace

GemmPlan plan_gemm_as(int64_t M, int64_t N, int64_t K, int kind, int splits, int epilogue) {
    GemmPlan p{};
    if (kind < 0 || kind >= kTileKinds) kind = kFarKind;
    p.kind = kind;
    const int bm = tile_bm(kind), bn = tile_bn(kind);
    p.m_tiles = (int)((M + bm - 1) / bm);
    p.n_tiles = (int)((N + bn - 1) / bn);
    const int64_t tiles = (int64_t)p.m_tiles * p.n_tiles;
    const int ksteps = (int)(K / kGemmBK);
    // only the plain epilogue of some kinds splits K, and only with a ticket per tile and wave
    if (epilogue != kEpiPlain || !(kTiles[kind].has & kHasSplit) ||
        tiles * tile_waves(kind) > (int64_t)(kGemmTicketBytes / sizeof(unsigned int)))
        splits = 1;
    if (splits > ksteps) splits = ksteps;
    if (splits < 1) splits = 1;
    p.splits = splits;
    // Many M-tiles (long prompts): tiles in groups of 4 M-tiles, so the 32
    // tiles an XCD runs at once re-read 4 activation and 8 weight tiles from
    // its L2 (5-8% at M = 4096).
    p.group_m = p.m_tiles >= 8 && splits == 1 ? 4 : 1;
    p.krot_on = 0;
    p.stat_groups = (int64_t)p.n_tiles * kTiles[kind].wn;
    p.part_off = kGemmTicketBytes;
    p.workspace_bytes =
        splits > 1 ? p.part_off + align256((size_t)tiles * splits * (size_t)bm * bn * sizeof(float)) : 0;
    return p;
}

bool gemm_strides_fit(int kind, int64_t lda, int64_t ldw) {
    if (kind < 0 || kind >= kTileKinds) return true;
    const uint64_t lim = 1ull << 32;
    return (uint64_t)(tile_bm(kind) - 1) * (uint64_t)lda + kGemmBK <= lim &&
           (uint64_t)(tile_bn(kind) - 1) * (uint64_t)ldw + kGemmBK <= lim;
}

bool lm_head_strides_limited(int64_t M, int64_t V, int64_t K) {
    if (M <= 80 || M > 320 || V < 12288 || K / kGemmBK % 2 != 0) return false;
    auto rows = [&](int64_t bn) { return ((M + 159) / 160 * ((V + bn - 1) / bn) + 255) / 256 * (160 + bn); };
    return rows(384) < rows(224) && (V % 192 != 0 || rows(384) < rows(192));
}

GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K, int epilogue, bool may_split) {
    GemmPlan p = best_plan(M, N, K, epilogue, may_split);
    // The logits stored with their statistics are the unsplit plain GEMM's bit
    // for bit: they stagger where that does (every kind with statistics has
    // tiles within one block of columns).
    if (epilogue == kEpiSilu) p.krot_on = stagger_pays(p);
    else if (epilogue == kEpiPlain) p.krot_on = plain_staggers(p);
    else p.krot_on = plain_staggers(best_plan(M, N, K, kEpiPlain, false));
    if (epilogue == kEpiPlain && p.workspace_bytes == 0 && gemm_workspace_required(M, N, K))
        p.workspace_bytes = kGemmTicketBytes;
    return p;
}

bool gemm_workspace_required(int64_t M, int64_t N, int64_t K) {
    const int64_t ksteps = K / kGemmBK;
    if (N >= 192 * 64 || M > 320) return false;
    if (M <= 80) return ksteps >= 16 && 2 * ((M + 63) / 64) * ((N + 63) / 64) <= 256;
    return ksteps >= 2 && (K >= 2 * N || N <= 4096);
}

AcceptPlan plan_accept(int64_t B, int64_t k, int64_t V) {
    AcceptPlan p{};
    p.chunk = kAcceptChunk;
    p.nchunk = (V + kAcceptChunk - 1) / kAcceptChunk;
    p.schunk = kAcceptSlice;
    p.nschunk = (V + kAcceptSlice - 1) / kAcceptSlice;
    const int64_t R = 2 * k + 1;
    p.stats_off = 0;
    p.fine_off = align256((size_t)B * R * p.nschunk * 8);     // after a float2 per (row, slice)
    p.ctr_off = p.fine_off + align256((size_t)B * p.nchunk * kAcceptThreads * sizeof(double));
    p.zx_off = p.ctr_off + align256((size_t)B * sizeof(unsigned int));
    p.bytes = p.zx_off + align256((size_t)B * k * 8);                // a float2 per (sequence, draft)
    if (B == 0) p.bytes = 0;
    return p;
}

}  // namespace specfp8
