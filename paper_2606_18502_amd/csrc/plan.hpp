// Launch geometry shared by the host-side planners (plan.cpp) and the
// kernels (gemm.hip, accept.hip).  Host-only code: no HIP here.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace specfp8 {

// ---- FP8 GEMM tiles ---------------------------------------------------------
// A tile is a WM x WN grid of waves, each wave holding WTM x WTN blocks of
// 16x16 outputs; STAGES LDS buffers rotate through the K-loop.  lspan8: a
// K-step's stage loads go out over the first lspan8/8 of its MFMAs.  t1 > 0:
// the alternating schedule of the large tiles, whose stage is free before MFMA
// t1; late8: with two stages, the next step's stage has to have landed before
// MFMA late8/8 of the step.  staged: the plain bf16 output leaves through LDS
// (statistics epilogues always do).  has: the kernels a kind has beside the
// plain one (each is compiled separately).  step_us: the time of one K-step of
// a workgroup alone on a compute unit, split_us and more_us: what a K split in
// two and each further split cost beyond the estimate's common term, and lds the
// KiB a workgroup holds, for the planner's estimate (plan.cpp).
struct TileShape {
    int wtm, wtn, wm, wn, stages, lspan8, late8, t1, staged, has;
    double step_us, split_us, more_us;
    int lds;
};
constexpr int kHasSplit = 1, kHasStats = 2, kHasSilu = 4;

// kind  BM x BN   waves (wave tile)  stages   chosen for
//  0   256 x 256  2x2 (128x128)      2        large M
//  1   160 x 384  2x2 (80x192)       2        M <= 320 and a very wide N (LM head)
//  2   160 x 224  2x2 (80x112)       3        wide N
//  3   128 x 256  2x2 (64x128)       3        wide N, large M
//  4   256 x 128  2x2 (128x64)       3        large M, short N
//  5   160 x 128  2x2 (80x64)        4        M from about 320 on
//  6   128 x 128  2x2 (64x64)        4
//  7   160 x 64   2x2 (80x32)        4        kinds 7 .. 12: small M or short N
//  8    64 x 128  2x2 (32x64)        4
//  9    80 x 128  1x4 (80x32)        3
// 10    80 x 64   1x4 (80x16)        4
// 11    64 x 64   2x2 (32x32)        4
// 12    32 x 64   1x4 (32x16)        4        (a 16 x 64 tile was no faster at any M)
constexpr TileShape kTiles[] = {
    {8, 8, 2, 2, 2, 6, 3, 5, 1, kHasStats, 0.991, 0, 0, 134},
    {5, 12, 2, 2, 2, 6, 3, 4, 1, kHasStats, 1.034, 0, 0, 139},
    {5, 7, 2, 2, 3, 6, 0, 3, 1, kHasSilu, 0.643, 0, 0, 146},
    {4, 8, 2, 2, 3, 6, 0, 3, 1, kHasSplit | kHasStats | kHasSilu, 0.668, 0, 0, 146},
    {8, 4, 2, 2, 3, 6, 0, 3, 0, kHasSplit, 0.659, 0, 0, 146},
    {5, 4, 2, 2, 4, 6, 0, 3, 0, kHasSplit, 0.479, 0, 0, 146},
    {4, 4, 2, 2, 4, 6, 0, 3, 0, kHasSplit | kHasStats | kHasSilu, 0.433, 0, 0, 129},
    {5, 2, 2, 2, 4, 8, 0, 0, 0, kHasSplit, 0.362, 0, 0.1, 113},
    {2, 4, 2, 2, 4, 8, 0, 0, 0, kHasSplit | kHasStats | kHasSilu, 0.319, 0, 0, 97},
    {5, 2, 1, 4, 3, 8, 0, 0, 0, kHasSplit | kHasSilu, 0.390, 0, 0, 79},
    {5, 1, 1, 4, 4, 8, 0, 0, 0, kHasSplit, 0.261, 0.5, 0, 73},
    {2, 2, 2, 2, 4, 8, 0, 0, 0, kHasSplit | kHasSilu, 0.207, 0, 0, 65},
    {2, 1, 1, 4, 4, 8, 0, 0, 0, kHasSplit, 0.169, 0, 0, 49},
};
constexpr int kTileKinds = sizeof(kTiles) / sizeof(kTiles[0]);
constexpr int kLmHeadKind = 1;
constexpr int kFarKind = 11;            // the kind that also has kernels with 64-bit operand offsets
constexpr int tile_bm(int k) { return 16 * kTiles[k].wtm * kTiles[k].wm; }
constexpr int tile_bn(int k) { return 16 * kTiles[k].wtn * kTiles[k].wn; }
constexpr int tile_waves(int k) { return kTiles[k].wm * kTiles[k].wn; }

constexpr int kGemmBK = 128;   // bytes (= E4M3 elements) of K per step

// Staggered K start: the tiles of a block of kStaggerCols columns start the nk
// K-steps at the same one.  A block is a whole number of tiles of every width
// but 224, so kinds of different widths sum a column in the same order, and
// neighbouring narrow tiles, which an XCD runs together, share the K columns
// they request (N = 28672, K = 4096, M = 64: 30.6 us with a start per tile,
// 29.4, 28.3, 27.9 and 27.7 with one per 256, 384, 768 and 1536 columns; the LM
// head at M = 320 173.5 per tile, 174.2 per 768).
constexpr int kStaggerCols = 768;
constexpr int gemm_k_start(int n0, int nk) { return n0 / kStaggerCols * 7 % nk; }
constexpr bool stats_tiles_within_blocks() {
    for (int k = 0; k < kTileKinds; ++k)
        if ((kTiles[k].has & kHasStats) && kStaggerCols % tile_bn(k) != 0) return false;
    return true;
}
static_assert(stats_tiles_within_blocks(), "statistics and plain kinds sum a column in the same order");

// Split-K reduction: every wave of a split tile stores its part of the partial
// tile in the workspace, and the last of the waves that hold the same part (an
// atomic ticket per tile and wave) adds all of them in split order and writes
// the output.  The tickets live in the first kGemmTicketBytes of the
// workspace, which must be zero before the first call and which every call
// leaves zero again.  Plans with more tiles than tickets do not split K.
constexpr size_t kGemmTicketBytes = 16384;   // 4096 tickets

// ---- acceptance ---------------------------------------------------------------
constexpr int kAcceptThreads = 256;
constexpr int kAcceptVecs = 8;                                           // 16-byte vectors per lane per item
constexpr int64_t kAcceptSlice = (int64_t)64 * kAcceptVecs * 8;          // 4096 logits per wave item
constexpr int kAcceptPerThread = kAcceptVecs * 8;                        // 64 logits per thread (sampling)
constexpr int64_t kAcceptChunk = (int64_t)kAcceptThreads * kAcceptPerThread;   // 16384 logits per sampling block

}  // namespace specfp8
