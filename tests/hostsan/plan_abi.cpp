// Test-only C view of the GEMM plans (plan.cpp), so that host tests can tell
// which kernel a shape runs and in which order it walks K.
#include "../../paper_2606_18502_amd/csrc/kernels.hpp"
#include "../../paper_2606_18502_amd/csrc/plan.hpp"

extern "C" {

// out: kind, splits, krot_on, m_tiles, n_tiles, tile columns, statistics groups, workspace bytes
void test_plan_gemm(int64_t M, int64_t N, int64_t K, int epilogue, int may_split, int64_t* out) {
    const specfp8::GemmPlan p = specfp8::plan_gemm(M, N, K, epilogue, may_split != 0);
    out[0] = p.kind;
    out[1] = p.splits;
    out[2] = p.krot_on;
    out[3] = p.m_tiles;
    out[4] = p.n_tiles;
    out[5] = specfp8::tile_bn(p.kind);
    out[6] = p.stat_groups;
    out[7] = (int64_t)p.workspace_bytes;
}

// the K-step (of nk) at which a staggered tile with first column n0 starts
int test_k_start(int n0, int nk) { return specfp8::gemm_k_start(n0, nk); }

// the kind and split with the smallest estimate, by a plain search over the table
void test_plan_search(int64_t M, int64_t N, int64_t K, int epilogue, int may_split, int64_t* out) {
    using namespace specfp8;
    const int need = epilogue == kEpiStats ? kHasStats : (epilogue == kEpiSilu ? kHasSilu : 0);
    double best = -1.0;
    for (int k = 0; k < kTileKinds; ++k) {
        const TileShape& t = kTiles[k];
        if ((t.has & need) != need) continue;
        const int64_t tiles = ((M + tile_bm(k) - 1) / tile_bm(k)) * ((N + tile_bn(k) - 1) / tile_bn(k));
        const bool can = may_split && epilogue == kEpiPlain && (t.has & kHasSplit) != 0;
        for (int s = 1; s <= (can ? 8 : 1); ++s) {
            if (s > 1 && (K / 128 / s < 3 || tiles * s > 640)) break;
            const int64_t per_cu = (tiles * s + 255) / 256, resident = 160 / t.lds;
            const double blocks = t.wtm * t.wtn;
            double us = t.step_us * (double)per_cu * (double)((K / 128 + s - 1) / s) +
                        (double)((per_cu + resident - 1) / resident) * (1.61 + 0.102 * blocks) +
                        ((double)N * (double)K + (double)M * (double)K) / 10.1e6 +
                        0.119e-6 * 2.0 * (double)M * (double)N;
            if (s > 1) us += 0.7 + t.split_us + (s - 2) * t.more_us + s * (0.3 + 0.062 * blocks);
            if (best < 0.0 || us < best) {
                best = us;
                out[0] = k;
                out[1] = s;
            }
        }
    }
}

// plans `reps` times (its answers go into the result, so none is left out)
int64_t test_plan_many(int64_t M, int64_t N, int64_t K, int epilogue, int reps) {
    int64_t sum = 0;
    for (int i = 0; i < reps; ++i) sum += specfp8::plan_gemm(M, N, K, epilogue).kind;
    return sum;
}

}  // extern "C"
