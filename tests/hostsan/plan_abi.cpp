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

}  // extern "C"
