// The FP8 GEMM (gemm_kernel.hpp): the choice of the kernel for a plan, and the
// path for operands whose rows lie too far apart for it.
#include "gemm_kernel.hpp"

namespace specfp8 {

extern template hipError_t launch_gemm_kind<0>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<1>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<2>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<3>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<4>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<5>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<6>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<7>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<8>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<9>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<10>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<11>(int, const GemmArgs&, hipStream_t);
extern template hipError_t launch_gemm_kind<12>(int, const GemmArgs&, hipStream_t);

namespace {

// Statistics of stored logits per column group (epilogues 1 and 2's entries),
// for the path whose GEMM kernel has no statistics epilogue: waves strided over
// the (row, group) pairs, lanes over a group's columns.
template <int STATS>
__device__ __forceinline__ void logit_group_stats(const GemmArgs& g, int64_t m, int64_t c, int64_t group_cols) {
    const int lane = threadIdx.x;
    const int64_t e0 = c * group_cols, e1 = min(e0 + group_cols, (int64_t)g.N);
    const uint16_t* row = reinterpret_cast<const uint16_t*>(g.y) + m * g.ldy;
    float mx = -INFINITY, s = STATS == 2 ? __int_as_float(0x7fffffff) : 0.0f;
    for (int64_t e = e0 + lane; e < e1; e += 64) {
        const float z = bf16_to_f32(row[e]);
        if (STATS == 2 && z > mx) s = __int_as_float((int)e);
        mx = fmaxf(mx, z);
    }
    if (STATS == 1) {
        mx = wave_max(mx) * g.c2;
        if (mx != -INFINITY)
            for (int64_t e = e0 + lane; e < e1; e += 64)
                s += __builtin_amdgcn_exp2f(bf16_to_f32(row[e]) * g.c2 - mx);
        s = wave_sum(s);
    } else {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const float m2 = __shfl_xor(mx, o, 64);
            const float s2 = __shfl_xor(s, o, 64);
            if (beats(m2, __float_as_int(s2), mx, __float_as_int(s))) { mx = m2; s = s2; }
        }
    }
    if (lane == 0) g.stats[m * g.ld_stats + c] = make_float2(mx, s);
}

template <int STATS>
__global__ __launch_bounds__(64) void logit_group_stats_kernel(GemmArgs g, int64_t groups, int64_t group_cols) {
    for (int64_t i = blockIdx.x; i < g.M * groups; i += gridDim.x)
        logit_group_stats<STATS>(g, i / groups, i % groups, group_cols);
}
constexpr int64_t kGroupStatsWaves = 256 * 32;   // what the chip holds

}  // namespace

hipError_t launch_gemm(const GemmPlan& p, const uint8_t* a, int64_t lda, const float* sa, int a_per_tensor,
                       const uint8_t* w, int64_t ldw, const float* sw, int w_per_tensor, int64_t M,
                       int64_t N, int64_t K, void* y, int64_t ldy, int out_f32, void* workspace,
                       hipStream_t stream, int stats_mode, float c2, float2* stats, int64_t ld_stats,
                       int64_t silu_inter) {
    const bool far = !gemm_strides_fit(p.kind, lda, ldw);
    GemmPlan q = p;
    if (far) {
        // K in the order the plan's kernel would walk it unsplit: what a call
        // stores does not depend on its strides
        q = plan_gemm_as(M, N, K, kFarKind, 1, kEpiPlain);
        q.krot_on = (p.splits > 1 ? plan_gemm(M, N, K, kEpiPlain, false) : p).krot_on;
    }
    GemmArgs g{};
    g.stats = stats; g.ld_stats = ld_stats; g.c2 = c2;
    g.silu_inter = (int)silu_inter;
    g.a = a; g.w = w; g.sa = sa; g.sw = sw; g.y = y;
    char* ws = reinterpret_cast<char*>(workspace);
    g.tickets = reinterpret_cast<unsigned int*>(ws);
    g.part = reinterpret_cast<uint64_t*>(ws ? ws + q.part_off : nullptr);
    g.lda = lda; g.ldw = ldw; g.ldy = ldy;
    g.M = (int)M; g.N = (int)N;
    g.a_per_tensor = a_per_tensor; g.w_per_tensor = w_per_tensor; g.out_f32 = out_f32;
    g.m_tiles = q.m_tiles; g.n_tiles = q.n_tiles; g.splits = q.splits; g.ksteps = (int)(K / kGemmBK);
    g.group_m = q.group_m;
    g.krot_on = q.krot_on;
    const int epi = silu_inter > 0 ? 3 : stats_mode;
    if (!far) {
        switch (q.kind) {
            case 0: return launch_gemm_kind<0>(epi, g, stream);
            case 1: return launch_gemm_kind<1>(epi, g, stream);
            case 2: return launch_gemm_kind<2>(epi, g, stream);
            case 3: return launch_gemm_kind<3>(epi, g, stream);
            case 4: return launch_gemm_kind<4>(epi, g, stream);
            case 5: return launch_gemm_kind<5>(epi, g, stream);
            case 6: return launch_gemm_kind<6>(epi, g, stream);
            case 7: return launch_gemm_kind<7>(epi, g, stream);
            case 8: return launch_gemm_kind<8>(epi, g, stream);
            case 9: return launch_gemm_kind<9>(epi, g, stream);
            case 10: return launch_gemm_kind<10>(epi, g, stream);
            case 11: return launch_gemm_kind<11>(epi, g, stream);
            case 12: return launch_gemm_kind<12>(epi, g, stream);
            default: return hipErrorInvalidValue;
        }
        static_assert(kTileKinds == 13, "every tile kind has a case");
    }
    // Rows of a tile that lie more than 4 GiB apart: the kernel with 64-bit
    // offsets, then the statistics (in the plan's groups) from its logits.
    // p's kind never splits K where a statistics or SiLU epilogue runs.
    hipError_t e = launch_gemm_far(epi == 3 ? 3 : 0, g, stream);
    if (e != hipSuccess || stats_mode == 0) return e;
    const int64_t cols = tile_bn(p.kind) / kTiles[p.kind].wn;
    const int64_t items = M * p.stat_groups;
    const dim3 grid((unsigned)(items < kGroupStatsWaves ? items : kGroupStatsWaves));
    if (stats_mode == 1)
        hipLaunchKernelGGL(logit_group_stats_kernel<1>, grid, dim3(64), 0, stream, g, p.stat_groups, cols);
    else hipLaunchKernelGGL(logit_group_stats_kernel<2>, grid, dim3(64), 0, stream, g, p.stat_groups, cols);
    return hipGetLastError();
}

}  // namespace specfp8
