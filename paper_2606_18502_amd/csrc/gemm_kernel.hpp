// Device code of the W8A8 FP8 GEMM for gfx950: Y = (A W^T) * sa[m] * sw[n], fp32
// accumulation.  Instantiated, a few tile kinds each, by the gemm_k*.hip units
// (one unit for all kernels compiles for minutes).
//
// Operands are E4M3 bytes, both K-contiguous (A [M,K] activations, W [N,K]
// weights).  The inner product runs on the CDNA4 matrix cores:
// v_mfma_f32_16x16x128_f8f6f4 multiplies a 16x128 by a 128x16 E4M3 tile into
// 16x16 fp32 accumulators (E4M3 products are exact; the hardware accumulates
// in fp32).  W takes the instruction's "row" operand and A its "column"
// operand, so the 4 accumulators a lane holds are 4 consecutive output
// channels n of one token row m.
//
// Data movement per K-step of 128 bytes:
//  * the workgroup's A tile (BM rows) and W tile (BN rows) are copied from
//    global memory straight into LDS with global_load_lds_dwordx4 (no VGPR
//    staging): one wave instruction moves 8 rows x 128 bytes = 1 KiB.  The
//    loads take the scalar-base form: the K-step's first bytes of A and W are
//    scalars, each lane keeps one 32-bit offset per load for the whole K loop
//    (a load is then one scalar move and one instruction; with 64-bit lane
//    addresses the four waves of a CU delivered 35 B/ns, with this form
//    50-75 B/ns in a loads-only probe);
//  * inside LDS each 128-byte row holds its eight 16-byte chunks in XOR-
//    swizzled slots (slot = chunk ^ swz(row)); the swizzle is applied on the
//    global side, so global reads stay fully coalesced, and the MFMA operand
//    reads (ds_read_b128, lane l reading logical chunk 2(l/16) + h of row
//    l % 16) put the lanes that one LDS cycle serves on distinct banks;
//  * STAGES buffers rotate.  A K-step's operand fragments live in registers
//    and are refilled in place for the next step, so a stage is free for the
//    loads of step it + STAGES as soon as step `it` starts.  The last STAGES
//    steps issue no loads.
//
// Two step schedules:
//  * small tiles (kstep): every fragment is refilled after its last MFMA; the
//    loads bound these tiles, so the wait for the last fragments is hidden by
//    the other workgroups of the CU;
//  * large tiles (kstep_large): the order of the MFMAs alternates between
//    W-block-major and A-block-major steps.  In either order the outer blocks
//    die early and the inner ones in the last round; the next step, in the
//    other order, needs the late ones one at a time over its whole length, so
//    no step waits for its last LDS reads (with one order for every step that
//    wait cost about 250 of 2,900 cycles per step).
//
// K is split across workgroups (split-K) when there are fewer output tiles
// than compute units.  The fp32 partial tiles are then added in split order
// (deterministic) by the last of the waves that hold the same part of the
// tile, which then applies the epilogue.
// Workgroup ids are remapped so that the tiles and K-splits that share
// operands run on the same XCD (blocks are dealt round-robin to the 8 XCDs),
// which keeps re-read operand bytes in that XCD's L2.
//
// Epilogue variants (a template argument, so each is its own kernel):
//  0  the scaled output, bf16 or fp32 (after the split-K reduction);
//  1  bf16 logits plus per-row softmax statistics of the stored values over
//     each wave's columns (the LM head of the verify pass);
//  2  bf16 logits plus per-row (max, lowest column) over each wave's columns;
//  3  the SiLU-gated FFN output h = bf16(silu(gate) * up) from a weight tile
//     whose 16-row blocks pair 8 gate rows with the matching 8 up rows.
#pragma once

#include <utility>

#include "device_common.hpp"
#include "kernels.hpp"
#include "plan.hpp"

namespace specfp8 {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct GemmArgs {
    const uint8_t* a;
    const uint8_t* w;
    const float* sa;
    const float* sw;
    void* y;
    uint64_t* part;   // split K: per tile, split and wave the accumulators of its lanes (two 8-byte halves each)
    unsigned int* tickets;   // split K: one per tile and wave, zero between calls
    float2* stats;    // [M][ld_stats] column-group statistics of the bf16 output (epilogues 1 and 2)
    int64_t lda, ldw, ldy, ld_stats;
    int M, N;
    int a_per_tensor, w_per_tensor, out_f32;
    int m_tiles, n_tiles, splits, ksteps;
    float c2;         // epilogue 1: t = z * c2
    int silu_inter;   // > 0: SiLU-gated output of I = silu_inter columns from W = [gate; up] (N = 2I)
    int group_m;      // > 1: tiles are ordered in groups of group_m M-tiles that walk the N-tiles together
    int krot_on;      // 1: blocks of columns start K at staggered steps (gemm_k_start)
};

// The kernel of a kind for an epilogue (instantiated in the gemm_k*.hip units).
template <int KIND>
hipError_t launch_gemm_kind(int epi, const GemmArgs& g, hipStream_t stream);
// Operand rows of any stride (kFarKind's tile; epilogues 0 and 3, K not split).
hipError_t launch_gemm_far(int epi, const GemmArgs& g, hipStream_t stream);

namespace {

constexpr int kBK = kGemmBK;   // bytes (= E4M3 elements) of K per step
constexpr int kXcds = 8;

// Weight row of logical output column n.  With the SiLU-gated epilogue every
// 16-row block of the weight tile pairs 8 gate rows with the matching 8 up
// rows (logical block b holds gate c, up c for c = 8b .. 8b+7), so that one
// lane exchange brings each h column's gate and up accumulators together.
__device__ __forceinline__ int w_row(const GemmArgs& g, int n) {
    if (g.silu_inter == 0) return n;
    const int c = (n >> 4) * 8 + (n & 7);
    return (n & 8) ? g.silu_inter + c : c;
}

__device__ __forceinline__ int xcd_remap(int b, int total) {
    // Blocks are dealt to XCDs round-robin (block b -> XCD b % 8).  Give each
    // XCD a contiguous range of logical ids.
    const int xcd = b % kXcds, idx = b / kXcds;
    const int per = total / kXcds, rem = total % kXcds;
    return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

// LDS swizzle.  gfx950's LDS has 64 banks of 4 bytes (256 bytes per cycle),
// so a ds_read_b128 takes at least 4 cycles, 16 lanes per cycle; the lanes
// served together are l and l + 16 for l % 16 < 8 (lanes 0-7 with 16-23,
// 8-15 with 24-31, 32-39 with 48-55, 40-47 with 56-63): a control kernel
// reading 16 contiguous bytes per lane counts no conflict, and the operand
// read counted 4 conflict cycles of 8 under a swizzle that only kept lanes
// 0-15 apart.  Rows are 128 bytes, so rows r and r^1 share a 256-byte bank
// line (their chunks land in the two halves); lanes l and l + 16 read rows
// 0-7 (or 8-15) at chunks differing by 2, so the XOR masks of the four row
// pairs must form a set F with F and F ^ 2 disjoint: F = {0, 1, 4, 5}.  Every
// cycle's 16 lanes then hit 16 different 16-byte bank groups.
__device__ __forceinline__ int swz(int row) { return (0x5410 >> (4 * ((row >> 1) & 3))) & 0xf; }

// vmcnt(N) with lgkmcnt/expcnt left alone (vmcnt field: bits [3:0] and [15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}


template <int KIND>
struct Cfg {
    static constexpr TileShape T = kTiles[KIND];
    static constexpr int WTM = T.wtm, WTN = T.wtn, WM = T.wm, WN = T.wn, STAGES = T.stages;
    static constexpr int kWaves = WM * WN;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int BM = 16 * WTM * WM;
    static constexpr int BN = 16 * WTN * WN;
    static constexpr int kRows = BM + BN;
    static constexpr int kGroups = kRows / 8;                   // 1 KiB load groups per stage
    static constexpr int kG = (kGroups + kWaves - 1) / kWaves;  // loads per wave and stage (the last ones may repeat)
    static constexpr int kStageBytes = kRows * kBK;
    static constexpr int kMfma = WTM * WTN;                     // per wave and K-step
    static constexpr int kDelay = kMfma < 2 ? kMfma : 2;        // MFMAs between a fragment's last use and its refill
    static constexpr bool kLarge = T.t1 > 0;
    // Large tiles: before MFMA kT1 every fragment of this step has been read (its stage is free), before MFMA kT2 the
    // next step's stage has landed.  With two stages kT2 lies later: a load then has up to 1.4 steps to land instead
    // of one (down at M = 4096: 182 -> 171 us).
    static constexpr int kT1 = T.t1;
    static constexpr int kT2 = STAGES == 2 && kMfma * T.late8 / 8 > kT1 ? kMfma * T.late8 / 8 : kT1;
    // MFMA before which load q of a step goes out: spread over lspan8/8 of the step
    static constexpr int kLSpan = (kMfma * T.lspan8 + 7) / 8;
    static constexpr int load_at(int q) { return kT1 + (q * kLSpan) / kG; }
    static constexpr int loads_before(int t) {
        int n = 0;
        for (int q = 0; q < kG; ++q) n += load_at(q) < t;
        return n;
    }
    // Large tiles, refill order of a step of order P (0: W blocks outer, A blocks inner; 1: the roles swapped): the
    // outer blocks but the last, then the inner blocks but the last two; the remaining three carry over into the next
    // step.  rd_at is the MFMA after which unit u goes out: kDelay after its last use, not before kT2, one per MFMA.
    static constexpr int outers(int P) { return P == 0 ? WTN : WTM; }
    static constexpr int inners(int P) { return P == 0 ? WTM : WTN; }
    static constexpr int units(int P) { return outers(P) - 1 + inners(P) - 2; }
    static constexpr int rd_at(int P, int u) {
        int t = -1;
        for (int x = 0; x <= u; ++x) {
            const int dead = x < outers(P) - 1 ? x * inners(P) + inners(P) - 1
                                               : (outers(P) - 1) * inners(P) + (x - (outers(P) - 1));
            int y = dead + kDelay;
            if (y < kT2) y = kT2;
            if (y < t + 1) y = t + 1;
            if (y > kMfma - 1) y = kMfma - 1;
            t = y;
        }
        return t;
    }
    // Staged bf16 epilogue: the tile in LDS, rows padded by 16 bytes so that the 8-byte writes and 16-byte reads of a
    // wave hit distinct banks.
    static constexpr int kPitch = BN * 2 + 16;
    static constexpr int kStagingBytes = BM * kPitch;
    static_assert(kRows % 16 == 0, "tile rows must be multiples of 16");
    static_assert((STAGES - 1) * kG < 64, "vmcnt range");
    static_assert(STAGES >= 2, "the refilled stage is not the one read next");
    static_assert(!kLarge || load_at(kG - 1) < kMfma, "every load within the step");
    static_assert(!kLarge || (WTM >= 4 && WTN >= 4 && kT1 >= 2 && kT1 < WTM && kT1 < WTN && kT2 < kMfma),
                  "alternating schedule");
};

// One load group (8 rows x 128 bytes) from base + off (base: the K-step's
// first byte of A or W, a scalar; off: this lane's row and chunk) to LDS at
// m0.  Inline asm to get the scalar-base form; the issuing code waits for it
// with explicit vmcnt waits.
__device__ __forceinline__ void stage_load(const uint8_t* base, uint32_t off, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(lds) : "memory");
}

// The same from a 64-bit lane address (operand rows too far apart for 32-bit offsets).
__device__ __forceinline__ void stage_load_far(const uint8_t* src, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "{m0}"(lds) : "memory");
}

// One scale per lane to LDS (64 consecutive floats).
__device__ __forceinline__ void scale_load(const float* src, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "{m0}"(lds) : "memory");
}

// ds_read_b128 at vaddr + OFF (an immediate).  Inline asm so that the compiler
// does not take it for a reader of the loads still in flight for other stages
// (it would drain them all); completion is awaited explicitly.
template <int OFF>
__device__ __forceinline__ u32x4 lds_read_imm(uint32_t vaddr) {
    static_assert(OFF >= 0 && OFF < 65536, "ds offset range");
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(vaddr), "n"(OFF));
    return v;
}

// The 16x128 operand block b (16 rows from the wave's first row of A or W,
// plus 16 b) of this lane: row r16 = lane % 16 of the block, logical chunks
// 2 kg, 2 kg + 1 (kg = lane / 16).  All blocks of a wave share the row bits
// that decide the swizzle, so each lane's two addresses are fixed per stage
// and the block is an immediate offset of 16 rows x 128.
template <int B>
__device__ __forceinline__ v8i block_frag(const uint32_t (&base)[2]) {
    const u32x4 lo = lds_read_imm<B * 2048>(base[0]);
    const u32x4 hi = lds_read_imm<B * 2048>(base[1]);
    return __builtin_bit_cast(v8i, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Operand fragments of one K-step held in registers.
template <int WTM, int WTN>
struct Frags {
    v8i a[WTM];
    v8i w[WTN];
};

// This lane's LDS read addresses of the A and W fragments in one stage.
struct ReadAt {
    uint32_t a[2], w[2];
};

// f(std::integral_constant<int, I>{}) for I = 0 .. N-1, in order, each I a
// compile-time constant (an immediate LDS offset, a fragment index).
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ void lds_wait_all() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// No use of the fragments may move above the wait that precedes this.
template <int WTM, int WTN>
__device__ __forceinline__ void pin_frags(Frags<WTM, WTN>& f) {
#pragma unroll
    for (int x = 0; x < WTM; ++x) asm volatile("" : "+v"(f.a[x]));
#pragma unroll
    for (int x = 0; x < WTN; ++x) asm volatile("" : "+v"(f.w[x]));
}

// Ends the accumulators' live ranges around the K loop.  Without it their
// registers in the loop follow those before and after it, and the compiler
// rotated them by copies in every step of the 64x128 SiLU and the 160x64 and
// 80x128 kernels, each copy waiting for the MFMA before it (SiLU-gated
// M = 200, 2I = 7168, K = 8192: 33.4 us, 27.5 without).  The other small kernels
// have no such copies and are left as they are.
template <int WTM, int WTN>
__device__ __forceinline__ void pin_acc(v4f (&acc)[WTN][WTM]) {
#pragma unroll
    for (int i = 0; i < WTN; ++i)
#pragma unroll
        for (int j = 0; j < WTM; ++j) asm volatile("" : "+a"(acc[i][j]));
}

// One K-step of a small tile: the fragments of step it are in f.  NEXT: there
// is a step it+1; its stage has landed once at most AFTER stages of later
// loads are in flight, and its fragments (at `nx`) replace f's after their
// last use.  issue(q): this wave's load q of step it + STAGES (LOADS), into
// the stage that held step it -- every wave has it in f after the barrier.
template <class C, bool LOADS, bool NEXT, int AFTER, class Issue>
__device__ __forceinline__ void kstep(Issue issue, const ReadAt& nx, v4f (&acc)[C::WTN][C::WTM],
                                      Frags<C::WTM, C::WTN>& f) {
    constexpr int WTM = C::WTM, WTN = C::WTN, kMfma = C::kMfma, kDelay = C::kDelay;
    if constexpr (NEXT) wait_vmcnt<(AFTER > 0 ? AFTER : 0) * C::kG>();
    if constexpr (NEXT || LOADS) __builtin_amdgcn_s_barrier();
    // W block i after its last MFMA (i WTM + WTM - 1), A block j after its last
    // one ((WTN - 1) WTM + j), each kDelay MFMAs later; the last W block at the end
    auto refill = [&](auto td_c) {
        constexpr int td = decltype(td_c)::value;
        if constexpr (td % WTM == WTM - 1 && td / WTM < WTN - 1) f.w[td / WTM] = block_frag<td / WTM>(nx.w);
        if constexpr (td >= (WTN - 1) * WTM) f.a[td - (WTN - 1) * WTM] = block_frag<td - (WTN - 1) * WTM>(nx.a);
    };
    static_for<kMfma>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int i = t / WTM, j = t % WTM;
        if constexpr (LOADS) {
            static_for<C::kG>([&](auto qc) {
                if constexpr (C::load_at(decltype(qc)::value) == t) issue(qc);
            });
        }
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f.w[i], f.a[j], acc[i][j], 0, 0, 0, 0, 0, 0);
        if constexpr (NEXT && t >= kDelay) refill(std::integral_constant<int, t - kDelay>{});
        __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (NEXT) {
        // the fragments whose last MFMAs issued just now (wait states first,
        // so that those MFMAs have read their operands)
        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
        static_for<kDelay>(
            [&](auto dc) { refill(std::integral_constant<int, kMfma - kDelay + decltype(dc)::value>{}); });
        f.w[WTN - 1] = block_frag<WTN - 1>(nx.w);
        lds_wait_all();
        pin_frags(f);
    }
}

// One K-step of a large tile, in MFMA order P (0: W blocks outer, 1: A blocks
// outer); consecutive steps alternate.  On entry the reads of this step's
// fragments are in flight, but for the three that carry over from the
// previous step (order 1 - P): its last-but-one inner block, its last outer
// and its last inner one, which go out after MFMAs 0 and 1 from `at` (this
// step's stage, still intact: it is refilled only after the barrier at kT1).
template <class C, int P, bool LOADS, bool NEXT, int AFTER, class Issue>
__device__ __forceinline__ void kstep_large(Issue issue, const ReadAt& at, const ReadAt& nx,
                                            v4f (&acc)[C::WTN][C::WTM], Frags<C::WTM, C::WTN>& f) {
    constexpr int WTM = C::WTM, WTN = C::WTN, kMfma = C::kMfma, T1 = C::kT1, T2 = C::kT2;
    constexpr int kOut = C::outers(P), kIn = C::inners(P);
    // this order's first outer block and its inner blocks but the last must be
    // there; the previous step's inner blocks 1 .. n-3, read after them, may
    // still be in flight (LDS reads complete in order; the counter holds 15)
    constexpr int kLater = 2 * (C::inners(1 - P) - 3);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(kLater > 14 ? 14 : kLater) : "memory");
    asm volatile("" : "+v"(f.a[0]));
    asm volatile("" : "+v"(f.w[0]));
    if constexpr (P == 0) {
#pragma unroll
        for (int x = 1; x < kIn - 1; ++x) asm volatile("" : "+v"(f.a[x]));
    } else {
#pragma unroll
        for (int x = 1; x < kIn - 1; ++x) asm volatile("" : "+v"(f.w[x]));
    }
    auto read_outer = [&](auto xc, const ReadAt& r) {
        constexpr int x = decltype(xc)::value;
        if constexpr (P == 0) f.w[x] = block_frag<x>(r.w);
        else f.a[x] = block_frag<x>(r.a);
    };
    auto read_inner = [&](auto xc, const ReadAt& r) {
        constexpr int x = decltype(xc)::value;
        if constexpr (P == 0) f.a[x] = block_frag<x>(r.a);
        else f.w[x] = block_frag<x>(r.w);
    };
    static_for<kMfma>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int i = P == 0 ? t / WTM : t % WTN, j = P == 0 ? t % WTM : t / WTN;
        if constexpr (t == T1) {
            lds_wait_all();
            pin_frags(f);
            if constexpr (NEXT && T2 == T1) wait_vmcnt<(C::STAGES == 2 ? 0 : (AFTER > 0 ? AFTER : 0) * C::kG)>();
            if constexpr (LOADS || (NEXT && T2 == T1)) __builtin_amdgcn_s_barrier();
        }
        if constexpr (NEXT && t == T2 && T2 != T1) {
            wait_vmcnt<(LOADS ? C::loads_before(t) : 0)>();
            __builtin_amdgcn_s_barrier();
        }
        if constexpr (LOADS) {
            static_for<C::kG>([&](auto qc) {
                if constexpr (C::load_at(decltype(qc)::value) == t) issue(qc);
            });
        }
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f.w[i], f.a[j], acc[i][j], 0, 0, 0, 0, 0, 0);
        // carried over: the previous step's inner blocks are this step's outer ones
        if constexpr (t == 0) read_outer(std::integral_constant<int, kOut - 2>{}, at);
        if constexpr (t == 1) {
            read_inner(std::integral_constant<int, kIn - 1>{}, at);
            read_outer(std::integral_constant<int, kOut - 1>{}, at);
        }
        if constexpr (NEXT) {
            static_for<C::units(P)>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                if constexpr (C::rd_at(P, u) == t) {
                    if constexpr (u < kOut - 1) read_outer(std::integral_constant<int, u>{}, nx);
                    else read_inner(std::integral_constant<int, u - (kOut - 1)>{}, nx);
                }
            });
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

__device__ __forceinline__ bool beats(float v, int i, float bv, int bi) {
    return v > bv || (v == bv && i < bi);
}

// Merge of two (max, sum) pairs; (-inf, 0) is the empty pair.
__device__ __forceinline__ void online_merge(float& m, float& s, float om, float os) {
    const float M = fmaxf(m, om);
    if (M == -INFINITY) return;
    s = (m == -INFINITY ? 0.0f : s * __builtin_amdgcn_exp2f(m - M)) +
        (om == -INFINITY ? 0.0f : os * __builtin_amdgcn_exp2f(om - M));
    m = M;
}

// The 4 lanes r16 + 16 kg that share a row combine their statistics by two
// xor shuffles in a fixed order; lane kg = 0 stores the row's entry of
// column group `col` (rows from mrow0 + 16 j + r16).  Empty groups hold
// (-inf, 0) (STATS 1) or (-inf, INT_MAX bits) (STATS 2).
template <int WTM, int STATS>
__device__ __forceinline__ void stats_store(const GemmArgs& g, const float (&sm)[WTM], const float (&ss)[WTM], int mrow0,
                                            int lane, int64_t col) {
    const int kg = lane >> 4;
    const int r16 = lane & 15;
#pragma unroll
    for (int j = 0; j < WTM; ++j) {
        float m1 = sm[j], s1 = ss[j];
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            const float m2 = __shfl_xor(m1, o, 64);
            const float s2 = __shfl_xor(s1, o, 64);
            if (STATS == 2) {
                if (beats(m2, __float_as_int(s2), m1, __float_as_int(s1))) { m1 = m2; s1 = s2; }
            } else {
                online_merge(m1, s1, m2, s2);
            }
        }
        const int m = mrow0 + j * 16 + r16;
        if (kg == 0 && m < g.M) g.stats[(int64_t)m * g.ld_stats + col] = make_float2(m1, s1);
    }
}


// y = fl32(fl32(acc * sa) * sw) of two neighbouring outputs, rounded to bf16
// (RNE, in hardware) and packed.
__device__ __forceinline__ uint32_t scaled_bf16x2(float a0, float a1, float sa, float s0, float s1) {
    return f32_to_bf16x2((a0 * sa) * s0, (a1 * sa) * s1);
}

// Direct epilogue: the 16x16 blocks of one wave's tile, stored from the MFMA
// layout (lane holds D[n = 4*(lane/16) + r][m = lane%16] of each block).
// EDGE: the tile crosses the last row or column, so every store is
// bounds-checked.  Plain output bf16 (8 bytes per lane and block) or fp32 (16
// bytes); SILU: the tile's weight rows pair gate and up rows (w_row), and each
// lane pair kg, kg ^ 2 of a block exchanges its bf16-rounded values, so lanes
// kg < 2 store h = bf16(silu(gate) * up) for 4 consecutive h columns: exactly
// what the bf16 output followed by the SiLU-gated quantize's input step gives
// for the same accumulators.
template <int WTM, int WTN, bool SILU, bool EDGE>
__device__ __forceinline__ void store_blocks(const GemmArgs& g, const v4f (&acc)[WTN][WTM], const float (&sa)[WTM],
                                             const float (&sw)[WTN][4], int m0, int n0, int wm, int wn, int lane) {
    const int kg = lane >> 4;
    const int r16 = lane & 15;
    if (!SILU && g.out_f32) {
#pragma unroll
        for (int j = 0; j < WTM; ++j) {
            const int m = m0 + (wm * WTM + j) * 16 + r16;
            float* row = reinterpret_cast<float*>(g.y) + (int64_t)m * g.ldy;
#pragma unroll
            for (int i = 0; i < WTN; ++i) {
                const int n = n0 + (wn * WTN + i) * 16 + 4 * kg;
                float y[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] = (acc[i][j][r] * sa[j]) * sw[i][r];
                if (!EDGE || n + 3 < g.N) {
                    if (!EDGE || m < g.M) *reinterpret_cast<float4*>(row + n) = make_float4(y[0], y[1], y[2], y[3]);
                } else if (m < g.M) {
                    for (int r = 0; r < 4 && n + r < g.N; ++r) row[n + r] = y[r];
                }
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < WTM; ++j) {
        const int m = m0 + (wm * WTM + j) * 16 + r16;
        uint16_t* row = reinterpret_cast<uint16_t*>(g.y) + (int64_t)m * g.ldy;
#pragma unroll
        for (int i = 0; i < WTN; ++i) {
            const int n = n0 + (wn * WTN + i) * 16 + 4 * kg;
            uint2 o;
            o.x = scaled_bf16x2(acc[i][j][0], acc[i][j][1], sa[j], sw[i][0], sw[i][1]);
            o.y = scaled_bf16x2(acc[i][j][2], acc[i][j][3], sa[j], sw[i][2], sw[i][3]);
            if constexpr (SILU) {
                // lanes 16 kg + r16 with kg < 2 hold the gate of h columns
                // (n - n0') / 2 + 4 kg + r (n0' = the block's first logical
                // column), lanes with kg >= 2 the matching up values
                const float y[4] = {__uint_as_float(o.x << 16), __uint_as_float(o.x & 0xffff0000u),
                                    __uint_as_float(o.y << 16), __uint_as_float(o.y & 0xffff0000u)};
                float up[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) up[r] = __shfl_xor(y[r], 32, 64);
                const int hc = (n0 + (wn * WTN + i) * 16) / 2 + 4 * kg;    // first h column of this lane
                if (kg < 2 && (!EDGE || (m < g.M && hc < g.silu_inter))) {
                    o.x = silu_mul_bf16x2(y[0], up[0], y[1], up[1]);
                    o.y = silu_mul_bf16x2(y[2], up[2], y[3], up[3]);
                    *reinterpret_cast<uint2*>(row + hc) = o;
                }
            } else if (!EDGE || n + 3 < g.N) {
                if (!EDGE || m < g.M) *reinterpret_cast<uint2*>(row + n) = o;
            } else if (m < g.M) {
                const uint32_t w[2] = {o.x, o.y};
                for (int r = 0; r < 4 && n + r < g.N; ++r) row[n + r] = (uint16_t)(w[r >> 1] >> (16 * (r & 1)));
            }
        }
    }
}

// Staged bf16 epilogue: the workgroup puts its tile into LDS (the K loop's
// stages are no longer read), then writes it out in 16-byte chunks, row by
// row, so that whole row segments of BN columns leave the CU at once.
// (Written from the MFMA layout, a row's cache line is filled 32 bytes at a
// time over the whole epilogue and can be written back several times while
// the other workgroups of the XCD stream their operands.)  The stores are
// nontemporal: the output would otherwise be allocated in, and written back
// through, the caches the operand streams use, and its last part only when
// the kernel ends (gate|up at M = 320 45.0 -> 43.6 us, up at M = 4096 201 ->
// 198 us).  EDGE: rows >= M and columns >= N are neither stored nor counted.
//
// STATS 1, 2 (the LM head): after its stores, every lane reads back from LDS
// the 4 WTN consecutive columns kg * 4 WTN ... of row 16 j + r16 of its wave's
// block, for every row block j, and forms their statistics: STATS 1 the
// maximum t = fl32(z * c2) first, then the sum of 2^(t - max); STATS 2 the
// maximum z and its lowest column (columns visited in increasing order, a
// strict comparison).  stats_store then combines the 4 lanes of a row, so
// each wave writes the statistics of its 16 WTN columns (one column group).
template <class C, int STATS, bool EDGE>
__device__ __forceinline__ void store_staged(const GemmArgs& g, const v4f (&acc)[C::WTN][C::WTM], const float* s_scale,
                                             int m0, int n0, int wm, int wn, int tid, int lane, const char* lds,
                                             int64_t col_group) {
    constexpr int WTM = C::WTM, WTN = C::WTN, kPitch = C::kPitch;
    const int kg = lane >> 4;
    const int r16 = lane & 15;
    const uint32_t base = lds_addr(lds);
    const uint32_t mine = base + (uint32_t)((wm * WTM * 16 + r16) * kPitch + wn * WTN * 32);   // row r16, column 0
    float sa[WTM];
#pragma unroll
    for (int j = 0; j < WTM; ++j) sa[j] = s_scale[(wm * WTM + j) * 16 + r16];
#pragma unroll
    for (int i = 0; i < WTN; ++i) {
        const float4 sw = *reinterpret_cast<const float4*>(s_scale + C::BM + (wn * WTN + i) * 16 + 4 * kg);
#pragma unroll
        for (int j = 0; j < WTM; ++j) {
            const uint32_t lo = scaled_bf16x2(acc[i][j][0], acc[i][j][1], sa[j], sw.x, sw.y);
            const uint32_t hi = scaled_bf16x2(acc[i][j][2], acc[i][j][3], sa[j], sw.z, sw.w);
            const uint32_t a = mine + (uint32_t)(j * 16 * kPitch + i * 32 + kg * 8);
            asm volatile("ds_write_b64 %0, %1" ::"v"(a), "v"((uint64_t)lo | ((uint64_t)hi << 32)) : "memory");
        }
    }
    lds_wait_all();
    __builtin_amdgcn_s_barrier();          // the tile is in LDS
    constexpr int kChunks = C::BN / 8;     // 16-byte chunks per row
    constexpr int kTotal = C::BM * kChunks;
    auto put = [&](int c, const u32x4& v) {
        const int64_t m = m0 + c / kChunks;
        const int n = n0 + (c % kChunks) * 8;
        uint16_t* dst = reinterpret_cast<uint16_t*>(g.y) + m * g.ldy + n;
        if (!EDGE || (m < g.M && n + 7 < g.N)) {
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
        } else if (m < g.M) {
            const uint32_t w[4] = {v[0], v[1], v[2], v[3]};
            for (int e = 0; e < 8 && n + e < g.N; ++e) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
        }
    };
    constexpr int kU = 4;                  // chunks per thread in flight
#pragma unroll 1
    for (int c0 = tid; c0 < kTotal; c0 += kU * C::kThreads) {
        u32x4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int c = min(c0 + u * C::kThreads, kTotal - 1);
            const uint32_t a = base + (uint32_t)((c / kChunks) * kPitch + (c % kChunks) * 16);
            asm volatile("ds_read_b128 %0, %1" : "=v"(v[u]) : "v"(a));
        }
        lds_wait_all();
#pragma unroll
        for (int u = 0; u < kU; ++u) asm volatile("" : "+v"(v[u]));   // no use moves above the wait
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (c0 + u * C::kThreads < kTotal) put(c0 + u * C::kThreads, v[u]);
    }
    if constexpr (STATS == 1 || STATS == 2) {
        static_assert(WTN % 2 == 0, "a lane's columns are whole 16-byte chunks");
        constexpr int kLaneCols = 4 * WTN;
        constexpr int kLaneChunks = kLaneCols / 8;
        const int c0 = n0 + wn * WTN * 16 + kg * kLaneCols;    // this lane's first column
        float sm[WTM], ss[WTM];
#pragma unroll 1
        for (int j = 0; j < WTM; ++j) {
            u32x4 v[kLaneChunks];
#pragma unroll
            for (int q = 0; q < kLaneChunks; ++q)
                asm volatile("ds_read_b128 %0, %1"
                             : "=v"(v[q])
                             : "v"(mine + (uint32_t)(j * 16 * kPitch + kg * kLaneCols * 2 + q * 16)));
            lds_wait_all();
            // the values are read only now: no use may move above the wait
#pragma unroll
            for (int q = 0; q < kLaneChunks; ++q) asm volatile("" : "+v"(v[q]));
            auto z_of = [&](int q, int e) {
                return __uint_as_float(((e & 1) ? v[q][e >> 1] : v[q][e >> 1] << 16) & 0xffff0000u);
            };
            if constexpr (STATS == 1) {
                float zmax = -INFINITY;
#pragma unroll
                for (int q = 0; q < kLaneChunks; ++q)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (!EDGE || c0 + q * 8 + e < g.N) zmax = fmaxf(zmax, z_of(q, e));
                const float M = zmax * g.c2;                 // = max t (c2 > 0; rounding is monotone)
                float s = 0.0f;
                if (M != -INFINITY) {                        // (also where z * c2 overflows to -inf: no mass)
#pragma unroll
                    for (int q = 0; q < kLaneChunks; ++q)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (!EDGE || c0 + q * 8 + e < g.N)
                                s += __builtin_amdgcn_exp2f(z_of(q, e) * g.c2 - M);
                }
                sm[j] = M;
                ss[j] = s;
            } else {
                float best = -INFINITY;
                int bi = 0x7fffffff;
#pragma unroll
                for (int q = 0; q < kLaneChunks; ++q)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float z = z_of(q, e);
                        const bool gt = (!EDGE || c0 + q * 8 + e < g.N) && z > best;
                        best = gt ? z : best;
                        bi = gt ? c0 + q * 8 + e : bi;
                    }
                sm[j] = best;
                ss[j] = __int_as_float(bi);
            }
        }
        stats_store<WTM, STATS>(g, sm, ss, m0 + wm * WTM * 16, lane, col_group);
    }
}

__device__ __forceinline__ uint64_t pack2(float lo, float hi) {
    return ((uint64_t)__float_as_uint(hi) << 32) | (uint64_t)__float_as_uint(lo);
}

// Split-K reduced in the kernel, wave by wave: the waves that hold the same
// part of a tile (one per split) share a ticket.  Every wave stores its fp32
// partial with device-coherent stores (relaxed agent-scope atomics: written
// through the non-coherent caches, so a wave on any XCD reads them), waits
// until all of them are acknowledged, then takes the ticket.  The wave that
// takes the last ticket -- every other partial is then already acknowledged --
// loads them with device-coherent loads issued after the ticket returned (the
// branch depends on its value), and adds all of them in split order, its own
// from registers, so the sums do not depend on which wave arrives last.  It
// returns the ticket to zero for the next call.  Each lane stores and reloads
// exactly the accumulators it holds (one float4 per 16x16 block, as two 8-byte
// halves in separate 512-byte rows, so every store and load instruction of a
// wave is contiguous); the loads of several splits are in flight at once
// (about 128 registers of them: with one split at a time, each added one
// memory round trip, 8 splits of 64x128 tiles 9 us).
// Returns false in the waves that are not last (they are done).
template <int WTM, int WTN, int WAVES>
__device__ __forceinline__ bool reduce_last(const GemmArgs& g, v4f (&acc)[WTN][WTM], int tile, int split, int wave,
                                            int lane) {
    constexpr int kBlocks = WTM * WTN;
    constexpr size_t kWaveWords = (size_t)kBlocks * 2 * 64;      // 8-byte words of one wave's partial tile
    uint64_t* const base = g.part + ((size_t)tile * g.splits * WAVES + wave) * kWaveWords + lane;
    const size_t zstride = (size_t)WAVES * kWaveWords;
    {
        uint64_t* const mine = base + split * zstride;
#pragma unroll
        for (int i = 0; i < WTN; ++i)
#pragma unroll
            for (int j = 0; j < WTM; ++j) {
                uint64_t* p = mine + (size_t)(i * WTM + j) * 128;
                __hip_atomic_store(p, pack2(acc[i][j][0], acc[i][j][1]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(p + 64, pack2(acc[i][j][2], acc[i][j][3]), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    unsigned int* const ticket = g.tickets + tile * WAVES + wave;
    unsigned int t = 0;
    if (lane == 0) t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    t = (unsigned int)__builtin_amdgcn_readfirstlane((int)t);
    if (t != (unsigned int)(g.splits - 1)) return false;
    if (lane == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::: "memory");
    // W blocks and splits per batch of loads: about 128 registers of partials
    constexpr int IB = 4 * kBlocks <= 128 ? WTN : (WTN % 2 == 0 && 2 * kBlocks <= 128 ? WTN / 2 : 1);
    constexpr int kFit = 128 / (4 * WTM * IB);
    constexpr int ZB = kFit > 8 ? 8 : (kFit < 1 ? 1 : kFit);
#pragma unroll
    for (int i0 = 0; i0 < WTN; i0 += IB) {
        v4f tot[IB][WTM];
        for (int z0 = 0; z0 < g.splits; z0 += ZB) {
            uint64_t lo[ZB][IB][WTM], hi[ZB][IB][WTM];
#pragma unroll
            for (int u = 0; u < ZB; ++u) {
                const int z = z0 + u;
                if (z < g.splits && z != split) {
                    const uint64_t* src = base + z * zstride + (size_t)i0 * WTM * 128;
#pragma unroll
                    for (int i = 0; i < IB; ++i)
#pragma unroll
                        for (int j = 0; j < WTM; ++j) {
                            const uint64_t* p = src + (size_t)(i * WTM + j) * 128;
                            lo[u][i][j] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            hi[u][i][j] = __hip_atomic_load(p + 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                } else {
#pragma unroll
                    for (int i = 0; i < IB; ++i)
#pragma unroll
                        for (int j = 0; j < WTM; ++j) {
                            lo[u][i][j] = pack2(acc[i0 + i][j][0], acc[i0 + i][j][1]);
                            hi[u][i][j] = pack2(acc[i0 + i][j][2], acc[i0 + i][j][3]);
                        }
                }
            }
#pragma unroll
            for (int u = 0; u < ZB; ++u) {
                const int z = z0 + u;
                if (z < g.splits) {
#pragma unroll
                    for (int i = 0; i < IB; ++i)
#pragma unroll
                        for (int j = 0; j < WTM; ++j) {
                            const uint64_t l = lo[u][i][j], h = hi[u][i][j];
                            const v4f p = {__uint_as_float((uint32_t)l), __uint_as_float((uint32_t)(l >> 32)),
                                           __uint_as_float((uint32_t)h), __uint_as_float((uint32_t)(h >> 32))};
                            tot[i][j] = z == 0 ? p : tot[i][j] + p;
                        }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int j = 0; j < WTM; ++j) acc[i0 + i][j] = tot[i][j];
    }
    return true;
}

// EPI: the epilogue (0 plain, 1 and 2 statistics, 3 SiLU-gated).  SPLIT: K is
// split (plain epilogue).  FAR: operand rows too far apart for 32-bit lane
// offsets within a tile; the addresses are recomputed in 64 bits per load.
template <int KIND, int EPI, bool SPLIT, bool FAR>
__global__ __launch_bounds__(64 * kTiles[KIND].wm * kTiles[KIND].wn) void gemm_fp8_kernel(GemmArgs g) {
    using C = Cfg<KIND>;
    constexpr int WTM = C::WTM, WTN = C::WTN, WM = C::WM, WN = C::WN, STAGES = C::STAGES;
    static_assert(!SPLIT || EPI == 0, "only the plain epilogue splits K");
    constexpr bool kStaged = EPI == 1 || EPI == 2 || (EPI == 0 && !SPLIT && C::T.staged);
    constexpr int kStageSum = STAGES * C::kStageBytes;
    constexpr int kLdsBytes = kStaged && C::kStagingBytes > kStageSum ? C::kStagingBytes : kStageSum;
    __shared__ __attribute__((aligned(1024))) char lds[kLdsBytes];
    constexpr int kScaleChunks = (C::kRows + 63) / 64;
    __shared__ __attribute__((aligned(256))) float s_scale[kScaleChunks * 64];   // scales of the tile's rows, then columns

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM;
    const int wn = wave / WM;

    // consecutive logical ids: K-splits of a tile, then M-tiles of an N-tile
    const int logical = xcd_remap(blockIdx.x, g.m_tiles * g.n_tiles * g.splits);
    const int split = SPLIT ? logical % g.splits : 0;
    const int tile = SPLIT ? logical / g.splits : logical;
    int mt, nt;
    if (g.group_m > 1) {
        // Large M: a group of group_m M-tiles walks the N-tiles, so the tiles
        // that run at once on one XCD form a group_m x (CUs / group_m) block
        // and re-read each other's operand rows from that XCD's L2.
        const int per_group = g.group_m * g.n_tiles;
        const int first = (tile / per_group) * g.group_m;
        const int gm = min(g.group_m, g.m_tiles - first);
        const int in = tile - (tile / per_group) * per_group;
        mt = first + in % gm;
        nt = in / gm;
    } else {
        mt = tile % g.m_tiles;
        nt = tile / g.m_tiles;
    }
    const int m0 = mt * C::BM;
    const int n0 = nt * C::BN;

    // this split's K-steps (shares differ by at most one)
    const int ks0 = SPLIT ? (int)((int64_t)g.ksteps * split / g.splits) : 0;
    const int nk = (SPLIT ? (int)((int64_t)g.ksteps * (split + 1) / g.splits) : g.ksteps) - ks0;
    // Blocks of columns may walk K from different starting points, so that
    // the workgroups do not all request the same K columns at once.
    const int krot = !SPLIT && g.krot_on ? gemm_k_start(n0, nk) : 0;

    // The epilogue's scales, loaded straight into LDS ahead of the operands
    // (rows and columns past the edge read a valid neighbour).
    static_for<(kScaleChunks + C::kWaves - 1) / C::kWaves>([&](auto sc) {
        const int c = wave + decltype(sc)::value * C::kWaves;
        if (c < kScaleChunks) {
            const int r = min(c * 64 + lane, C::kRows - 1);
            const float* const src = r < C::BM
                                         ? (g.a_per_tensor ? g.sa : g.sa + min(m0 + r, g.M - 1))
                                         : (g.w_per_tensor ? g.sw : g.sw + w_row(g, min(n0 + r - C::BM, g.N - 1)));
            scale_load(src, lds_addr(s_scale) + c * 256);
        }
    });

    // Load groups: this wave's group q holds the tile rows 8 grp .. 8 grp + 7
    // (A rows, then W rows; with the SiLU-gated epilogue a W group is all gate
    // or all up rows).  A lane's offset is taken from the tile's first operand
    // row of that sort; rows past the edge re-read the last row.
    const int chunk = (lane & 7) ^ swz(lane >> 3);
    auto group_of = [&](int q) {
        const int grp = wave + q * C::kWaves;
        return C::kGroups % C::kWaves == 0 ? grp : min(grp, C::kGroups - 1);
    };
    auto is_a = [&](int q) {          // the group holds A rows (known at compile time where every wave's does)
        return C::BM % (8 * C::kWaves) == 0 ? q < C::BM / (8 * C::kWaves) : group_of(q) * 8 < C::BM;
    };
    auto is_up = [&](int q) { return EPI == 3 && !is_a(q) && (group_of(q) & 1) != 0; };
    const int wfirst = EPI == 3 ? n0 / 2 : n0;   // (SiLU: the first gate row; n0 is a multiple of 16)
    const uint8_t* const a0 = g.a + (int64_t)m0 * g.lda + (int64_t)ks0 * kBK;
    const uint8_t* const w0 = g.w + (int64_t)wfirst * g.ldw + (int64_t)ks0 * kBK;
    const int64_t up_off = EPI == 3 ? (int64_t)g.silu_inter * g.ldw : 0;
    auto row_of = [&](int q) {        // operand row of this lane's part of group q, from the tile's first
        const int row = group_of(q) * 8 + (lane >> 3);
        if (is_a(q)) return min(m0 + row, g.M - 1) - m0;
        const int n = n0 + row - C::BM;
        if (EPI == 3) return min((n >> 4) * 8 + (n & 7), g.silu_inter - 1) - wfirst;   // of the gate or of the up rows
        return min(n, g.N - 1) - n0;
    };
    uint32_t off[C::kG];
    if constexpr (!FAR) {
        static_for<C::kG>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const uint32_t ld = (uint32_t)(is_a(q) ? g.lda : g.ldw);
            off[q] = (uint32_t)row_of(q) * ld + (uint32_t)(chunk * 16);
        });
    }
    const uint32_t st0 = lds_addr(lds);
    const uint8_t *abase = a0, *wbase = w0;      // first bytes of the K-step being loaded
    int lp = krot;                               // that step (rotated)
    auto advance = [&]() {
        abase = a0 + (int64_t)lp * kBK;
        wbase = w0 + (int64_t)lp * kBK;
        lp = lp + 1 == nk ? 0 : lp + 1;
    };
    auto load_group = [&](auto qc, uint32_t stage) {
        constexpr int q = decltype(qc)::value;
        const int grp = group_of(q);
        const uint8_t* const base = is_a(q) ? abase : (is_up(q) ? wbase + up_off : wbase);
        if constexpr (FAR) {
            const int64_t ld = is_a(q) ? g.lda : g.ldw;
            stage_load_far(base + (int64_t)row_of(q) * ld + chunk * 16, stage + grp * 1024);
        } else {
            stage_load(base, off[q], stage + grp * 1024);
        }
    };

    const int kg = lane >> 4, r16 = lane & 15;
    ReadAt r0;                                   // this lane's fragment addresses in stage 0
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t in_row = (uint32_t)(r16 * kBK + (((2 * kg + h) ^ swz(r16)) << 4));
        r0.a[h] = st0 + (uint32_t)(wm * WTM * 16 * kBK) + in_row;
        r0.w[h] = st0 + (uint32_t)((C::BM + wn * WTN * 16) * kBK) + in_row;
    }
    auto at_stage = [&](uint32_t s) {
        return ReadAt{{r0.a[0] + s, r0.a[1] + s}, {r0.w[0] + s, r0.w[1] + s}};
    };

    v4f acc[WTN][WTM];
#pragma unroll
    for (int i = 0; i < WTN; ++i)
#pragma unroll
        for (int j = 0; j < WTM; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // prologue: every stage in flight (with fewer K-steps than stages the rest
    // repeat the last one and are never read), then the fragments of step 0
    static_for<STAGES>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if (s < nk) advance();
        static_for<C::kG>([&](auto qc) { load_group(qc, st0 + s * C::kStageBytes); });
    });
    wait_vmcnt<(STAGES - 1) * C::kG>();
    __builtin_amdgcn_s_barrier();
    Frags<WTM, WTN> f;
    static_for<WTM>([&](auto x) { f.a[decltype(x)::value] = block_frag<decltype(x)::value>(r0.a); });
    static_for<WTN>([&](auto x) { f.w[decltype(x)::value] = block_frag<decltype(x)::value>(r0.w); });
    lds_wait_all();
    pin_frags(f);

    // step it is in stage `cur` (byte offset), step it + 1 in the next one
    uint32_t cur = 0;
    auto step = [&](auto loads, auto next, auto after, auto order) {
        constexpr bool kLoads = decltype(loads)::value, kNext = decltype(next)::value;
        uint32_t nxt = cur + C::kStageBytes;
        if (nxt == (uint32_t)kStageSum) nxt = 0;
        if constexpr (kLoads) advance();
        auto issue = [&](auto qc) { load_group(qc, st0 + cur); };
        if constexpr (C::kLarge)
            kstep_large<C, decltype(order)::value, kLoads, kNext, decltype(after)::value>(issue, at_stage(cur),
                                                                                       at_stage(nxt), acc, f);
        else
            kstep<C, kLoads, kNext, decltype(after)::value>(issue, at_stage(nxt), acc, f);
        cur = nxt;
    };
    std::true_type yes;
    std::false_type no;
    std::integral_constant<int, STAGES - 2> full;
    std::integral_constant<int, 0> p0;
    std::integral_constant<int, 1> p1;
    int it = 0;
    if constexpr (C::kLarge) {
        // steps with loads in pairs of both orders; an odd one first, in order 1
        if (nk > STAGES && ((nk - STAGES) & 1)) {
            step(yes, yes, full, p1);
            ++it;
        }
        for (; it + STAGES < nk; it += 2) {
            step(yes, yes, full, p0);
            step(yes, yes, full, p1);
        }
    } else {
        constexpr bool kPin = C::kMfma > 8 || (C::kMfma == 8 && EPI == 3);
        if constexpr (kPin) pin_acc<WTM, WTN>(acc);
        for (; it + STAGES < nk; ++it) step(yes, yes, full, p0);
        if constexpr (kPin) pin_acc<WTM, WTN>(acc);
    }
    // the last STAGES steps (nk of them if there are fewer), no loads
    static_for<STAGES>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (nk >= STAGES - j)
            step(no, std::integral_constant<bool, (j < STAGES - 1)>{}, std::integral_constant<int, STAGES - 2 - j>{},
                 std::integral_constant<int, j & 1>{});
    });
    wait_vmcnt<0>();   // no direct-to-LDS write may outlive the workgroup

    __syncthreads();   // the scales are in LDS; no stage is read any more
    if constexpr (SPLIT) {
        if (!reduce_last<WTM, WTN, C::kWaves>(g, acc, tile, split, wave, lane)) return;
    }
    const bool edge = m0 + C::BM > g.M || n0 + C::BN > g.N;
    if constexpr (kStaged) {
        if (EPI != 0 || !g.out_f32) {
            const int64_t col_group = (int64_t)nt * WN + wn;
            if (edge) store_staged<C, EPI, true>(g, acc, s_scale, m0, n0, wm, wn, tid, lane, lds, col_group);
            else store_staged<C, EPI, false>(g, acc, s_scale, m0, n0, wm, wn, tid, lane, lds, col_group);
            return;
        }
    }
    if constexpr (EPI == 0 || EPI == 3) {
        float sa[WTM], sw[WTN][4];
#pragma unroll
        for (int j = 0; j < WTM; ++j) sa[j] = s_scale[(wm * WTM + j) * 16 + r16];
#pragma unroll
        for (int i = 0; i < WTN; ++i) {
            const float4 v = *reinterpret_cast<const float4*>(s_scale + C::BM + (wn * WTN + i) * 16 + 4 * kg);
            sw[i][0] = v.x; sw[i][1] = v.y; sw[i][2] = v.z; sw[i][3] = v.w;
        }
        if (edge) store_blocks<WTM, WTN, EPI == 3, true>(g, acc, sa, sw, m0, n0, wm, wn, lane);
        else store_blocks<WTM, WTN, EPI == 3, false>(g, acc, sa, sw, m0, n0, wm, wn, lane);
    }
}

// ---- launching (the kinds and their epilogues: plan.hpp, kTiles) ---------------

template <int KIND, int EPI, bool SPLIT, bool FAR>
hipError_t launch_one(const GemmArgs& g, hipStream_t stream) {
    const dim3 grid(g.m_tiles * g.n_tiles * g.splits), block(Cfg<KIND>::kThreads);
    hipLaunchKernelGGL((gemm_fp8_kernel<KIND, EPI, SPLIT, FAR>), grid, block, 0, stream, g);
    return hipGetLastError();
}

}  // namespace

// The kernel of kind KIND for epilogue epi, if the kind has it (plan.hpp).
template <int KIND>
hipError_t launch_gemm_kind(int epi, const GemmArgs& g, hipStream_t stream) {
    constexpr int kHas = kTiles[KIND].has;
    if (g.splits > 1) {
        if constexpr ((kHas & kHasSplit) != 0)
            if (epi == 0) return launch_one<KIND, 0, true, false>(g, stream);
        return hipErrorInvalidValue;
    }
    if (epi == 0) return launch_one<KIND, 0, false, false>(g, stream);
    if constexpr ((kHas & kHasStats) != 0) {
        if (epi == 1) return launch_one<KIND, 1, false, false>(g, stream);
        if (epi == 2) return launch_one<KIND, 2, false, false>(g, stream);
    }
    if constexpr ((kHas & kHasSilu) != 0)
        if (epi == 3) return launch_one<KIND, 3, false, false>(g, stream);
    return hipErrorInvalidValue;
}

}  // namespace specfp8
