// Acceptance test of the speculative-decoding verify step.
//
// Greedy (T == 0):
//   greedy_partial_kernel  (row, slice) items -> max logit and its lowest index
//   greedy_final_kernel    b -> argmax per position, longest matching prefix
// Speculative sampling (T > 0):
//   stoch_stats_kernel     (row, slice) items -> slice max m and sum 2^(t - m) of
//                          t = z * log2(e)/T (the tempered logit in base 2), for
//                          target rows 0..k and draft rows 0..k-1
//   stoch_sample_kernel    (chunk, b) -> every block merges the slice statistics
//                          of its sequence in slice order, takes the (identical)
//                          accept/reject decisions and sums the residual
//                          distribution over its chunk's 64-element ranges;
//                          the last block of the sequence to finish (an atomic
//                          ticket) locates the range holding u*R, scans it in
//                          vocabulary order and writes the tokens.
//
// Two variants reuse these kernels:
//   target statistics given (the LM head's epilogue wrote them): the streaming
//     kernel reads only the draft rows, and the merges read the given entries
//     for the target rows (clear_tickets_kernel when nothing is streamed);
//   token trees: the streaming kernels run over the N+1 target rows of every
//     sequence, then tree_greedy_kernel / tree_sample_kernel walk the tree
//     (see the token-tree section below).
//
// The two streaming kernels run a persistent grid in which every WAVE walks
// (row, slice) items of 4096 logits with the loads of its next item in flight
// while it reduces the current one, so HBM sees one continuous stream of
// 2 bytes per logit and no item needs a workgroup barrier.  Items are strided
// over the waves, so at any moment the chip reads one contiguous stretch of
// the logit tensors.  The sample kernel re-reads only the row(s) of the
// position where sampling happens (<= 2 rows per sequence), with every load of
// a thread issued before it computes.  All reductions use a fixed order, so
// results are deterministic.
#include <atomic>
#include <mutex>
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"
#include "plan.hpp"

// Fixed acceptance scratch for callers that cannot allocate
// (spec_verify_accept_noalloc).  Each GPU holds its own copy at its own
// address; host code reaches it only through the address accept_scratch()
// looks up, never through this name (a host-side stand-in).
static __device__ __align__(256) unsigned char scratch[specfp8::kAcceptScratchBytes];

namespace specfp8 {

namespace {

constexpr int kAThreads = kAcceptThreads;
constexpr int kWavesPerBlock = kAThreads / kWave;
constexpr int kVecs = kAcceptVecs;                     // 16-byte vectors per lane per item
constexpr int64_t kSlice = kAcceptSlice;               // 4096 logits per wave item
constexpr int kPerThread = kAcceptPerThread;           // 64 logits per thread (sample kernel)
constexpr int64_t kChunk = kAcceptChunk;               // 16384 logits per sample block
static_assert(kSlice == (int64_t)kWave * kVecs * 8 && kChunk == (int64_t)kAThreads * kPerThread, "accept geometry");
constexpr int kMaxChunks = kAThreads;                 // V <= 2^22: one chunk per thread
constexpr int kStreamWavesPerCU = 12;

struct AcceptArgs {
    const uint16_t* zt;
    const uint16_t* zd;
    const int32_t* x;
    const float* u;
    int32_t* out;
    int32_t* num;
    const int32_t* parent; // token tree: parent node of each node, -1 for the root's candidates (tree mode)
    int32_t* nodes;        // token tree: accepted node indices [B][k] (tree mode)
    float2* stats;         // [B][Rs][nslice] statistics of the streamed rows
    const float2* tst;     // target rows' statistics from the LM-head epilogue, or null
    int64_t ldtst;         // row stride of tst (entries)
    uint32_t ntst;         // entries per target row in tst
    float2* tsm;           // [B][k+1] tst merged to one entry per row by the statistics kernel, or null
    float2* zx;            // [B][k] (target, draft) logits at the draft tokens, gathered by the statistics
                           // kernel for the sampling kernel, or null (no statistics pass, greedy)
    uint32_t sw;           // streaming waves of the statistics grid (the first sw waves)
    double* finem;         // [B][nchunk][256] residual mass per 64-element range
    unsigned int* ctr;     // [B]
    int64_t V, nchunk;
    uint32_t nslice, items;   // slices per row; rows * nslice (< 2^31)
    int B, k;
    uint32_t R;            // rows per sequence whose statistics are merged (k+1, or 2k+1 with draft logits)
    uint32_t Rs;           // of these, the rows the statistics kernel streams (R, or R - (k+1) with tst)
    uint32_t rt0;          // first streamed row within the sequence (0, or k+1 with tst)
    float c2;              // log2(e) / T
};

// Statistics entries of row r (0..R-1) of sequence b: the target rows from
// the LM-head epilogue when given, else (and for draft rows) the streamed ones.
__device__ __forceinline__ const float2* row_stats(const AcceptArgs& a, int b, int r, uint32_t& n) {
    if ((uint32_t)r < a.rt0) {
        if (a.tsm) {
            n = 1;
            return a.tsm + (int64_t)b * (a.k + 1) + r;
        }
        n = a.ntst;
        return a.tst + ((int64_t)b * (a.k + 1) + r) * a.ldtst;
    }
    n = a.nslice;
    return a.stats + ((int64_t)b * a.Rs + (r - (int)a.rt0)) * a.nslice;
}

using Raw = uint4[kVecs];

// Slice layout: vector j of lane l starts at element e0 + (j * 64 + l) * 8, so
// one load instruction of a wave reads 1 KiB contiguous.
__device__ __forceinline__ int64_t slice_vec(int64_t e0, int j, int lane) {
    return e0 + ((int64_t)j * kWave + lane) * 8;
}

// How the logit rows are read, 8 logits at a time:
//   kAligned  rows on 16-byte boundaries, V % 8 == 0: no group is cut
//   kLoose    any other rows of at least 8 logits: the same 16-byte loads, from
//             any 2-byte boundary (global memory takes them so); a group that
//             runs past the row's end is read from the row's last 8 logits
//   kShort    rows of fewer than 8 logits, element by element
// What bounds 2-byte loads is their count: greedy over [104, 32001] took 17.5 us
// with them and 8.3 us with kLoose.
enum RowLoad { kAligned, kLoose, kShort };
typedef unsigned int stream_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int loose_u32x4 __attribute__((ext_vector_type(4), aligned(2)));

inline RowLoad row_load(int64_t V, const void* zt, const void* zd) {
    if (V < 8) return kShort;
    return V % 8 == 0 && (uintptr_t)zt % 16 == 0 && (uintptr_t)zd % 16 == 0 ? kAligned : kLoose;
}

// The 8 logits at e of a row.  Where the group runs past e1 (or lies past it)
// the last 8 before e1 are read instead (cut8 puts a cut group right).
template <RowLoad LD, bool STREAM>
__device__ __forceinline__ uint4 load8(const uint16_t* __restrict__ row, int64_t e, int64_t e1) {
    if constexpr (LD == kShort) {
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 8; q += 2)
            w[q / 2] = (uint32_t)row[min((int64_t)q, e1 - 1)] | ((uint32_t)row[min((int64_t)q + 1, e1 - 1)] << 16);
        return make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        using Vec = std::conditional_t<LD == kAligned, stream_u32x4, loose_u32x4>;
        const Vec* p = reinterpret_cast<const Vec*>(row + min(e, e1 - 8));
        const Vec v = STREAM ? __builtin_nontemporal_load(p) : *p;
        return make_uint4(v.x, v.y, v.z, v.w);
    }
}

// Issue the loads of one slice.  Lanes past the slice's end load its last
// group; their values are masked where they are used.  The loads are nontemporal:
// the statistics pass reads each logit once, and cache-allocating loads of
// 148 MB would push the model's weights and the dirty outputs of the layer
// out of the Infinity Cache (measured in the verify step: the statistics pass
// 31.1 -> 27.0 us, the next gate|up and down GEMMs ~1 us faster each; the
// sampling kernel's re-read of the residual rows then comes from HBM).
template <RowLoad LD>
__device__ __forceinline__ void load_slice(const uint16_t* __restrict__ row, int64_t e0, int64_t e1, int lane,
                                           Raw& raw) {
#pragma unroll
    for (int j = 0; j < kVecs; ++j) raw[j] = load8<LD, true>(row, slice_vec(e0, j, lane), e1);
}

// Puts the group at e right where it is cut by e1: load8 read the last 8
// logits before e1, which are shifted down to start at e; the elements from
// e1 on become the bf16 `fill`.
template <RowLoad LD>
__device__ __forceinline__ void cut8(uint4& raw, int64_t e, int64_t e1, uint16_t fill) {
    if (LD == kAligned || e + 8 <= e1 || e >= e1) return;
    uint64_t lo = raw.x | ((uint64_t)raw.y << 32), hi = raw.z | ((uint64_t)raw.w << 32);
    const int sh = LD == kShort ? 0 : 16 * (int)(8 - (e1 - e));
    if (sh >= 64) {
        lo = hi >> (sh - 64);
    } else if (sh > 0) {
        lo = (lo >> sh) | (hi << (64 - sh));
        hi >>= sh;
    }
    const int keep = 16 * (int)(e1 - e);                     // 16 .. 112 bits
    const uint64_t f = 0x0001000100010001ull * fill;
    const uint64_t ml = keep >= 64 ? ~0ull : (1ull << keep) - 1;
    const uint64_t mh = keep > 64 ? (1ull << (keep - 64)) - 1 : 0;
    lo = (lo & ml) | (f & ~ml);
    hi = (hi & mh) | (f & ~mh);
    raw = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// cut8 over one slice's groups.
template <RowLoad LD>
__device__ __forceinline__ void cut_slice(Raw& raw, int64_t e0, int64_t e1, int lane, uint16_t fill) {
    if (LD == kAligned || e1 - e0 == kSlice) return;
#pragma unroll
    for (int j = 0; j < kVecs; ++j) cut8<LD>(raw[j], slice_vec(e0, j, lane), e1, fill);
}
constexpr uint16_t kBf16NaN = 0x7fc0, kBf16NegInf = 0xff80;

// Element e + q of a group of 8 starting at e < e1 exists (with kAligned every
// range end is a multiple of 8, so the whole group does).
template <RowLoad LD>
__device__ __forceinline__ bool in8(int64_t e, int q, int64_t e1) { return LD == kAligned || e + q < e1; }

// Workgroups of the streaming kernels: at most kStreamWavesPerCU waves per
// compute unit, the items spread so that every wave takes the same count (but
// the last).  Past one workgroup per CU the count is rounded up to a whole
// number of workgroups per CU, so every CU streams the same share: a CU
// holding one workgroup more than its neighbours sets the kernel's end
// (measured on the C4 workload: 3.6 workgroups per CU 27.9 us, exactly 3 per
// CU 25.8 us).  Waves past the last item return at once.
inline unsigned stream_blocks(int64_t items, int cus) {
    const int64_t cap = (int64_t)cus * kStreamWavesPerCU;
    const int64_t per = (items + cap - 1) / cap;
    const int64_t waves = (items + per - 1) / per;
    int64_t blocks = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > cus) blocks = (blocks + cus - 1) / cus * cus;
    return (unsigned)blocks;
}

// Persistent wave loop over items it = gw, gw + GW, ...: the slice of item
// it + GW is loaded while item it is reduced (two register buffers).  The
// wave id is read from the first lane, so the item, row and slice indices are
// known to be wave-uniform and their arithmetic runs on the scalar unit
// (C4 stochastic acceptance 46.4 -> 46.1 us).
// Only the first a.sw waves of the grid stream (workgroups past them do side
// work).
template <RowLoad LD, class RowOf, class Body>
__device__ __forceinline__ void stream_items(const AcceptArgs& a, RowOf row_of, Body body) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t gw = blockIdx.x * kWavesPerBlock + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t GW = a.sw;
    auto lo = [&](uint32_t it) { return (int64_t)(it % a.nslice) * kSlice; };
    auto hi = [&](uint32_t it) { return min(lo(it) + kSlice, a.V); };
    auto clampi = [&](uint32_t it) { return it < a.items ? it : a.items - 1; };
    if (gw >= GW || gw >= a.items) return;
    Raw r0, r1;
    load_slice<LD>(row_of(gw / a.nslice), lo(gw), hi(gw), lane, r0);
    for (uint32_t it = gw; it < a.items; it += 2 * GW) {
        const uint32_t n1 = clampi(it + GW), n2 = clampi(it + 2 * GW);
        load_slice<LD>(row_of(n1 / a.nslice), lo(n1), hi(n1), lane, r1);
        body(it, r0);
        load_slice<LD>(row_of(n2 / a.nslice), lo(n2), hi(n2), lane, r0);
        if (it + GW < a.items) body(it + GW, r1);
    }
}

// ------------------------------------------------------------------ greedy

__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
    return v > bv || (v == bv && i < bi);
}

// Lane maximum of the logits of one slice (8-element groups, v_max3 pairs).
// Elements past e1 in a cut group hold NaN, which fmaxf ignores, or -inf.
template <bool FULL>
__device__ __forceinline__ float slice_max(const Raw& raw, int64_t e0, int64_t e1, int lane) {
    float zm = -INFINITY;
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
        const int64_t e = slice_vec(e0, j, lane);
        if (FULL || e < e1) {
            float v[8];
            unpack8(raw[j], v);
#pragma unroll
            for (int q = 0; q < 8; q += 2) zm = fmaxf(fmaxf(zm, v[q]), v[q + 1]);
        }
    }
    return zm;
}

// (max logit, lowest index holding it) of one slice, reduced over the wave.
template <bool FULL>
__device__ __forceinline__ float2 slice_argmax(const Raw& raw, int64_t e0, int64_t e1, int lane) {
    const float M = wave_max(slice_max<FULL>(raw, e0, e1, lane));
    // lowest index of M in the lane: scan backwards, the last hit wins
    int bi = 0x7fffffff;
#pragma unroll
    for (int j = kVecs - 1; j >= 0; --j) {
        const int64_t e = slice_vec(e0, j, lane);
        if (FULL || e < e1) {
            float v[8];
            unpack8(raw[j], v);
#pragma unroll
            for (int q = 7; q >= 0; --q) bi = (v[q] == M) ? (int)(e + q) : bi;
        }
    }
    return make_float2(M, __int_as_float(wave_min_i32(bi)));
}

template <RowLoad LD>
__global__ __launch_bounds__(kAThreads) void greedy_partial_kernel(AcceptArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    auto row_of = [&](uint32_t row) { return a.zt + (int64_t)row * a.V; };
    stream_items<LD>(a, row_of, [&](uint32_t it, Raw& raw) {
        const uint32_t row = it / a.nslice, c = it % a.nslice;
        const int64_t e0 = (int64_t)c * kSlice, e1 = min(e0 + kSlice, a.V);
        cut_slice<LD>(raw, e0, e1, lane, kBf16NaN);
        const float2 r = (e1 - e0 == kSlice) ? slice_argmax<true>(raw, e0, e1, lane)
                                                    : slice_argmax<false>(raw, e0, e1, lane);
        if (lane == 0) a.stats[(int64_t)row * a.nslice + c] = r;
    });
}

// Entry `lane` of row r's (max logit, lowest index) statistics, or the
// neutral (-inf, INT_MAX) past the row's entries.
__device__ __forceinline__ float2 argmax_entry(const AcceptArgs& a, int b, int r, int lane) {
    uint32_t nst;
    const float2* st = row_stats(a, b, r, nst);
    return (uint32_t)lane < nst ? st[lane] : make_float2(-INFINITY, __int_as_float(0x7fffffff));
}

// Merged (max logit, lowest index) of row r of sequence b, for lanes of one
// wave; `first` is the row's entry `lane` (argmax_entry), loaded beforehand.
// The order of `better` is total, so the merge order does not matter.
__device__ __forceinline__ int merged_argmax(const AcceptArgs& a, int b, int r, int lane, float2 first) {
    uint32_t nst;
    const float2* st = row_stats(a, b, r, nst);
    float bv = first.x;
    int bi = __float_as_int(first.y);
    // the entries past the first 64 (many when they come from the LM-head
    // epilogue: 668 per row at V = 128256), 16 per lane per round trip
    for (int64_t c0 = lane + 64; c0 < nst; c0 += 16 * 64) {
        float2 pv[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int64_t c = c0 + q * 64;
            pv[q] = c < nst ? st[c] : make_float2(-INFINITY, __int_as_float(0x7fffffff));
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int pi = __float_as_int(pv[q].y);
            if (better(pv[q].x, pi, bv, bi)) { bv = pv[q].x; bi = pi; }
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    return bi;
}

__global__ __launch_bounds__(1024) void greedy_final_kernel(AcceptArgs a) {
    __shared__ int g[17], s_x[16];
    const int b = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    // the drafts are loaded first, so their round trip overlaps the merge
    const int32_t xt = t < a.k ? a.x[(int64_t)b * a.k + t] : 0;
    // wave wv merges positions wv, wv+16, ... (one round for k < 16); lanes
    // stride over the slices
    const int nw = (int)(blockDim.x >> 6);
    for (int pos = wv; pos <= a.k; pos += nw) {
        const int bi = merged_argmax(a, b, pos, lane, argmax_entry(a, b, pos, lane));
        if (lane == 0) g[pos] = bi;
    }
    if (t < a.k) s_x[t] = xt;
    __syncthreads();
    if (t <= a.k) {
        // a_b = number of leading drafts equal to the target argmax
        int acc = a.k;
        for (int i = 0; i < a.k; ++i)
            if (s_x[i] != g[i]) { acc = i; break; }
        int32_t* out = a.out + (int64_t)b * (a.k + 1);
        out[t] = t < acc ? g[t] : (t == acc ? g[acc] : -1);
        if (t == 0) a.num[b] = acc;
    }
}

// ------------------------------------------------------------- stochastic

// (m, sum 2^(t - m)) of t = z * c2 over one slice, reduced over the wave:
// the wave maximum first (c2 > 0, so max t = fl(max z * c2)), then one
// exponential per element with the wave's m, so no partial sum is rescaled.
template <bool FULL>
__device__ __forceinline__ float2 slice_stats(const Raw& raw, int64_t e0, int64_t e1, int lane,
                                              float c2) {
    const float M = wave_max(slice_max<FULL>(raw, e0, e1, lane)) * c2;
    float s = 0.0f;
    if (M != -INFINITY) {
#pragma unroll
        for (int j = 0; j < kVecs; ++j) {
            const int64_t e = slice_vec(e0, j, lane);
            if (FULL || e < e1) {
                float v[8];
                unpack8(raw[j], v);
#pragma unroll
                for (int q = 0; q < 8; ++q) s += __builtin_amdgcn_exp2f(fmaf(v[q], c2, -M));
            }
        }
    }
    return make_float2(M, wave_sum(s));
}

// Online merge of (max, sum 2^(t - max)) pairs.
__device__ __forceinline__ void merge_ms(float& m, float& z, float om, float oz) {
    if (om == -INFINITY) return;
    if (om > m) {
        z = (m == -INFINITY ? 0.0f : z * exp2f(m - om)) + oz;
        m = om;
    } else {
        z += oz * exp2f(om - m);
    }
}

// A lane's share of a row's n statistics entries st[0..n): entries lane,
// lane + 64, lane + 128, ... merged in that order.
__device__ __forceinline__ float2 lane_ms(const float2* st, uint32_t n, int lane) {
    float m = -INFINITY, z = 0.0f;
    // loads issued 8 per lane before they are merged, in entry order
    for (int64_t q0 = lane; q0 < n; q0 += 8 * kWave) {
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t q = q0 + u * kWave;
            v[u] = q < n ? st[q] : make_float2(-INFINITY, 0.0f);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) merge_ms(m, z, v[u].x, v[u].y);
    }
    return make_float2(m, z);
}

// (M, Z) of a row from the lanes' shares.  A row given as its single merged
// entry gives back that entry exactly (the other lanes add zeros).
__device__ __forceinline__ float2 wave_ms(float2 v) {
    const float M = wave_max(v.x);
    const float Z = wave_sum(v.x == -INFINITY ? 0.0f : v.y * exp2f(v.x - M));
    return make_float2(M, Z);
}

// (M, Z) of rows 0 .. rows-1 (at most ROWS) of sequence b into sM and sZ:
// wave wv merges rows wv, wv + 4, ....  Rows of at most 64 entries (V <=
// 262144, or merged by the statistics kernel) are all loaded before any is
// merged, and the wave reductions of four rows, which are independent,
// overlap.  Longer ones are merged row by row in a loop: unrolled, its code
// alone made the kernels wait for instructions (a tree's 26 rows 4.2 us, 3.2 so).
template <int ROWS>
__device__ __forceinline__ void merge_rows(const AcceptArgs& a, int b, int rows, int lane, int wv, float* sM,
                                           float* sZ) {
    constexpr int kPer = (ROWS + kWavesPerBlock - 1) / kWavesPerBlock;
    const bool given = a.rt0 > 0 && a.tsm == nullptr;         // target rows as the LM-head epilogue left them
    if ((given && a.ntst > (uint32_t)kWave) || a.nslice > (uint32_t)kWave) {
        for (int r = wv; r < rows; r += kWavesPerBlock) {
            uint32_t n;
            const float2* st = row_stats(a, b, r, n);
            const float2 mz = wave_ms(lane_ms(st, n, lane));
            if (lane == 0) { sM[r] = mz.x; sZ[r] = mz.y; }
        }
        return;
    }
    float2 v[(kPer + 3) / 4 * 4];
#pragma unroll
    for (int i = 0; i < (kPer + 3) / 4 * 4; ++i) {
        const int r = wv + i * kWavesPerBlock;
        v[i] = make_float2(-INFINITY, 0.0f);
        if (i < kPer && r < rows) {
            uint32_t n;
            const float2* st = row_stats(a, b, r, n);
            if ((uint32_t)lane < n) v[i] = st[lane];
        }
    }
#pragma unroll
    for (int i0 = 0; i0 < kPer; i0 += 4) {
        if (wv + i0 * kWavesPerBlock >= rows) break;
        float2 mz[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mz[i] = wave_ms(v[i0 + i]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = wv + (i0 + i) * kWavesPerBlock;
            if (lane == 0 && r < rows) { sM[r] = mz[i].x; sZ[r] = mz[i].y; }
        }
    }
}

template <RowLoad LD>
__global__ __launch_bounds__(kAThreads) void stoch_stats_kernel(AcceptArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    if (a.tsm) {
        // Target statistics from the LM-head epilogue (many entries per row):
        // merged here to one entry per row, so that every sampling block
        // reads one entry per target row.  The waves with the highest ids
        // hold the fewest items (often none), so they take the merges.
        const uint32_t gw = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
        const uint32_t GW = gridDim.x * kWavesPerBlock;
        const uint32_t rows = (uint32_t)a.B * (uint32_t)(a.k + 1);
        for (uint32_t m = GW - 1 - gw; m < rows; m += GW) {
            const float2* st = a.tst + (int64_t)m * a.ldtst;
            const float2 r = wave_ms(lane_ms(st, a.ntst, lane));
            if (lane == 0) a.tsm[m] = r;
        }
    }
    auto row_of = [&](uint32_t row) -> const uint16_t* {
        const int64_t b = row / a.Rs;
        const int r = (int)(a.rt0 + row % a.Rs);
        return (r <= a.k) ? a.zt + (b * (a.k + 1) + r) * a.V : a.zd + (b * a.k + (r - a.k - 1)) * a.V;
    };
    // The logits at the draft tokens, which the sampling kernel's accept
    // tests need, are gathered by the workgroups past the streaming ones (64
    // (sequence, draft) pairs per wave), so the sampling kernel reads them in
    // one round trip with the statistics instead of two dependent ones (the
    // draft ids, then the logits at them).
    const uint32_t gwave = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (a.zx && gwave >= a.sw) {
        const uint32_t pz = (gwave - a.sw) * kWave + (uint32_t)lane;
        if (pz < (uint32_t)a.B * (uint32_t)a.k) {
            const int32_t xg = a.x[pz];
            float gt = 0.0f, gd = 0.0f;
            const int64_t b = pz / (uint32_t)a.k, i = pz % (uint32_t)a.k;
            // a tree's node is scored by its parent's row
            const int64_t row = a.parent ? (int64_t)a.parent[pz] + 1 : i;
            if (xg >= 0 && xg < a.V && row >= 0 && row <= i) {
                gt = bf16_to_f32(a.zt[(b * (a.k + 1) + row) * a.V + xg]);
                if (a.zd) gd = bf16_to_f32(a.zd[(b * a.k + i) * a.V + xg]);
            }
            a.zx[pz] = make_float2(gt, gd);
        }
        return;
    }
    stream_items<LD>(a, row_of, [&](uint32_t it, Raw& raw) {
        const uint32_t row = it / a.nslice, c = it % a.nslice;
        const int64_t e0 = (int64_t)c * kSlice, e1 = min(e0 + kSlice, a.V);
        if (c == 0 && (row % a.Rs) == 0 && lane == 0) a.ctr[row / a.Rs] = 0u;   // ticket of the sample kernel
        cut_slice<LD>(raw, e0, e1, lane, kBf16NegInf);
        const float2 r = (e1 - e0 == kSlice) ? slice_stats<true>(raw, e0, e1, lane, a.c2)
                                                    : slice_stats<false>(raw, e0, e1, lane, a.c2);
        if (lane == 0) a.stats[(int64_t)row * a.nslice + c] = r;
    });
}

// Residual (or bonus) distribution at the sampled position j.
struct Dist {
    const uint16_t* zt_row;   // target row j
    const uint16_t* zd_row;   // draft row j, or null (one-hot drafts / bonus)
    float mt, inv_zt;         // merged max and 1/sum of the target row
    float md, inv_zd;
    int64_t skip;             // element forced to zero (one-hot draft), -1 if none
};

// Probabilities of the 8 elements at e (< e1) from loaded vectors: with a
// draft row (HAS_D) the residual max(0, p - q), else p with element `skip`
// (the one-hot draft token, or -1) and the elements of the bit mask `kill` set
// to zero.
template <RowLoad LD, bool HAS_D>
__device__ __forceinline__ void dist8(const Dist& d, float c2, uint4 rt, uint4 rd, int64_t e,
                                      int64_t e1, unsigned kill, float r[8]) {
    float zt[8];
    cut8<LD>(rt, e, e1, 0);
    unpack8(rt, zt);
    if constexpr (HAS_D) {
        float zd[8];
        cut8<LD>(rd, e, e1, 0);
        unpack8(rd, zd);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float p = __builtin_amdgcn_exp2f(fmaf(zt[q], c2, -d.mt)) * d.inv_zt;
            const float qq = __builtin_amdgcn_exp2f(fmaf(zd[q], c2, -d.md)) * d.inv_zd;
            r[q] = in8<LD>(e, q, e1) ? fmaxf(p - qq, 0.0f) : 0.0f;
        }
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float p = __builtin_amdgcn_exp2f(fmaf(zt[q], c2, -d.mt)) * d.inv_zt;
            r[q] = (in8<LD>(e, q, e1) && e + q != d.skip && !((kill >> q) & 1u)) ? p : 0.0f;
        }
    }
}

// The same probability for one element e < V (bit-identical to dist8).
template <bool HAS_D>
__device__ __forceinline__ float dist1(const Dist& d, float c2, int64_t e) {
    const float p = __builtin_amdgcn_exp2f(fmaf(bf16_to_f32(d.zt_row[e]), c2, -d.mt)) * d.inv_zt;
    if constexpr (HAS_D) {
        const float qq = __builtin_amdgcn_exp2f(fmaf(bf16_to_f32(d.zd_row[e]), c2, -d.md)) * d.inv_zd;
        return fmaxf(p - qq, 0.0f);
    } else {
        return e != d.skip ? p : 0.0f;
    }
}

// Masses of the kAThreads ranges of kPerThread elements of chunk ch, read with
// coalesced loads: wave wv covers the chunk's elements [wv*4096, (wv+1)*4096)
// in kVecs loads of 512 (16 bytes per lane, consecutive lanes on consecutive
// 16-byte pieces, so one load instruction reads 1 KiB contiguous).  The 8 lanes
// that share a range add their sums by xor exchanges in a fixed order, and the
// first of them stores the mass of range wv*64 + j*8 + lane/8 into s_rm.  `kill`
// (without a draft row, or null) is a bit per element of the chunk: those
// elements have no mass.  Called by the whole block; s_rm is complete after the
// caller's next barrier.
template <RowLoad LD, bool HAS_D>
__device__ __forceinline__ void chunk_masses(const Dist& d, float c2, int64_t ch, int64_t V, int t,
                                             double* s_rm, const uint8_t* kill) {
    static_assert(kChunk == (int64_t)kWavesPerBlock * kVecs * kWave * 8 && kPerThread == 8 * 8,
                  "a range is 8 lanes of one load");
    const int lane = t & (kWave - 1), wv = t / kWave;
    const int64_t base = ch * kChunk + (int64_t)wv * (kVecs * kWave * 8) + (int64_t)lane * 8;
    Raw rt, rd;
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
        const int64_t e = base + (int64_t)j * kWave * 8;
        if (e < V) {
            rt[j] = load8<LD, false>(d.zt_row, e, V);
            if (HAS_D) rd[j] = load8<LD, false>(d.zd_row, e, V);
        }
    }
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
        const int64_t e = base + (int64_t)j * kWave * 8;
        double m = 0.0;
        if (e < V) {
            float r[8];
            const unsigned kb = !HAS_D && kill ? kill[(e - ch * kChunk) / 8] : 0u;
            dist8<LD, HAS_D>(d, c2, rt[j], rd[j], e, V, kb, r);
            m = (((double)r[0] + (double)r[1]) + ((double)r[2] + (double)r[3])) +
                (((double)r[4] + (double)r[5]) + ((double)r[6] + (double)r[7]));
        }
        m += __shfl_xor(m, 1);
        m += __shfl_xor(m, 2);
        m += __shfl_xor(m, 4);
        if ((lane & 7) == 0) s_rm[wv * (kVecs * 8) + j * 8 + (lane >> 3)] = m;
    }
}

__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ void store_coherent(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double load_coherent(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Running sums over the lanes of a wave, on DPP lane shifts: within 16-lane
// rows, then the totals of the rows before.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_scan_d(double v) {
    v += dpp_or_zero<0x111, 0xF>(v);    // row_shr 1
    v += dpp_or_zero<0x112, 0xF>(v);
    v += dpp_or_zero<0x114, 0xF>(v);
    v += dpp_or_zero<0x118, 0xF>(v);
    v += dpp_or_zero<0x142, 0xA>(v);    // rows 1 and 3: the last lane of the row before
    v += dpp_or_zero<0x143, 0xC>(v);    // rows 2 and 3: lane 31
    return v;
}

constexpr int kRunRegs = 16;   // chunks whose masses a thread holds at a time (all of them up to V = 262144)

// What the last block of a sequence shares while it searches.
struct Search {
    double tot[kRunRegs * kWavesPerBlock];  // mass of each wave's 64 ranges of each chunk, in vocabulary order
    double base[kWavesPerBlock];            // the mass before each wave's candidate
    int own[kWavesPerBlock];                // the candidate range, -1 where the wave has none
};
static_assert(kRunRegs * kWavesPerBlock == kWave, "a wave total per lane");

// The inverse-CDF search down to one 64-element range, by the whole last
// block of a sequence: its masses fm[0 .. nchunk * 256), one per 64-element
// range in vocabulary order (range th of chunk ch at ch * 256 + th, stored by
// every block of the sequence), are read with consecutive threads on
// consecutive ranges; every wave scans its 64 ranges of each chunk and then
// (each wave for itself) the wave totals, with no search from level to level.
// Returns R (the total), the last range with mass whose preceding mass is at
// most target = u * R, and that mass; range 0 where there is none (R == 0 or
// not finite).  The scans add in different orders, so the mass before a range
// and the end of the one before it may differ in the last bits: an interval
// test could leave target to a range without mass, or to none.  This rule
// always takes a range with mass when R > 0: nothing but zeros lies before the
// first of them.  Beyond kRunRegs chunks they are read in batches, twice (the
// total comes first).
//
// Round trips and barriers bound it (all but one block of the sequence have
// left).  V = 128256: 4.4 us with a run of consecutive ranges per thread (every
// load of a wave on 64 lines), shuffle scans and a walk of the owner's run;
// 3.3 us so.
struct Range {
    double total, before;
    int rng;
};

__device__ __forceinline__ Range locate_range(const double* fm, int64_t nchunk, float u, Search& s) {
    const int t = threadIdx.x, lane = t & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(t / kWave);
    double incl[kRunRegs], pre = 0.0;
    unsigned mass = 0;                       // bit i: this thread's range of chunk c0 + i has mass
    // running sums over this thread's wave of chunks c0 .., and over all waves' totals
    auto scan = [&](int64_t c0) {
        double v[kRunRegs];
#pragma unroll
        for (int i = 0; i < kRunRegs; ++i) v[i] = c0 + i < nchunk ? load_coherent(fm + (c0 + i) * kAThreads + t) : 0.0;
        __syncthreads();                     // s's previous readers are done
        mass = 0;
#pragma unroll
        for (int i = 0; i < kRunRegs; ++i) {
            incl[i] = 0.0;
            mass |= (v[i] > 0.0 ? 1u : 0u) << i;
            if (c0 + i < nchunk) incl[i] = wave_scan_d(v[i]);
            if (lane == kWave - 1) s.tot[i * kWavesPerBlock + wv] = incl[i];
        }
        __syncthreads();
        pre = wave_scan_d(s.tot[lane]);
    };
    auto lane_of = [](double v, int l) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                                __builtin_amdgcn_readlane(__double2loint(v), l));
    };
    double R = 0.0;
    for (int64_t c0 = 0; c0 < nchunk; c0 += kRunRegs) {
        scan(c0);
        R += lane_of(pre, kWave - 1);
    }
    const double target = (double)u * R;
    int mine = -1;                           // this thread's last range with mass that starts by target
    double mine_base = 0.0;
    double sum = 0.0;
    for (int64_t c0 = 0; c0 < nchunk; c0 += kRunRegs) {
        if (nchunk > kRunRegs) scan(c0);
#pragma unroll
        for (int i = 0; i < kRunRegs; ++i) {
            if (c0 + i < nchunk) {
                const int w = i * kWavesPerBlock + wv;
                const double start = w > 0 ? sum + lane_of(pre, w - 1) : sum;
                const double lo = start + dpp_or_zero<0x138, 0xF>(incl[i]);    // (the lane before)
                if (((mass >> i) & 1u) && lo <= target) {
                    mine = (int)((c0 + i) * kAThreads) + t;
                    mine_base = lo;
                }
            }
        }
        sum += lane_of(pre, kWave - 1);
    }
    const int last = wave_max_i32(mine);
    if (lane == 0) s.own[wv] = last;
    if (mine == last && last >= 0) s.base[wv] = mine_base;
    __syncthreads();
    int own = -1, ow = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w)
        if (s.own[w] > own) { own = s.own[w]; ow = w; }
    if (own < 0) return {R, 0.0, 0};
    return {R, s.base[ow], own};
}

// The element to take within the found range, one per lane of wave 0 (all 64
// active): the last one with mass r whose preceding mass is at most target, by
// the same rule (the last with mass, or lane 0, where there is none).
__device__ __forceinline__ int pick_element(float r, double before, double target) {
    const double incl = wave_scan_d((double)r);
    const double excl = dpp_or_zero<0x138, 0xF>(incl);       // the lane before
    const unsigned long long own = __ballot(r > 0.0f && before + excl <= target);
    const unsigned long long pos = __ballot(r > 0.0f);
    const unsigned long long from = own ? own : pos;
    return from ? 63 - __builtin_clzll(from) : 0;
}

// Sampling from the residual (or bonus) distribution of position j by inverse
// CDF in vocabulary order: every block stores the masses of its chunk's 256
// ranges of 64 elements (thread t owns range t); the last block of the
// sequence finds the range holding u*R (locate_range), then the element
// within the range (one lane each).
template <RowLoad LD>
__global__ __launch_bounds__(kAThreads) void stoch_sample_kernel(AcceptArgs a) {
    __shared__ float sM[33], sZ[33];
    __shared__ double s_rm[kAThreads];
    __shared__ int s_x[16];
    __shared__ int s_j, s_last;
    __shared__ float s_uk;
    __shared__ Search s_find;
    const int64_t c = blockIdx.x;
    const int b = blockIdx.y;
    const int t = threadIdx.x;
    const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int k = a.k;

    // The operands of the accept tests are loaded first (draft id, then the
    // two logits at it), so their round trips overlap the statistics merge;
    // so are the resampling uniform and the drafts the outputs repeat.
    // With a statistics pass the logits at the draft tokens were gathered by
    // it, and load with the draft ids in one round trip.
    int32_t xi = -1;
    float zx_t = 0.0f, zx_d = 0.0f, ui = 0.0f;
    if (t <= k) ui = a.u[(int64_t)b * (k + 1) + t];
    if (t < k) {
        xi = a.x[(int64_t)b * k + t];
        if (a.zx) {
            const float2 g = a.zx[(int64_t)b * k + t];
            zx_t = g.x;
            zx_d = g.y;
        } else if (xi >= 0 && xi < a.V) {
            zx_t = bf16_to_f32(a.zt[((int64_t)b * (k + 1) + t) * a.V + xi]);
            if (a.zd) zx_d = bf16_to_f32(a.zd[((int64_t)b * k + t) * a.V + xi]);
        }
    }

    // 1. merge the slice statistics of every row of sequence b, in a fixed order
    merge_rows<33>(a, b, (int)a.R, lane, wv, sM, sZ);   // R <= 2*16+1
    if (t < k) s_x[t] = xi;
    if (t == k) s_uk = ui;
    __syncthreads();

    // 2. accept tests of the k drafts, evaluated in parallel (identical in
    //    every block of sequence b), one lane each: the first rejection is j.
    //    t - M is formed exactly in double (bf16 * fp32 fits in 53 bits).
    if (wv == 0) {
        bool acc = true;
        if (lane < k) {
            double p = 0.0, q = 0.0;
            if (xi >= 0 && xi < a.V) {
                p = exp2((double)zx_t * (double)a.c2 - (double)sM[t]) / (double)sZ[t];
                q = a.zd ? exp2((double)zx_d * (double)a.c2 - (double)sM[k + 1 + t]) / (double)sZ[k + 1 + t] : 1.0;
            }
            acc = (double)ui * q < p;
        }
        const unsigned long long rej = __ballot(!acc);
        if (lane == 0) s_j = rej ? __ffsll((long long)rej) - 1 : k;
    }
    __syncthreads();
    const int j = s_j;

    Dist d;
    d.zt_row = a.zt + ((int64_t)b * (k + 1) + j) * a.V;
    d.mt = sM[j];
    d.inv_zt = 1.0f / sZ[j];
    d.zd_row = nullptr;
    d.md = 0.0f;
    d.inv_zd = 0.0f;
    d.skip = -1;
    if (j < k) {
        if (a.zd) {
            d.zd_row = a.zd + ((int64_t)b * k + j) * a.V;
            d.md = sM[k + 1 + j];
            d.inv_zd = 1.0f / sZ[k + 1 + j];
        } else {
            d.skip = s_x[j];
        }
    }

    double* fm = a.finem + (int64_t)b * a.nchunk * kAThreads;   // range masses
    auto range_of = [&](int64_t ch, int th, int64_t& e0, int64_t& e1) {
        e0 = ch * kChunk + (int64_t)th * kPerThread;
        e1 = min(e0 + kPerThread, a.V);
    };
    // the mass of this thread's range of chunk ch (every thread of the block calls it)
    auto mass_of = [&](int64_t ch) {
        __syncthreads();                     // s_rm's previous readers are done
        if (d.zd_row) chunk_masses<LD, true>(d, a.c2, ch, a.V, t, s_rm, nullptr);
        else chunk_masses<LD, false>(d, a.c2, ch, a.V, t, s_rm, nullptr);
        __syncthreads();
        return s_rm[t];
    };

    // 3. this block's range masses, stored device-coherently (relaxed
    //    agent-scope atomic stores, written through the L2) and acknowledged
    //    before the ticket is taken; the last block reads them with
    //    device-coherent loads.  No agent-scope fence is needed (on this chip
    //    such a fence writes back and invalidates the XCD's whole L2).
    {
        const double m = mass_of(c);
        store_coherent(fm + c * kAThreads + t, m);
        wait_stores();
        __syncthreads();
        if (t == 0) {
            const unsigned int ticket = __hip_atomic_fetch_add(a.ctr + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = (ticket == (unsigned int)(a.nchunk - 1));
        }
        __syncthreads();
        if (!s_last) return;
    }

    // 4. last block of sequence b: the range of 64 elements holding u*R.
    Range at = locate_range(fm, a.nchunk, s_uk, s_find);
    if (!(at.total > 0.0)) {
        // The residual vanished (p_j == q_j wherever it is positive): sample
        // p_j itself.  This block recomputes every range mass.
        d.zd_row = nullptr;
        d.skip = -1;
        for (int64_t ch = 0; ch < a.nchunk; ++ch) store_coherent(fm + ch * kAThreads + t, mass_of(ch));
        wait_stores();
        __syncthreads();
        at = locate_range(fm, a.nchunk, s_uk, s_find);
    }
    const double target = (double)s_uk * at.total;

    // Then the element within the range (wave 0, one element per lane).
    if (wv == 0) {
        int64_t e0, e1;
        range_of(at.rng / kAThreads, at.rng % kAThreads, e0, e1);
        const int64_t e = e0 + lane;
        const float r = e < e1 ? (d.zd_row ? dist1<true>(d, a.c2, e) : dist1<false>(d, a.c2, e)) : 0.0f;
        const int pick = pick_element(r, at.before, target);
        if (lane <= k) {
            int32_t* out = a.out + (int64_t)b * (k + 1);
            out[lane] = lane < j ? s_x[lane] : (lane == j ? (int)min(e0 + pick, a.V - 1) : -1);
            if (lane == 0) {
                a.num[b] = j;
                a.ctr[b] = 0u;
            }
        }
    }
}

// ------------------------------------------------------------- token tree
//
// Tree mode: the N drafted nodes of a sequence form a tree (parent[n] in
// [-1, n), -1 for candidates of the first new position); target row 0 scores
// the first new position and row n+1 the position after node n, so a
// sequence has N+1 target rows, whose statistics the streaming kernels above
// compute as for k = N.  The children of a node are its candidates, tested
// in index order.  A node whose parent is out of range is never reached.

constexpr int kMaxTree = 64;   // nodes per sequence


// Writes sequence b's outputs: the tokens of the accepted path, then the
// emitted token, -1 padded to N+1; the path's node indices, -1 padded to N.
__device__ __forceinline__ void tree_outputs(const AcceptArgs& a, int b, const int* path, const int* x, int depth,
                                             int token, int i0, int step) {
    const int N = a.k;
    for (int i = i0; i <= N; i += step) {
        a.out[(int64_t)b * (N + 1) + i] = i < depth ? x[path[i]] : (i == depth ? token : -1);
        if (i < N) a.nodes[(int64_t)b * N + i] = i < depth ? path[i] : -1;
    }
}

// Greedy walk (one block per sequence): the argmax of every row from its
// slice statistics, then from the root the first child whose token is the
// current row's argmax, until no child matches; that argmax is emitted.
__global__ __launch_bounds__(1024) void tree_greedy_kernel(AcceptArgs a) {
    __shared__ int g[kMaxTree + 1];
    __shared__ int s_x[kMaxTree], s_path[kMaxTree];
    __shared__ int s_depth, s_tok;
    const int b = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int N = a.k;
    // the tree and the first statistics entry of every row of the wave are
    // loaded before anything waits for them (one round trip for all)
    int par = -2, xv = -1;
    if (t < N) {
        par = a.parent[(int64_t)b * N + t];
        xv = a.x[(int64_t)b * N + t];
    }
    // rows over the 16 waves: wave wv merges rows wv, wv+16, ...
    constexpr int kGreedyWaves = 1024 / kWave;
    constexpr int kRowsPerWaveG = (kMaxTree + 1 + kGreedyWaves - 1) / kGreedyWaves;
    float2 first[kRowsPerWaveG];
#pragma unroll
    for (int i = 0; i < kRowsPerWaveG; ++i) {
        const int r = wv + i * kGreedyWaves;
        first[i] = r <= N ? argmax_entry(a, b, r, lane) : make_float2(-INFINITY, __int_as_float(0x7fffffff));
    }
#pragma unroll
    for (int i = 0; i < kRowsPerWaveG; ++i) {
        const int r = wv + i * kGreedyWaves;
        if (r > N) break;
        const int bi = merged_argmax(a, b, r, lane, first[i]);
        if (lane == 0) g[r] = bi;
    }
    if (t < N) s_x[t] = xv;
    __syncthreads();
    if (wv == 0) {                     // a node per lane of wave 0
        int cur = -1, depth = 0, gv;
        for (;;) {
            gv = __builtin_amdgcn_readfirstlane(g[cur + 1]);
            const uint64_t hit = __ballot(par == cur && lane > cur && xv == gv);
            if (hit == 0) break;
            cur = __builtin_ctzll(hit);
            if (lane == 0) s_path[depth] = cur;
            ++depth;
        }
        if (lane == 0) {
            s_depth = depth;
            s_tok = gv;
        }
    }
    __syncthreads();
    tree_outputs(a, b, s_path, s_x, s_depth, s_tok, t, blockDim.x);
    if (t == 0) a.num[b] = s_depth;
}

// Sampling walk, block (chunk c, sequence b).  Every block merges the row
// statistics, gets every candidate's target probability in parallel (one
// round trip for all of them) and walks the tree identically: at the current
// node, child n with token x is accepted iff u[n] (1 - S) < P(x), S the mass
// of the tokens already rejected there (a repeated token has P = 0); on
// acceptance the walk moves to n, else x is removed.  Where every child is
// rejected (or there is none) the final draw comes from P with the removed
// tokens zeroed: each block sums its chunk as for chains (the removed tokens
// of the chunk are a bit mask in LDS), and the last block of the sequence
// searches the range and the element holding u[N] R.
//
// A chain of latencies bounds it, so the tree lies in the lanes of wave 0 (one
// node each, N <= 64) and a step of the walk is a ballot and a few lane reads,
// not a scan of LDS, the candidates' logits come with the statistics in one
// round trip, and the chunk is read with coalesced loads (64 trees of 25 nodes,
// V = 128256: the call 88.1 us; 92.2 with a lane per 64-element range, the walk
// in LDS and a second round trip for the logits).
template <RowLoad LD>
__global__ __launch_bounds__(kAThreads) void tree_sample_kernel(AcceptArgs a) {
    __shared__ float sM[kMaxTree + 1], sZ[kMaxTree + 1];
    __shared__ double s_rm[kAThreads];
    __shared__ uint32_t s_kill[kChunk / 32];
    __shared__ int s_x[kMaxTree], s_path[kMaxTree];
    __shared__ int s_f, s_last;
    __shared__ float s_un;
    __shared__ Search s_find;
    static_assert(kMaxTree <= kWave, "a node per lane of wave 0");
    const int64_t c = blockIdx.x;
    const int b = blockIdx.y;
    const int t = threadIdx.x;
    const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int N = a.k;

    // the tree, the uniforms, the first statistics entries and the
    // candidates' logits (gathered by the statistics kernel) are loaded before
    // anything waits for them: one round trip
    int par = -2, xv = -1;
    float uv = 0.0f, zx = 0.0f;
    if (t < N) {
        par = a.parent[(int64_t)b * N + t];
        xv = a.x[(int64_t)b * N + t];
        zx = a.zx[(int64_t)b * N + t].x;
    }
    if (t <= N) uv = a.u[(int64_t)b * (N + 1) + t];
    merge_rows<kMaxTree + 1>(a, b, N + 1, lane, wv, sM, sZ);
    const bool ok = par >= -1 && par < t && xv >= 0 && xv < a.V;
    if (t < N) s_x[t] = xv;
    if (t == N) s_un = uv;
    for (int i = t; i < (int)(kChunk / 32); i += kAThreads) s_kill[i] = 0u;
    __syncthreads();
    int depth = 0;                     // wave 0's: accepted nodes,
    uint64_t rejected = 0;             // and the nodes whose tokens are removed
    if (wv == 0) {
        // every candidate's probability under its parent's row; t - M is
        // formed exactly in double (bf16 * fp32 fits in 53 bits), as for chains
        const double p = ok ? exp2((double)zx * (double)a.c2 - (double)sM[par + 1]) / (double)sZ[par + 1] : 0.0;
        const int p_lo = __double2loint(p), p_hi = __double2hiint(p);
        int cur = -1;
        for (;;) {
            uint64_t kids = __ballot(par == cur && lane > cur);
            double S = 0.0;
            int nxt = -1;
            rejected = 0;
            while (kids) {
                const int n = __builtin_ctzll(kids);
                kids &= kids - 1;
                const int x = __builtin_amdgcn_readlane(xv, n);
                const bool valid = x >= 0 && x < a.V && (__ballot(xv == x) & rejected) == 0;
                const double px = valid ? __hiloint2double(__builtin_amdgcn_readlane(p_hi, n),
                                                           __builtin_amdgcn_readlane(p_lo, n))
                                        : 0.0;
                const float un = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(uv), n));
                if ((double)un * (1.0 - S) < px) { nxt = n; break; }
                if (valid) {
                    rejected |= 1ull << n;
                    S += px;
                }
            }
            if (nxt < 0) break;
            if (lane == 0) s_path[depth] = nxt;
            ++depth;
            cur = nxt;
        }
        if (lane == 0) s_f = cur;
        const int64_t off = (int64_t)xv - c * kChunk;
        if (((rejected >> lane) & 1ull) && off >= 0 && off < kChunk) atomicOr(&s_kill[off / 32], 1u << (off % 32));
    }
    __syncthreads();
    const int f = s_f;

    Dist d;
    d.zt_row = a.zt + ((int64_t)b * (N + 1) + f + 1) * a.V;
    d.mt = sM[f + 1];
    d.inv_zt = 1.0f / sZ[f + 1];
    d.zd_row = nullptr;
    d.md = 0.0f;
    d.inv_zd = 0.0f;
    d.skip = -1;
    double* fm = a.finem + (int64_t)b * a.nchunk * kAThreads;
    {
        chunk_masses<LD, false>(d, a.c2, c, a.V, t, s_rm, reinterpret_cast<const uint8_t*>(s_kill));
        __syncthreads();
        store_coherent(fm + c * kAThreads + t, s_rm[t]);
        wait_stores();
        __syncthreads();
        if (t == 0) {
            const unsigned int ticket = __hip_atomic_fetch_add(a.ctr + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = (ticket == (unsigned int)(a.nchunk - 1));
        }
        __syncthreads();
        if (!s_last) return;
    }
    Range at = locate_range(fm, a.nchunk, s_un, s_find);
    if (!(at.total > 0.0)) {
        // the removed tokens held all the mass: draw from P itself
        rejected = 0;
        for (int64_t ch = 0; ch < a.nchunk; ++ch) {
            __syncthreads();                     // s_rm's previous readers are done
            chunk_masses<LD, false>(d, a.c2, ch, a.V, t, s_rm, nullptr);
            __syncthreads();
            store_coherent(fm + ch * kAThreads + t, s_rm[t]);
        }
        wait_stores();
        __syncthreads();
        at = locate_range(fm, a.nchunk, s_un, s_find);
    }
    const double target = (double)s_un * at.total;
    if (wv == 0) {
        const int64_t e0 = (int64_t)at.rng * kPerThread, e1 = min(e0 + kPerThread, a.V);
        const int64_t e = e0 + lane;
        float r = e < e1 ? dist1<false>(d, a.c2, e) : 0.0f;
        for (uint64_t m = rejected; m; m &= m - 1)
            if (e == __builtin_amdgcn_readlane(xv, __builtin_ctzll(m))) r = 0.0f;
        const int pick = pick_element(r, at.before, target);
        tree_outputs(a, b, s_path, s_x, depth, (int)min(e0 + pick, a.V - 1), lane, kWave);
        if (lane == 0) {
            a.num[b] = depth;
            a.ctr[b] = 0u;
        }
    }
}

// Clears the sample kernel's tickets when no statistics kernel runs (target
// statistics given and no draft logits to stream).
__global__ __launch_bounds__(256) void clear_tickets_kernel(unsigned int* ctr, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) ctr[i] = 0u;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
std::atomic<int> g_cus[kMaxDevices];

// Compute units of the current device (256 on MI355X), looked up once per
// device; the streaming grids are sized from it.
hipError_t device_cus(int* cus) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    int n = g_cus[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        if (n <= 0) return hipErrorInvalidDevice;
        g_cus[dev].store(n, std::memory_order_relaxed);
    }
    *cus = n;
    return hipSuccess;
}

}  // namespace

hipError_t accept_scratch(void** ptr) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

#define SPEC_ROW_LOAD(kernel, ...)                                                 \
    do {                                                                           \
        if (ld == kAligned) hipLaunchKernelGGL(kernel<kAligned>, __VA_ARGS__);     \
        else if (ld == kLoose) hipLaunchKernelGGL(kernel<kLoose>, __VA_ARGS__);    \
        else hipLaunchKernelGGL(kernel<kShort>, __VA_ARGS__);                      \
    } while (0)

hipError_t launch_accept(const AcceptPlan& p, const uint16_t* zt, const uint16_t* zd, const int32_t* x,
                         const float* u, int64_t B, int64_t k, int64_t V, float temperature,
                         int32_t* out_tokens, int32_t* num_accepted, void* workspace, hipStream_t stream,
                         const float2* tstats, int64_t n_tstats, int64_t ld_tstats) {
    int cus = 0;
    if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
    AcceptArgs a{};
    a.tst = tstats; a.ntst = (uint32_t)n_tstats; a.ldtst = ld_tstats; a.tsm = nullptr;
    char* ws = reinterpret_cast<char*>(workspace);
    a.zt = zt; a.zd = zd; a.x = x; a.u = u; a.out = out_tokens; a.num = num_accepted;
    a.stats = reinterpret_cast<float2*>(ws + p.stats_off);
    a.finem = reinterpret_cast<double*>(ws + p.fine_off);
    a.ctr = reinterpret_cast<unsigned int*>(ws + p.ctr_off);
    a.V = V; a.nchunk = p.nchunk; a.nslice = (uint32_t)p.nschunk; a.B = (int)B; a.k = (int)k;
    const RowLoad ld = row_load(V, zt, zd);
    a.rt0 = tstats ? (uint32_t)(k + 1) : 0u;
    if (temperature == 0.0f) {
        a.R = (uint32_t)(k + 1);
        a.Rs = a.R - a.rt0;
        a.c2 = 0.0f;
        a.items = (uint32_t)(B * a.Rs * p.nschunk);
        if (a.items > 0) {
            const unsigned g1 = stream_blocks(a.items, cus);
            a.sw = g1 * kWavesPerBlock;
            SPEC_ROW_LOAD(greedy_partial_kernel, dim3(g1), dim3(kAThreads), 0, stream, a);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        // one wave per position (k + 1 <= 17 positions, at most 16 waves)
        const unsigned fw = (unsigned)(k + 1 < 16 ? k + 1 : 16);
        hipLaunchKernelGGL(greedy_final_kernel, dim3((unsigned)B), dim3(64 * fw), 0, stream, a);
        return hipGetLastError();
    }
    a.R = (uint32_t)((k + 1) + (zd ? k : 0));
    a.Rs = a.R - a.rt0;
    a.c2 = (float)(1.4426950408889634 / (double)temperature);
    a.items = (uint32_t)(B * a.Rs * p.nschunk);
    // with target statistics and streamed draft rows, the statistics kernel
    // merges the target rows' entries into the statistics area after the
    // streamed rows' (B*Rs*nslice + B*(k+1) <= B*R*nslice entries)
    if (tstats && a.items > 0) a.tsm = a.stats + (int64_t)B * a.Rs * p.nschunk;
    if (a.items > 0) {
        const unsigned g1 = stream_blocks(a.items, cus);
        a.sw = g1 * kWavesPerBlock;
        // workgroups past the streaming ones gather the logits at the draft
        // tokens, 64 (sequence, draft) pairs per wave
        a.zx = reinterpret_cast<float2*>(ws + p.zx_off);
        const unsigned gz = (unsigned)((B * k + kAThreads - 1) / kAThreads);
        SPEC_ROW_LOAD(stoch_stats_kernel, dim3(g1 + gz), dim3(kAThreads), 0, stream, a);
    } else {
        hipLaunchKernelGGL(clear_tickets_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, stream, a.ctr,
                           (int)B);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 g2((unsigned)p.nchunk, (unsigned)B);
    SPEC_ROW_LOAD(stoch_sample_kernel, g2, dim3(kAThreads), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_accept_tree(const AcceptPlan& p, const uint16_t* zt, const int32_t* parent, const int32_t* x,
                              const float* u, int64_t B, int64_t N, int64_t V, float temperature,
                              int32_t* out_tokens, int32_t* accepted_nodes, int32_t* num_accepted, void* workspace,
                              hipStream_t stream) {
    int cus = 0;
    if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
    AcceptArgs a{};
    char* ws = reinterpret_cast<char*>(workspace);
    a.zt = zt; a.zd = nullptr; a.x = x; a.u = u; a.out = out_tokens; a.num = num_accepted;
    a.parent = parent; a.nodes = accepted_nodes;
    a.stats = reinterpret_cast<float2*>(ws + p.stats_off);
    a.finem = reinterpret_cast<double*>(ws + p.fine_off);
    a.ctr = reinterpret_cast<unsigned int*>(ws + p.ctr_off);
    a.tst = nullptr; a.ntst = 0; a.ldtst = 0;
    a.V = V; a.nchunk = p.nchunk; a.nslice = (uint32_t)p.nschunk; a.B = (int)B; a.k = (int)N;
    a.R = a.Rs = (uint32_t)(N + 1);
    a.rt0 = 0;
    a.items = (uint32_t)(B * a.Rs * p.nschunk);
    const RowLoad ld = row_load(V, zt, nullptr);
    const unsigned g1 = stream_blocks(a.items, cus);
    a.sw = g1 * kWavesPerBlock;
    if (temperature == 0.0f) {
        a.c2 = 0.0f;
        SPEC_ROW_LOAD(greedy_partial_kernel, dim3(g1), dim3(kAThreads), 0, stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(tree_greedy_kernel, dim3((unsigned)B), dim3(1024), 0, stream, a);
        return hipGetLastError();
    }
    a.c2 = (float)(1.4426950408889634 / (double)temperature);
    // the candidates' logits are gathered as the chains' are
    a.zx = reinterpret_cast<float2*>(ws + p.zx_off);
    const unsigned gz = (unsigned)((B * N + kAThreads - 1) / kAThreads);
    SPEC_ROW_LOAD(stoch_stats_kernel, dim3(g1 + gz), dim3(kAThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 g2((unsigned)p.nchunk, (unsigned)B);
    SPEC_ROW_LOAD(tree_sample_kernel, g2, dim3(kAThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace specfp8
