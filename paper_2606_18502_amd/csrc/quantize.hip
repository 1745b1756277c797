// Row quantization of bf16 activations/weights to E4M3 with fp32 scales, and
// the SiLU-gated variant that feeds the down projection.
//
// One workgroup owns one row.  The row is read from HBM once with 16-byte
// loads (8 bf16 per load, consecutive threads on consecutive 16-byte chunks,
// so every wave reads 1 KiB contiguous per instruction), all issued before any
// is used, and kept in registers as packed bf16; the block reduces max|v| (wave
// shuffles, then LDS across waves), derives the scale, and encodes the
// registers it already holds ([2048, 14336] 18.7 us, [4096, 14336] 35.3, timed in
// turn over rotated inputs; 20.3 and 35.8 with the loads issued one by one into
// fp32 registers).  HBM traffic
// is therefore the algorithmic 2 bytes in + 1 byte out per element (4 + 1 for
// the SiLU-gated input) plus 4 bytes of scale per row.  Rows wider than
// 65536 elements take a second pass that re-reads the row.
#include "device_common.hpp"
#include "kernels.hpp"

namespace specfp8 {

namespace {

constexpr int kQThreads = 256;       // threads of the element-wise kernel
constexpr int kQMaxThreads = 1024;   // threads per row of the row kernel, at most

// One chunk of 8 input values as they are loaded: the bf16 values themselves,
// or the gate and up values of the SiLU-gated input.
template <int IN_KIND>
struct RawChunk {
    uint4 a;
    uint4 b[IN_KIND];     // (IN_KIND 1: the up values)
};

template <int IN_KIND>
__device__ __forceinline__ RawChunk<IN_KIND> load_raw(const uint16_t* __restrict__ xrow, int64_t cols, int64_t c) {
    RawChunk<IN_KIND> r;
    r.a = *reinterpret_cast<const uint4*>(xrow + c * 8);
    if constexpr (IN_KIND == 1) r.b[0] = *reinterpret_cast<const uint4*>(xrow + cols + c * 8);
    return r;
}

// The 8 values to encode, packed bf16 (h of the gated input is a bf16 value by
// definition, so nothing is lost by keeping it packed until it is encoded).
template <int IN_KIND>
__device__ __forceinline__ uint4 chunk_values(const RawChunk<IN_KIND>& r) {
    if constexpr (IN_KIND == 0) {
        return r.a;
    } else {
        float g[8], u[8];
        unpack8(r.a, g);
        unpack8(r.b[0], u);
        uint4 h;
        h.x = silu_mul_bf16x2(g[0], u[0], g[1], u[1]);
        h.y = silu_mul_bf16x2(g[2], u[2], g[3], u[3]);
        h.z = silu_mul_bf16x2(g[4], u[4], g[5], u[5]);
        h.w = silu_mul_bf16x2(g[6], u[6], g[7], u[7]);
        return h;
    }
}

__device__ __forceinline__ float abs_max8(const uint4& h, float amax) {
    float v[8];
    unpack8(h, v);
#pragma unroll
    for (int e = 0; e < 8; e += 2) amax = fmaxf(fmaxf(amax, fabsf(v[e])), fabsf(v[e + 1]));
    return amax;
}

__device__ __forceinline__ void store_codes(uint8_t* __restrict__ qrow, int64_t c, const float (&v)[8], float inv) {
    uint2 o;
    o.x = e4m3x4(v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv);
    o.y = e4m3x4(v[4] * inv, v[5] * inv, v[6] * inv, v[7] * inv);
    *reinterpret_cast<uint2*>(qrow + c * 8) = o;
}

__device__ __forceinline__ void store_codes(uint8_t* __restrict__ qrow, int64_t c, const uint4& h, float inv) {
    float v[8];
    unpack8(h, v);
    store_codes(qrow, c, v, inv);
}

__device__ __forceinline__ void row_scale(float amax, float* s_out, float* inv_out) {
    float s = (float)((double)amax / 448.0);
    s = fmaxf(s, 0x1p-100f);
    *s_out = s;
    *inv_out = (float)(1.0 / (double)s);
}

// Static calibration: running[0] = max(running[0], s).  Scales are finite and
// non-negative, and the bit patterns of non-negative floats order like
// unsigned integers, so an integer atomic max is exact and order-independent.
__device__ __forceinline__ void calibrate_max(float* running, float s) {
    atomicMax(reinterpret_cast<unsigned int*>(running), __float_as_uint(s));
}

// Per-row scales (MODE 0, written) or calibration only (MODE 2): one workgroup
// per row.
// NCH > 0: the row lives in registers, NCH chunks of 8 per thread, all of them
// loaded before any is used (one memory round trip; a chunk past the row's end
// reloads its last one and is not stored).
// NCH == 0: rows too wide for registers; amax pass and encode pass each read the row.
template <int IN_KIND, int MODE, int NCH>
__global__ __launch_bounds__(kQMaxThreads) void quantize_rows_kernel(
    const uint16_t* __restrict__ x, int64_t cols, int64_t ld_x, float* __restrict__ scales,
    uint8_t* __restrict__ q, int64_t ld_q) {
    __shared__ float red[16];
    const int64_t row = blockIdx.x;
    const int64_t nchunks = cols / 8;
    const uint16_t* xrow = x + row * ld_x;
    uint8_t* qrow = q + row * ld_q;
    const int t = threadIdx.x;
    const int nt = blockDim.x;

    uint4 h[NCH > 0 ? NCH : 1];
    float amax = 0.0f;
    if constexpr (NCH > 0) {
        RawChunk<IN_KIND> raw[NCH];
#pragma unroll
        for (int j = 0; j < NCH; ++j)
            raw[j] = load_raw<IN_KIND>(xrow, cols, min(t + (int64_t)j * nt, nchunks - 1));
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            h[j] = chunk_values<IN_KIND>(raw[j]);
            amax = abs_max8(h[j], amax);
        }
    } else {
        for (int64_t c = t; c < nchunks; c += nt)
            amax = abs_max8(chunk_values<IN_KIND>(load_raw<IN_KIND>(xrow, cols, c)), amax);
    }
    float s, inv;
    row_scale(block_max(amax, red), &s, &inv);
    if constexpr (MODE == 2) {
        if (t == 0) calibrate_max(scales, s);
        return;
    }
    if (t == 0) scales[row] = s;
    if constexpr (NCH > 0) {
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int64_t c = t + (int64_t)j * nt;
            if (c < nchunks) store_codes(qrow, c, h[j], inv);
        }
    } else {
        for (int64_t c = t; c < nchunks; c += nt)
            store_codes(qrow, c, chunk_values<IN_KIND>(load_raw<IN_KIND>(xrow, cols, c)), inv);
    }
}

// One given scale, one workgroup per row.  HOW 1: at most one chunk per thread;
// 2: a thread's two chunks are unpacked before any is encoded; 0: its chunks
// are encoded one after the other.
template <int IN_KIND, int HOW>
__global__ __launch_bounds__(kQMaxThreads) void quantize_static_rows_kernel(
    const uint16_t* __restrict__ x, int64_t cols, int64_t ld_x, const float* __restrict__ scale,
    uint8_t* __restrict__ q, int64_t ld_q) {
    const int64_t row = blockIdx.x;
    const int64_t nchunks = cols / 8;
    const uint16_t* xrow = x + row * ld_x;
    uint8_t* qrow = q + row * ld_q;
    const int t = threadIdx.x, nt = blockDim.x;
    if constexpr (HOW == 1) {
        const RawChunk<IN_KIND> raw = load_raw<IN_KIND>(xrow, cols, min((int64_t)t, nchunks - 1));
        const float inv = (float)(1.0 / (double)scale[0]);
        if (t < nchunks) store_codes(qrow, t, chunk_values<IN_KIND>(raw), inv);
    } else if constexpr (HOW == 2) {
        float v[2][8];
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (t + j * nt < nchunks) unpack8(chunk_values<IN_KIND>(load_raw<IN_KIND>(xrow, cols, t + j * nt)), v[j]);
        const float inv = (float)(1.0 / (double)scale[0]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (t + j * nt < nchunks) store_codes(qrow, t + j * nt, v[j], inv);
    } else {
        const float inv = (float)(1.0 / (double)scale[0]);
        auto encode = [&](int64_t c) {
            store_codes(qrow, c, chunk_values<IN_KIND>(load_raw<IN_KIND>(xrow, cols, c)), inv);
        };
        if (t < nchunks) encode(t);
        if (t + nt < nchunks) encode(t + nt);
        for (int64_t c = t + 2 * nt; c < nchunks; c += nt) encode(c);
    }
}

// One given scale and few rows: with no row maximum to reduce, the columns of
// a row are shared by per_row workgroups, one chunk per thread.
template <int IN_KIND>
__global__ __launch_bounds__(kQThreads) void quantize_static_kernel(
    const uint16_t* __restrict__ x, int64_t cols, int64_t ld_x, const float* __restrict__ scale,
    uint8_t* __restrict__ q, int64_t ld_q, unsigned per_row) {
    const int64_t row = blockIdx.x / per_row;
    const int64_t c = (int64_t)(blockIdx.x % per_row) * kQThreads + threadIdx.x;
    if (c >= cols / 8) return;
    const RawChunk<IN_KIND> raw = load_raw<IN_KIND>(x + row * ld_x, cols, c);
    const float inv = (float)(1.0 / (double)scale[0]);
    store_codes(q + row * ld_q, c, chunk_values<IN_KIND>(raw), inv);
}

__global__ __launch_bounds__(kQThreads) void silu_mul_bf16_kernel(
    const uint16_t* __restrict__ x, int64_t rows, int64_t cols, int64_t ld_x,
    uint16_t* __restrict__ h, int64_t ld_h) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cols / 8) return;
    for (int64_t row = blockIdx.y; row < rows; row += gridDim.y) {
        *reinterpret_cast<uint4*>(h + row * ld_h + c * 8) =
            chunk_values<1>(load_raw<1>(x + row * ld_x, cols, c));
    }
}

// Values the static per-tensor quantizer saturates, |fl32(x * fl32(1/s))| >
// 448 (the calibration clip rate of a test batch): grid-stride over 8-value
// chunks read with 16-byte loads, a wave then block sum, one 64-bit atomic
// add per block into the caller's counter.
__global__ __launch_bounds__(kQThreads) void clip_count_kernel(const uint16_t* __restrict__ x, int64_t rows,
                                                               int64_t cols, int64_t ld_x,
                                                               const float* __restrict__ scale,
                                                               unsigned long long* __restrict__ count) {
    __shared__ unsigned int red[kQThreads / 64];
    const float inv = (float)(1.0 / (double)scale[0]);
    const int64_t nch = cols / 8;
    const int64_t total = rows * nch;
    unsigned int c = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / nch;
        const int64_t ch = i - r * nch;
        const uint4 p = *reinterpret_cast<const uint4*>(x + r * ld_x + ch * 8);
        float v[8];
        unpack8(p, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) c += fabsf(v[e] * inv) > 448.0f ? 1u : 0u;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
        for (int w = 0; w < kQThreads / 64; ++w) sum += red[w];
        if (sum) atomicAdd(count, sum);
    }
}

template <int IN_KIND, int MODE>
hipError_t launch_rows(const uint16_t* x, int64_t rows, int64_t cols, int64_t ld_x, float* scales, uint8_t* q,
                       int64_t ld_q, hipStream_t stream) {
    // One workgroup per row, wide enough that a thread holds at most 8 chunks
    // (up to 1024 threads; wider rows take the two-pass path): few waves with
    // many loads in flight each reach the reduction's barrier soonest (8 chunks
    // against 4, 2 or 1: [1005, 14336] rows 9.7 us against 10.1, 11.1 and 10.1,
    // the SiLU-gated [320, 14336] 8.0 against 8.3, 8.6 and 8.7).
    const int64_t nchunks = cols / 8;
    int threads = 256;
    while (threads < kQMaxThreads && nchunks > 8 * (int64_t)threads) threads *= 2;
    if (nchunks < threads) threads = (int)(((nchunks + 63) / 64) * 64);
    const int64_t per = (nchunks + threads - 1) / threads;
    dim3 grid((unsigned)rows), block(threads);
#define SPEC_Q_CASE(N)                                                                        \
    case N:                                                                                   \
        hipLaunchKernelGGL((quantize_rows_kernel<IN_KIND, MODE, N>), grid, block, 0, stream, x, \
                           cols, ld_x, scales, q, ld_q);                                      \
        break;
    switch (per) {
        SPEC_Q_CASE(1)
        SPEC_Q_CASE(2)
        SPEC_Q_CASE(3)
        SPEC_Q_CASE(4)
        SPEC_Q_CASE(5)
        SPEC_Q_CASE(6)
        SPEC_Q_CASE(7)
        SPEC_Q_CASE(8)
        default:
            hipLaunchKernelGGL((quantize_rows_kernel<IN_KIND, MODE, 0>), grid, block, 0, stream, x,
                               cols, ld_x, scales, q, ld_q);
    }
#undef SPEC_Q_CASE
    return hipGetLastError();
}

template <int IN_KIND>
hipError_t launch_static(const uint16_t* x, int64_t rows, int64_t cols, int64_t ld_x, const float* scale, uint8_t* q,
                         int64_t ld_q, hipStream_t stream) {
    // Rows wider than one chunk per thread are split over workgroups (one chunk
    // per thread) while these are hardly more than the chip holds at once (2048:
    // 8 per compute unit), for the SiLU-gated input a little beyond where every
    // one is full, and wherever a row exceeds two chunks per thread of the
    // largest workgroup.  Rows against split rows: 64 x 14336 3.1 -> 2.6 us,
    // 400 x 9000 4.1 -> 3.9 and SiLU-gated 5.6 -> 5.4, SiLU-gated 320 x 14336
    // 7.5 -> 7.0, 300 x 20000 5.9 -> 5.5; beyond the line 450 x 9000 4.2 -> 4.3
    // and 6.2 -> 6.9.
    // Otherwise one workgroup per row: a chunk per thread where that covers it
    // (8192 x 2048 11.9 us, 12.4 with the code for more chunks), else chunk by
    // chunk, but for long streams of plain rows (4096 x 14336 33.6 -> 32.9 us
    // with both chunks first, 8192 x 4096 21.0 -> 20.4; 4096 x 4096 11.9 -> 12.1).
    const int64_t nchunks = cols / 8;
    const int64_t per_row = (nchunks + kQThreads - 1) / kQThreads, blocks = rows * per_row;
    const bool full = IN_KIND == 1 && nchunks % kQThreads == 0;
    const bool split = nchunks > 2 * kQMaxThreads || (nchunks > kQThreads && blocks <= (full ? 2340 : 2100));
    if (split && blocks * kQThreads <= 4294967295LL) {      // (a grid's threads are counted in 32 bits)
        hipLaunchKernelGGL(quantize_static_kernel<IN_KIND>, dim3((unsigned)blocks), dim3(kQThreads), 0, stream, x, cols,
                           ld_x, scale, q, ld_q, (unsigned)per_row);
        return hipGetLastError();
    }
    int threads = 64;
    while (threads < kQMaxThreads && nchunks > (threads < kQThreads ? 1 : 2) * (int64_t)threads) threads *= 2;
    const dim3 grid((unsigned)rows), block(threads);
    if (nchunks <= threads)
        hipLaunchKernelGGL((quantize_static_rows_kernel<IN_KIND, 1>), grid, block, 0, stream, x, cols, ld_x, scale, q,
                           ld_q);
    else if (IN_KIND == 0 && rows * nchunks > 3000000 && nchunks <= 2 * (int64_t)threads)
        hipLaunchKernelGGL((quantize_static_rows_kernel<IN_KIND, 2>), grid, block, 0, stream, x, cols, ld_x, scale, q,
                           ld_q);
    else
        hipLaunchKernelGGL((quantize_static_rows_kernel<IN_KIND, 0>), grid, block, 0, stream, x, cols, ld_x, scale, q,
                           ld_q);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_quantize(const uint16_t* x, int64_t rows, int64_t cols, int64_t ld_x, int in_kind,
                           int mode, float* scales, uint8_t* q, int64_t ld_q, hipStream_t stream) {
    if (mode == 1)
        return in_kind == 0 ? launch_static<0>(x, rows, cols, ld_x, scales, q, ld_q, stream)
                            : launch_static<1>(x, rows, cols, ld_x, scales, q, ld_q, stream);
    if (in_kind == 0)
        return mode == 0 ? launch_rows<0, 0>(x, rows, cols, ld_x, scales, q, ld_q, stream)
                         : launch_rows<0, 2>(x, rows, cols, ld_x, scales, q, ld_q, stream);
    return mode == 0 ? launch_rows<1, 0>(x, rows, cols, ld_x, scales, q, ld_q, stream)
                     : launch_rows<1, 2>(x, rows, cols, ld_x, scales, q, ld_q, stream);
}

hipError_t launch_clip_count(const uint16_t* x, int64_t rows, int64_t cols, int64_t ld_x, const float* scale,
                             unsigned long long* count, hipStream_t stream) {
    const int64_t total = rows * (cols / 8);
    int64_t blocks = (total + kQThreads - 1) / kQThreads;
    if (blocks > 2048) blocks = 2048;           // 8 workgroups per compute unit, grid-stride beyond
    hipLaunchKernelGGL(clip_count_kernel, dim3((unsigned)blocks), dim3(kQThreads), 0, stream, x, rows, cols, ld_x,
                       scale, count);
    return hipGetLastError();
}

hipError_t launch_silu_mul(const uint16_t* x, int64_t rows, int64_t cols, int64_t ld_x,
                           uint16_t* h, int64_t ld_h, hipStream_t stream) {
    const int64_t nchunks = cols / 8;
    const int64_t gy = rows < 65535 ? rows : 65535;
    dim3 block(kQThreads), grid((unsigned)((nchunks + kQThreads - 1) / kQThreads), (unsigned)gy);
    hipLaunchKernelGGL(silu_mul_bf16_kernel, grid, block, 0, stream, x, rows, cols, ld_x, h, ld_h);
    return hipGetLastError();
}

}  // namespace specfp8
