// FP8 GEMM kernels (gemm_kernel.hpp) of tile kinds 7 to 12, and with 64-bit operand offsets.
#include "gemm_kernel.hpp"

namespace specfp8 {

template hipError_t launch_gemm_kind<7>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<8>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<9>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<10>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<11>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<12>(int, const GemmArgs&, hipStream_t);

hipError_t launch_gemm_far(int epi, const GemmArgs& g, hipStream_t stream) {
    if (g.splits != 1) return hipErrorInvalidValue;
    if (epi == 0) return launch_one<kFarKind, 0, false, true>(g, stream);
    if (epi == 3) return launch_one<kFarKind, 3, false, true>(g, stream);
    return hipErrorInvalidValue;
}

}  // namespace specfp8
