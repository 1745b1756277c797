// FP8 GEMM kernels (gemm_kernel.hpp) of tile kinds 4, 5, 6.
#include "gemm_kernel.hpp"

namespace specfp8 {

template hipError_t launch_gemm_kind<4>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<5>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<6>(int, const GemmArgs&, hipStream_t);

}  // namespace specfp8
