// FP8 GEMM kernels (gemm_kernel.hpp) of tile kinds 2, 3.
#include "gemm_kernel.hpp"

namespace specfp8 {

template hipError_t launch_gemm_kind<2>(int, const GemmArgs&, hipStream_t);
template hipError_t launch_gemm_kind<3>(int, const GemmArgs&, hipStream_t);

}  // namespace specfp8
