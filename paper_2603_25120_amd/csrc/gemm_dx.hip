// dX = dY.W^T: both operands k-contiguous.
#include "gemm_wide.h"

namespace mllm {
template hipError_t launch_gemm_tile<false, false>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
template hipError_t launch_gemm_wide<false, false>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
}  // namespace mllm
