// dW = X^T.dY: both operands stored [K, .]; and A stored [K, M] with B stored [N, K].
#include "gemm_wide.h"

namespace mllm {
template hipError_t launch_gemm_tile<true, true>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
template hipError_t launch_gemm_tile<true, false>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
template hipError_t launch_gemm_wide<true, true>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
}  // namespace mllm
