// Y = X.W: W stored [K, N].
#include "gemm_wide.h"

namespace mllm {
template hipError_t launch_gemm_tile<false, true>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
template hipError_t launch_gemm_wide<false, true>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
}  // namespace mllm
