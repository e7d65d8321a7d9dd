// dX = dY.W^T: both operands k-contiguous.
#include "gemm_tile.h"

namespace mllm {
template hipError_t launch_gemm_tile<false, false>(const GemmParams&, GemmTile, bool, int, dim3, hipStream_t);
}  // namespace mllm
