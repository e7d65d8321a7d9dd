// Products in 64 x 64 tiles: on their own, and a linear map's input gradient and weight gradient in one launch.
#include "gemm_small.h"

namespace mllm {
namespace {
template <bool X_F32>   // dX in parts: fp32
__global__ __launch_bounds__(512, 2) void gemm_pair_small_kernel(GemmPairParams P) {
  __shared__ __attribute__((aligned(1024))) char lds[SMALL_LDS_B];
  const int pid = blockIdx.x;
  const bool head = pid < P.first;
  const int local = head ? pid : pid - P.first;
  if (head == (P.x_first != 0)) gemm_small_tile<false, false, X_F32>(P.x, local % P.x_tiles, P.x_tiles, local / P.x_tiles, lds);
  else gemm_small_tile<true, true, true>(P.w, local % P.w_tiles, P.w_tiles, local / P.w_tiles, lds);
}
}  // namespace

hipError_t launch_gemm_small(const GemmParams& p, bool a_t, bool b_t, bool out_f32, dim3 grid, hipStream_t s) {
  if (p.K <= 0 || (p.K % BK != 0 && !(a_t && b_t))) return hipErrorInvalidValue;
#define MLLM_SMALL(AT, BT, F32)                                                                \
  if (a_t == AT && b_t == BT && out_f32 == F32) {                                              \
    hipLaunchKernelGGL((gemm_small_kernel<AT, BT, F32>), grid, dim3(512), 0, s, p);            \
    return hipGetLastError();                                                                  \
  }
  MLLM_SMALL(false, true, false)
  MLLM_SMALL(false, true, true)
  MLLM_SMALL(false, false, false)
  MLLM_SMALL(false, false, true)
  MLLM_SMALL(true, true, false)
  MLLM_SMALL(true, true, true)
#undef MLLM_SMALL
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_pair_small(const GemmPairParams& p, bool x_f32, int workgroups, hipStream_t s) {
  if (x_f32) hipLaunchKernelGGL(gemm_pair_small_kernel<true>, dim3((unsigned)workgroups), dim3(512), 0, s, p);
  else hipLaunchKernelGGL(gemm_pair_small_kernel<false>, dim3((unsigned)workgroups), dim3(512), 0, s, p);
  return hipGetLastError();
}
}  // namespace mllm
