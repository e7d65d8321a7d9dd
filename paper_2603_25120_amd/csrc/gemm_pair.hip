// A linear map's input gradient and weight gradient in one launch: the workgroups of one product follow those of the
// other, each with its own tile size, and run the same code as in a launch of its own (the larger of the two tiles decides
// registers and LDS, so a 128x128 tile beside larger ones has a CU to itself, which costs it little: its k-loop is
// bound by the 32 KB a k-tile that its CU takes from L2, 36 of the 40 bytes a clock that plain loads reach).  What it
// gives and when it is taken: plan_pair in gemm.hip.
#include "gemm_wide.h"

namespace mllm {
namespace {
// (32 XM) x (32 XN) tiles of the input gradient and (32 WW) x (32 WW) tiles of the weight gradient on four wavefronts.
template <int XM, int XN, bool X_F32, int X_EPI, int WW>
__global__ __launch_bounds__(256, XM * XN <= 16 && WW <= 4 ? 2 : 1) void gemm_pair_kernel(GemmPairParams P) {
  constexpr int SA = 32 * (XM > WW ? XM : WW) * BK, SB = 32 * (XN > WW ? XN : WW) * BK;
  __shared__ __attribute__((aligned(1024))) bf16_t As0[SA], As1[SA], Bs0[SB], Bs1[SB];
  const int pid = blockIdx.x;
  const bool head = pid < P.first;
  const int local = head ? pid : pid - P.first;
  if (head == (P.x_first != 0))
    gemm_dma_tile<XM, XN, false, false, X_F32, X_EPI>(P.x, local % P.x_tiles, P.x_tiles, local / P.x_tiles, As0, As1, Bs0, Bs1);
  else
    gemm_dma_tile<WW, WW, true, true, true, EPI_PLAIN>(P.w, local % P.w_tiles, P.w_tiles, local / P.w_tiles, As0, As1, Bs0, Bs1);
}

// Both in 128x128 tiles on eight wavefronts, as long as every workgroup has a CU to itself.  (With large tiles the eight
// wavefronts lose beside the k-contiguous product what they gain for the other one: 200 maps 0.99x, 0.95x above 8192
// columns; small tiles in halves of a large tile's stages wait for each other's loads, 0.8x.)
template <bool X_F32>
__global__ __launch_bounds__(512, 2) void gemm_pair_wide_kernel(GemmPairParams P) {
  __shared__ __attribute__((aligned(1024))) bf16_t As0[128 * BK], As1[128 * BK], As2[128 * BK], As3[128 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t Bs0[128 * BK], Bs1[128 * BK], Bs2[128 * BK], Bs3[128 * BK];
  const int pid = blockIdx.x;
  const bool head = pid < P.first;
  const int local = head ? pid : pid - P.first;
  if (head == (P.x_first != 0))
    gemm_wide_tile<4, 2, 4, false, false, X_F32, EPI_PLAIN>(P.x, local % P.x_tiles, P.x_tiles, local / P.x_tiles, As0, As1, As2, As3, Bs0, Bs1, Bs2, Bs3);
  else
    gemm_wide_tile<4, 2, 4, true, true, true, EPI_PLAIN>(P.w, local % P.w_tiles, P.w_tiles, local / P.w_tiles, As0, As1, As2, As3, Bs0, Bs1, Bs2, Bs3);
}
}  // namespace

hipError_t launch_gemm_pair_tiles(const GemmPairParams& p, GemmTile x_tile, bool x_f32, int x_epi, GemmTile w_tile, int workgroups, hipStream_t s) {
  const dim3 grid((unsigned)workgroups), block(256);
  if (x_tile == GemmTile::T128 && w_tile == GemmTile::T128 && workgroups <= GEMM_CUS && x_epi == EPI_PLAIN) {
    if (x_f32) hipLaunchKernelGGL((gemm_pair_wide_kernel<true>), grid, dim3(512), 0, s, p);
    else hipLaunchKernelGGL((gemm_pair_wide_kernel<false>), grid, dim3(512), 0, s, p);
    return hipGetLastError();
  }
#define MLLM_PAIR(XM, XN, F32, EPI, WW)                                                                \
  do {                                                                                                 \
    hipLaunchKernelGGL((gemm_pair_kernel<XM, XN, F32, EPI, WW>), grid, block, 0, s, p);                \
    return hipGetLastError();                                                                          \
  } while (0)
#define MLLM_PAIR_X(XM, XN, F32, EPI)                         \
  do {                                                        \
    if (w_tile == GemmTile::T256) MLLM_PAIR(XM, XN, F32, EPI, 8); \
    if (w_tile == GemmTile::T128) MLLM_PAIR(XM, XN, F32, EPI, 4); \
  } while (0)
  if (x_epi == EPI_SWIGLU_BWD) {
    if (x_tile == GemmTile::T256) MLLM_PAIR_X(8, 8, false, EPI_SWIGLU_BWD);
    if (x_tile == GemmTile::T224) MLLM_PAIR_X(7, 8, false, EPI_SWIGLU_BWD);
    return hipErrorInvalidValue;
  }
  if (x_f32) {
    if (x_tile == GemmTile::T256) MLLM_PAIR_X(8, 8, true, EPI_PLAIN);
    if (x_tile == GemmTile::T224) MLLM_PAIR_X(7, 8, true, EPI_PLAIN);
    if (x_tile == GemmTile::T192) MLLM_PAIR_X(6, 8, true, EPI_PLAIN);
    if (x_tile == GemmTile::T128) MLLM_PAIR_X(4, 4, true, EPI_PLAIN);
  } else {
    if (x_tile == GemmTile::T256) MLLM_PAIR_X(8, 8, false, EPI_PLAIN);
    if (x_tile == GemmTile::T224) MLLM_PAIR_X(7, 8, false, EPI_PLAIN);
    if (x_tile == GemmTile::T192) MLLM_PAIR_X(6, 8, false, EPI_PLAIN);
    if (x_tile == GemmTile::T128) MLLM_PAIR_X(4, 4, false, EPI_PLAIN);
  }
#undef MLLM_PAIR_X
#undef MLLM_PAIR
  return hipErrorInvalidValue;
}
}  // namespace mllm
