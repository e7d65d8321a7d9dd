// The form of the MFMA GEMM kernel for products with few tiles: quarters (64 x 64) of 128x128 tiles on eight wavefronts.
#pragma once
#include "gemm_common.h"

namespace mllm {

namespace {

// ---------------------------------------------------------------------------------------------
// What bounds a product that leaves most CUs idle is latency: a 128x128 tile of the other forms walks its k-tiles one after
// the other, three of them requested ahead, on a few dozen CUs.  Here a tile is a quarter of that, on four times as many CUs, and
// seven k-tiles of 16 KB are requested ahead (all of them up to K = 448), so that from the first one on a CU takes them as
// fast as L2 gives them.  Each wavefront owns 16 x 32 of the tile and walks all of K in its order, as every other tile does: a quarter
// is the same to the bit as its part of the 128x128 tile that it stands for, so which of the two a product takes cannot be
// seen in its result.  The loop is short code on purpose: in a row of small launches a kernel's instructions come from L2.
// Against the 128x128 form, back to back, operands from memory (us): 148 x 768 x 256 5.1 -> 4.1, 576 x 512 x 512 6.6 -> 5.4, 576 x 1024
// x 1024 8.9 -> 7.3, dX of 1728 x 512 x 3584 23.2 -> 16.4; both gradients of a map, 148 tokens x 192 x 768 7.7 -> 6.1, 576 x 512 x 512
// 7.7 -> 6.2, 148 x 256 x 2048 with dX in four parts 9.4 -> 8.2.  (Eight wavefronts that deal the k-tiles out between them and add
// their sums in LDS are within a tenth of that either way, and add in another order than every other tile.)
// ---------------------------------------------------------------------------------------------
constexpr int SMALL_TILE = 64, SMALL_WAVES = 8, SMALL_STAGES = 8;
constexpr int SMALL_OPERAND_B = SMALL_TILE * BK * 2, SMALL_STAGE_B = 2 * SMALL_OPERAND_B, SMALL_LDS_B = SMALL_STAGES * SMALL_STAGE_B;

// One operand's k-tile in LDS: 64 LDS rows of 128 bytes, 16-byte chunk c of row r at chunk position c ^ swz(r).
//   K_ROWS = false (operand stored [EXT, K]): LDS rows are rows of C, read 16 bytes a lane, 16 rows by 4 chunks.
//   K_ROWS = true (stored [K, EXT]): LDS rows are k, read transposed, rows k .. k+3 and k+8 .. k+11 by 32 bytes per 32 lanes.
// A load instruction covers 8 rows, one for each wavefront.
template <bool K_ROWS>
struct SmallLoader {
  uint32_t off, kstep;   // byte offset of the lane's chunk in k-tile 0, OOB if never valid; bytes per k-tile
  static __device__ __forceinline__ int swz(int r) {
    if constexpr (K_ROWS) return ((r & 2) | ((r >> 1) & 4));
    else return (r >> 1) & 7;
  }
  __device__ __forceinline__ void init(int64_t ld, int64_t fixed0, int64_t nfixed, int lane, int wave) {
    const int r = 8 * wave + lane / 8, cc = ((lane % 8) ^ swz(r)) * 8;
    // rows past the operand's end lie past its buffer; columns past its width would not
    if constexpr (K_ROWS) off = fixed0 + cc < nfixed ? (uint32_t)(((int64_t)r * ld + fixed0 + cc) * 2) : OOB;
    else off = fixed0 + r < nfixed ? (uint32_t)(((fixed0 + r) * ld + cc) * 2) : OOB;
    kstep = K_ROWS ? (uint32_t)(BK * ld * 2) : BK * 2;
  }
  // Fragment of the 16 rows (columns) from n0: lane l holds row l%16, k = 32 kk + 8 (l/16) .. +7.
  static __device__ __forceinline__ bf16x8 frag(const char* tile, int n0, int kk, int lane) {
    Frag8 f;
    const int g = lane >> 4, i16 = lane & 15;
    if constexpr (!K_ROWS) {
      f.u = *reinterpret_cast<const uint4*>(tile + (n0 + i16) * 128 + 16 * ((4 * kk + g) ^ swz(i16)));
    } else {
      const int k = 32 * kk + 8 * g + (i16 >> 2), n = n0 + 4 * (i16 & 3);
      const char* q = tile + k * 128 + 16 * ((n >> 3) ^ swz(8 * g + (i16 >> 2))) + 2 * (n & 7);
      f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLLM_LDS s16x4*)q);
      f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLLM_LDS s16x4*)(q + 4 * 128));
    }
    return f.v;
  }
};

// pid of nblk workgroups of the product, each of them with part `split` of the K loop.  Operands start on 16 bytes; K is a
// multiple of 64, or k runs along the rows of both operands (the rows of the last k-tile that lie past K are then past the
// operands' ends).
template <bool A_T, bool B_T, bool OUT_F32>
__device__ __forceinline__ void gemm_small_tile(GemmParams p, int pid, int nblk, int split, char* lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  tile_of_block(pid, nblk, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
  const int64_t m0 = (int64_t)tm * SMALL_TILE, n0 = (int64_t)tn * SMALL_TILE;
  const int kt0 = split * p.kt_per_split, nk = min(p.kt_per_split, (int)((p.K + BK - 1) / BK) - kt0);   // at least one
  SmallLoader<A_T> la;
  SmallLoader<B_T> lb;
  la.init(p.lda, m0, p.M, lane, wave);
  lb.init(p.ldb, n0, p.N, lane, wave);
  const i32x4_t ra = raw_rsrc(p.a, p.a_bytes), rb = raw_rsrc(p.b, p.b_bytes);
  const uint32_t to = __builtin_amdgcn_readfirstlane(lds_address((MLLM_LDS const void*)lds) + wave * 1024);
  // Past the last k-tile the descriptors are empty: zeros into a stage that nobody reads, no traffic, and the count of loads stays.
  auto issue = [&](int kt) {
    const bool have = kt < nk;
    const uint32_t k = have ? (uint32_t)(kt0 + kt) : 0u, at = to + (uint32_t)(kt % SMALL_STAGES) * SMALL_STAGE_B;
    i32x4_t sa = ra, sb = rb;
    sa[2] = have ? ra[2] : 0;
    sb[2] = have ? rb[2] : 0;
    load_to_lds_b128(sa, at, la.off, k * la.kstep);
    load_to_lds_b128(sb, at + SMALL_OPERAND_B, lb.off, k * lb.kstep);
  };
  constexpr int AHEAD = SMALL_STAGES - 1;
#pragma unroll
  for (int kt = 0; kt < AHEAD; kt++) issue(kt);
  const int wm = wave >> 1, wn = wave & 1;
  f32x4 acc[1][2] = {{f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}}};
  for (int kt = 0; kt < nk; kt++) {
    wait_loads<2 * (AHEAD - 1)>();
    // every wavefront's share of this k-tile has landed, and the fragments of the one before are in registers: its stage is free
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue(kt + AHEAD);
    const char* const at = lds + kt % SMALL_STAGES * SMALL_STAGE_B;
    bf16x8 af[2], bfr[2][2];
#pragma unroll
    for (int kk = 0; kk < 2; kk++) {
      af[kk] = SmallLoader<A_T>::frag(at, 16 * wm, kk, lane);
#pragma unroll
      for (int j = 0; j < 2; j++) bfr[kk][j] = SmallLoader<B_T>::frag(at + SMALL_OPERAND_B, 32 * wn + 16 * j, kk, lane);
    }
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int j = 0; j < 2; j++) acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[kk][j], af[kk], acc[0][j], 0, 0, 0);
  }
  wait_loads<0>();   // the empty tiles
  __syncthreads();
  if constexpr (OUT_F32) p.c = reinterpret_cast<float*>(p.c) + split * p.c_split_stride;
  store_blocks<1, 2, OUT_F32>(p, acc, m0 + 16 * wm, n0 + 32 * wn, lane, reinterpret_cast<uint32_t*>(lds + wave * SMALL_STAGE_B));
}

template <bool A_T, bool B_T, bool OUT_F32>
__global__ __launch_bounds__(512, 2) void gemm_small_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[SMALL_LDS_B];
  gemm_small_tile<A_T, B_T, OUT_F32>(p, blockIdx.x, gridDim.x, blockIdx.y, lds);
}

}  // namespace

}  // namespace mllm
