// The form of the MFMA GEMM kernel for products with few tiles: 64 x 64 tiles on eight wavefronts that share out the K loop.
#pragma once
#include "gemm_common.h"

namespace mllm {

namespace {

// ---------------------------------------------------------------------------------------------
// What bounds a product that leaves most CUs idle is latency: a 128x128 tile of the other forms walks its k-tiles one after
// the other with a barrier each, on a few dozen CUs.  Here a tile is a quarter of that, and its k-tiles are dealt to the
// eight wavefronts of the workgroup, each with 16 KB of LDS of its own: no barrier in the loop, the first eight k-tiles all
// requested at once, a wavefront asks for its next one when it has read the last.  The eight partial sums meet in LDS and are
// added in the order of the wavefronts; each wavefront then writes a 16 x 32 part of the tile.  The loop is short code on
// purpose: in a row of small launches a kernel's instructions come from L2.
// Against the 128x128 form, back to back, weights from memory (us): 148 x 768 x 256 4.8 -> 4.1, 450 x 256 x 1024 9.1 -> 6.0, 576 x
// 512 x 512 6.7 -> 6.0; both gradients of a map, 148 tokens x 192 x 768 7.4 -> 5.6, 576 x 512 x 512 7.6 -> 6.0.  A k-tile of all
// eight wavefronts is 128 KB, 1.4 us of what a CU takes from L2, so with more tiles than CUs the larger tiles, which read half
// as much for their work, are better (where the line lies: takes_small_form in gemm.hip).
// ---------------------------------------------------------------------------------------------
constexpr int SMALL_TILE = 64, SMALL_WAVES = 8, SMALL_STAGE_B = 2 * SMALL_TILE * BK * 2, SMALL_LDS_B = SMALL_WAVES * SMALL_STAGE_B;

// One operand's k-tile in LDS: 64 LDS rows of 128 bytes, 16-byte chunk c of row r at chunk position c ^ swz(r).
//   K_ROWS = false (operand stored [EXT, K]): LDS rows are rows of C, read 16 bytes a lane, 16 rows by 4 chunks.
//   K_ROWS = true (stored [K, EXT]): LDS rows are k, read transposed, rows k .. k+3 and k+8 .. k+11 by 32 bytes per 32 lanes.
// A load instruction covers 8 rows.  The permutation sees bits 1 to 3 of the row, so instruction i differs from i - 2 by 16
// rows of memory alone: a scalar offset.
template <bool K_ROWS>
struct SmallLoader {
  uint32_t off[2], pitch, kstep;   // byte offsets of the lane's chunks in instructions 0 and 1; bytes per row and per k-tile
  static __device__ __forceinline__ int swz(int r) {
    if constexpr (K_ROWS) return ((r & 2) | ((r >> 1) & 4));
    else return (r >> 1) & 7;
  }
  __device__ __forceinline__ void init(int64_t ld, int64_t fixed0, int64_t nfixed, int lane) {
    pitch = (uint32_t)(ld * 2);
    kstep = K_ROWS ? BK * pitch : BK * 2;
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int r = 8 * i + lane / 8, cc = ((lane % 8) ^ swz(r)) * 8;
      // rows past the operand's end lie past its buffer; columns past its width would not
      if constexpr (K_ROWS) off[i] = fixed0 + cc < nfixed ? (uint32_t)(((int64_t)r * ld + fixed0 + cc) * 2) : OOB;
      else off[i] = fixed0 + r < nfixed ? (uint32_t)(((fixed0 + r) * ld + cc) * 2) : OOB;
    }
  }
  __device__ __forceinline__ void load(i32x4_t rsrc, uint32_t lds, int kt, int64_t fixed0, int64_t nfixed) const {
#pragma unroll
    for (int i = 0; i < 8; i++) {
      if (!K_ROWS && fixed0 + 8 * i >= nfixed) break;   // (uniform) no row of this instruction exists: what LDS holds there ends in rows that are not stored
      load_to_lds_b128(rsrc, lds + i * 1024, off[i & 1], (uint32_t)kt * kstep + (uint32_t)(16 * (i >> 1)) * pitch);
    }
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
  const int kt0 = split * p.kt_per_split, nk = min(p.kt_per_split, (int)((p.K + BK - 1) / BK) - kt0);
  SmallLoader<A_T> la;
  SmallLoader<B_T> lb;
  la.init(p.lda, m0, p.M, lane);
  lb.init(p.ldb, n0, p.N, lane);
  const i32x4_t ra = raw_rsrc(p.a, p.a_bytes), rb = raw_rsrc(p.b, p.b_bytes);
  char* const at = lds + wave * SMALL_STAGE_B;
  char* const bt = at + SMALL_STAGE_B / 2;
  const uint32_t a_lds = __builtin_amdgcn_readfirstlane(lds_address((MLLM_LDS const void*)at)), b_lds = a_lds + SMALL_STAGE_B / 2;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kt = wave; kt < nk; kt += SMALL_WAVES) {
    la.load(ra, a_lds, kt0 + kt, m0, p.M);
    lb.load(rb, b_lds, kt0 + kt, n0, p.N);
    wait_loads<0>();
    bf16x8 af[2][4], bfr[2][4];
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        af[kk][i] = SmallLoader<A_T>::frag(at, 16 * i, kk, lane);
        bfr[kk][i] = SmallLoader<B_T>::frag(bt, 16 * i, kk, lane);
      }
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the fragments are read: the next loads may take their place
  }
  // Partial sums: 16 x 32 part r of the tile (rows 16 (r / 2), columns 32 (r % 2)) of wavefront w at (8 r + w) * 2 KB, so that what a
  // wavefront adds up is 16 KB of its own, which then stage its rows.
  const int sources = min(nk, SMALL_WAVES);
  __syncthreads();
  if (wave < sources) {
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int j = 0; j < 4; j++)
        *reinterpret_cast<f32x4*>(lds + (8 * (2 * i + j / 2) + wave) * 2048 + j % 2 * 1024 + lane * 16) = acc[i][j];
  }
  __syncthreads();
  f32x4 sum[1][2];
  char* const mine = lds + wave * SMALL_WAVES * 2048;
#pragma unroll
  for (int j = 0; j < 2; j++) sum[0][j] = *reinterpret_cast<const f32x4*>(mine + j * 1024 + lane * 16);
  for (int w = 1; w < sources; w++)
#pragma unroll
    for (int j = 0; j < 2; j++) sum[0][j] += *reinterpret_cast<const f32x4*>(mine + w * 2048 + j * 1024 + lane * 16);
  asm volatile("" ::: "memory");
  if constexpr (OUT_F32) p.c = reinterpret_cast<float*>(p.c) + split * p.c_split_stride;
  store_blocks<1, 2, OUT_F32>(p, sum, m0 + 16 * (wave >> 1), n0 + 32 * (wave & 1), lane, reinterpret_cast<uint32_t*>(mine));
}

template <bool A_T, bool B_T, bool OUT_F32>
__global__ __launch_bounds__(512, 2) void gemm_small_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[SMALL_LDS_B];
  gemm_small_tile<A_T, B_T, OUT_F32>(p, blockIdx.x, gridDim.x, blockIdx.y, lds);
}

}  // namespace

}  // namespace mllm
