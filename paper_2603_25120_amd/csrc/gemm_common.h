// Pieces shared by the GEMM kernels: launch parameters, buffer resources, the XCD-aware tile
// order and the LDS-staged epilogues.
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace mllm {

constexpr int BK = 64;
constexpr int GEMM_CUS = 256;   // compute units; one workgroup of the larger forms on each

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t OOB = 0xFFFFFFFFu;  // byte offset beyond any buffer these kernels accept (< 4 GiB - 16)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

struct GemmParams {
  const bf16_t* a;
  const bf16_t* b;
  void* c;
  const bf16_t* bias;
  const bf16_t* res;
  int64_t M, N, K, lda, ldb, ldc, ldres;
  uint32_t a_bytes, b_bytes;
  int accumulate;
  int tiles_m, tiles_n;
  int group_m;              // tile-rows of a panel in the walk over the tiles
  int kt_per_split;         // k-tiles handled by one workgroup row (gridDim.y splits of the K loop)
  int64_t c_split_stride;   // elements between the partial outputs of consecutive splits
  bf16_t* act;              // fused SwiGLU: silu(gate) * up, [M, N / 2]
  const bf16_t* pre;        // fused SwiGLU gradient: [gate | up], [M, 2 N]
  bf16_t* dpre;             //                        [d gate | d up], [M, 2 N]
  const float* rope_table;  // fused rotary positions: [positions, head_dim] fp32, cos then sin
  const int32_t* rope_pos;  //                         position of every row of C
  int64_t rope_cols;        //                         leading columns of C that are rotated heads
};

inline GemmParams make_gemm_params(const GemmArgs& g, int bm, int bn) {
  GemmParams p;
  p.a = (const bf16_t*)g.a; p.b = (const bf16_t*)g.b; p.c = g.c;
  p.bias = (const bf16_t*)g.bias; p.res = (const bf16_t*)g.residual;
  p.M = g.m; p.N = g.n; p.K = g.k; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc; p.ldres = g.ldres;
  p.accumulate = g.accumulate;
  p.a_bytes = (uint32_t)((g.a_layout ? g.k : g.m) * g.lda * 2);
  p.b_bytes = (uint32_t)((g.b_layout ? g.n : g.k) * g.ldb * 2);
  p.tiles_m = (int)((g.m + bm - 1) / bm);
  p.tiles_n = (int)((g.n + bn - 1) / bn);
  // An XCD's 32 resident tiles are a block of group_m x 32 / group_m.  8 x 4 fetches as much as 4 x 8, but reads A once
  // for every 4 columns of tiles: once A no longer stays in the 256 MB memory-side cache, 4 x 8 halves what
  // comes from memory (32768 x 4096 x 14336, A 0.94 GB: 1408 -> 1446 TFLOP/s; x 28672 k-contiguous 1528 -> 1559; 8192 x
  // 4096 x 22016, A 0.36 GB: 1425 -> 1442; below, 26496 x 1024 x 4096, A 0.22 GB: 1328 -> 1304).
  p.group_m = g.m * g.k * 2 > (int64_t)320 << 20 ? 4 : 8;
  p.kt_per_split = (int)((g.k + BK - 1) / BK);
  p.c_split_stride = 0;
  p.act = (bf16_t*)g.swiglu_act;
  p.pre = (const bf16_t*)g.swiglu_pre;
  p.dpre = (bf16_t*)g.swiglu_dpre;
  p.rope_table = g.rope_table;
  p.rope_pos = g.rope_pos;
  p.rope_cols = g.rope_cols;
  return p;
}

// Output tiles of the MFMA kernel (gemm_tile.h) and its epilogues.
enum class GemmTile { T256, T224, T192, T128, T64 };   // 256 x 256, 224 and 192 x 256 (A stored [M, K]), 128 x 128, 64 x 64 (gemm_small.h)
inline int tile_rows(GemmTile t) { return t == GemmTile::T256 ? 256 : t == GemmTile::T224 ? 224 : t == GemmTile::T192 ? 192 : t == GemmTile::T128 ? 128 : 64; }
inline int tile_cols(GemmTile t) { return t == GemmTile::T128 ? 128 : t == GemmTile::T64 ? 64 : 256; }
enum { EPI_PLAIN = 0, EPI_SWIGLU = 1, EPI_SWIGLU_BWD = 2, EPI_ROPE128 = 3, EPI_ROPE64 = 4 };
template <bool A_T, bool B_T>
hipError_t launch_gemm_tile(const GemmParams& p, GemmTile tile, bool out_f32, int epi, dim3 grid, hipStream_t s);
template <bool A_T, bool B_T>   // the same on eight wavefronts (gemm_wide.h)
hipError_t launch_gemm_wide(const GemmParams& p, GemmTile tile, bool out_f32, int epi, dim3 grid, hipStream_t s);

hipError_t launch_gemm_small(const GemmParams& p, bool a_t, bool b_t, bool out_f32, dim3 grid, hipStream_t s);   // 64 x 64 tiles (gemm_small.hip)

// A linear map's input gradient (x) and weight gradient (w) in one launch (gemm_pair.hip).
struct GemmPairParams {
  GemmParams x, w;
  int x_tiles, w_tiles;   // workgroups of one part of the K loop
  int first;              // workgroups of the product that comes first
  int x_first;
};
hipError_t launch_gemm_pair_tiles(const GemmPairParams& p, GemmTile x_tile, bool x_f32, int x_epi, GemmTile w_tile, int workgroups, hipStream_t s);
hipError_t launch_gemm_pair_small(const GemmPairParams& p, bool x_f32, int workgroups, hipStream_t s);   // both in 64 x 64 tiles (gemm_small.hip)

// Workgroups are dealt round-robin to the 8 XCDs.  Renumber so that each XCD gets a contiguous
// range of tile ids, then walk the tile grid in panels of group_m tile-rows.
__device__ __forceinline__ void tile_of_block(int pid, int nblk, int tiles_m, int tiles_n, int group_m,
                                              int& tm, int& tn) {
  const int per = (nblk + 7) >> 3, r = nblk & 7;
  const int x = pid & 7, local = pid >> 3;
  int off = (r == 0 || x <= r) ? x * per : r * per + (x - r) * (per - 1);
  int t = off + local;
  const int in_group = group_m * tiles_n;
  const int gid = t / in_group;
  const int first_m = gid * group_m;
  const int gsz = min(tiles_m - first_m, group_m);
  tm = first_m + (t % in_group) % gsz;
  tn = (t % in_group) / gsz;
}

// Epilogue.  The MFMAs are issued with the operands swapped, so an accumulator block holds C
// transposed: a lane owns C row (lane%32) and acc[v] is column 8*(v/4) + 4*(lane/32) + v%4, i.e.
// runs of four consecutive columns.  One 32-row band at a time goes through a per-wavefront fp32
// staging area in LDS (32 x (WN+4) floats at `stage`) and leaves as 16-byte chunks (256 or 512
// contiguous bytes per row), with bias / residual / accumulate applied in fp32 and a single
// rounding on the way out.  Every wavefront of the workgroup must call it (it synchronises).
template <int TM, int TN, bool OUT_F32>
__device__ __forceinline__ void store_tile(const GemmParams& p, f32x16 (&acc)[TM][TN], float* stage,
                                           int64_t row0, int64_t col0, int lane) {
  constexpr int WN = 32 * TN, ST_STRIDE = WN + 4;
  const int h = lane >> 5, cl = lane & 31;
  constexpr int EPC = OUT_F32 ? 4 : 8;  // output elements per 16-byte chunk
  constexpr int ESIZE = OUT_F32 ? 4 : 2;
  constexpr int CHUNKS_PER_ROW = WN / EPC, CHUNKS = 32 * CHUNKS_PER_ROW, PER_BAND = CHUNKS / 64;
  static_assert(64 % CHUNKS_PER_ROW == 0, "a lane keeps its columns from chunk to chunk");
  // chunk t of a band: row rr0 + t * ROWS_PER_PASS of the band, columns [cc, cc + EPC) for every t
  constexpr int ROWS_PER_PASS = 64 / CHUNKS_PER_ROW;
  const int rr0 = lane / CHUNKS_PER_ROW, cc = (lane % CHUNKS_PER_ROW) * EPC;
  const int64_t col = col0 + cc;
  const bool col_ok = col < p.N;
  // Addresses: a wavefront-uniform 64-bit base per matrix (the sub-tile's first element) plus a
  // 32-bit offset of the lane's first chunk plus a uniform multiple of the row pitch (a sub-tile
  // spans at most 128 rows: the host keeps 128 row pitches below 4 GiB).
  const int rows_left = (int)min((int64_t)(32 * TM), p.M - row0);   // rows of this sub-tile inside C
  char* const c_base = reinterpret_cast<char*>(p.c) + (row0 * p.ldc + col0) * ESIZE;
  const uint32_t c_pitch = (uint32_t)(p.ldc * ESIZE), c_lane = (uint32_t)rr0 * c_pitch + (uint32_t)(cc * ESIZE);
  const char* const r_base = reinterpret_cast<const char*>(p.res) + (row0 * p.ldres + col0) * 2;
  const uint32_t r_pitch = (uint32_t)(p.ldres * 2), r_lane = (uint32_t)rr0 * r_pitch + (uint32_t)(cc * 2);
  // the bias of this lane's columns, once for the whole tile
  float bias_f[EPC];
#pragma unroll
  for (int q = 0; q < EPC; q++) bias_f[q] = 0.f;
  if (p.bias && col_ok) {
#pragma unroll
    for (int q = 0; q < EPC / 2; q++) {
      const uint32_t bb = *reinterpret_cast<const uint32_t*>(p.bias + col + 2 * q);
      bias_f[2 * q] = bf16lo(bb);
      bias_f[2 * q + 1] = bf16hi(bb);
    }
  }
  // FULL: the whole sub-tile lies inside C (wavefront-uniform), no per-chunk predicate.
  auto emit = [&](auto full_c) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full_c)::value;
#pragma unroll
    for (int i = 0; i < TM; i++) {
      __syncthreads();   // the band staged before (or the last tile's fragments) has been read
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int g4 = 0; g4 < 4; g4++)
          *reinterpret_cast<float4*>(stage + cl * ST_STRIDE + 32 * j + 8 * g4 + 4 * h) =
              make_float4(acc[i][j][4 * g4], acc[i][j][4 * g4 + 1], acc[i][j][4 * g4 + 2], acc[i][j][4 * g4 + 3]);
      __syncthreads();
#pragma unroll
      for (int t = 0; t < PER_BAND; t++) {
        const int rr = rr0 + t * ROWS_PER_PASS;
        const int r = 32 * i + t * ROWS_PER_PASS;
        if (!FULL && !(r + rr0 < rows_left && col_ok)) continue;
        float f[EPC];
#pragma unroll
        for (int q = 0; q < EPC / 4; q++) {
          const float4 v = *reinterpret_cast<const float4*>(stage + rr * ST_STRIDE + cc + 4 * q);
          f[4 * q] = v.x; f[4 * q + 1] = v.y; f[4 * q + 2] = v.z; f[4 * q + 3] = v.w;
        }
        if (p.bias) {
#pragma unroll
          for (int q = 0; q < EPC; q++) f[q] += bias_f[q];
        }
        char* const dst_b = c_base + (c_lane + (uint32_t)r * c_pitch);
        if constexpr (OUT_F32) {
          float4* dst = reinterpret_cast<float4*>(dst_b);
          if (p.accumulate) {
            const float4 old = *dst;
            f[0] += old.x; f[1] += old.y; f[2] += old.z; f[3] += old.w;
          }
          *dst = make_float4(f[0], f[1], f[2], f[3]);
        } else {
          if (p.res) {
            const uint4 rv = *reinterpret_cast<const uint4*>(r_base + (r_lane + (uint32_t)r * r_pitch));
            f[0] += bf16lo(rv.x); f[1] += bf16hi(rv.x); f[2] += bf16lo(rv.y); f[3] += bf16hi(rv.y);
            f[4] += bf16lo(rv.z); f[5] += bf16hi(rv.z); f[6] += bf16lo(rv.w); f[7] += bf16hi(rv.w);
          }
          *reinterpret_cast<uint4*>(dst_b) =
              make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
        }
      }
    }
  };
  if (rows_left >= 32 * TM && col0 + WN <= p.N) emit(std::true_type{});
  else emit(std::false_type{});
}

// ---------------------------------------------------------------------------------------------
// Epilogues of the tile kernel.  The MFMAs (16x16x32) are issued with the operands swapped, so an accumulator
// block holds C transposed: lane l owns row l%16 of the block and columns 4*(l/16) .. +3.  Stored like that,
// consecutive lanes write 16 bytes to 16 different rows, and the memory pipeline takes such a store apart: fp32
// tiles of 256 x 256, one per CU (1024 x 12800), leave in 12.0 us that way and in 9.4 when every four lanes write 64
// contiguous bytes (permuting half rows so that a store covers 8 rows of 128 bytes, lanes still in row order: 12.0).  So
// a row of blocks at a time passes through the wavefront's own part of the LDS that the tiles have left (`stage`,
// two buffers, no barrier: a wavefront's LDS accesses execute in order) and leaves in row order, 16 bytes a lane, 128 to 512
// contiguous bytes a row; bf16 operands of the epilogue (residual, gate, up) come in in the same order.  What needs
// nothing added is staged already rounded.  The padding of 4 words leaves fp32 rows without bank conflicts
// and bf16 rows with 384 conflict cycles a wavefront (an exclusive-or order with two thirds of them was no faster).  Whole products,
// stores from the accumulators -> staged: 5120 x 11008 x 100 weight gradient 53 -> 44 us, 1024 x 12800 x 480 24.4 -> 21.9;
// forward 7488 x 4096 x 1024 64.8 -> 61.6, 2880 x 4096 x 1024 26.6 -> 25.3.
// Addresses: a buffer over the wavefront's rows of the matrix that starts at the sub-tile's first
// element (rows past the matrix are past its end and dropped by the range check; the host keeps 128
// row pitches below 4 GiB); chunks past the last column get an offset that is never in range.
// ---------------------------------------------------------------------------------------------
// Sixteen bytes of a staged row.  Kept out of the accumulation registers, where the allocator would put it and move
// accumulators out of its way.
__device__ __forceinline__ u32x4 staged_chunk(const uint32_t* src) {
  u32x4 c = *reinterpret_cast<const u32x4*>(src);
  asm volatile("" : "+v"(c));
  return c;
}
__device__ __forceinline__ u32x2 pack4(const f32x4& v) { return u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])}; }
// Rows [0, rows_left) of a matrix from `first` on (row pitch in bytes); rows_left <= 0: empty.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_buffer(const void* first, int rows_left, uint32_t pitch) {
  return make_rsrc(first, rows_left > 0 ? (uint32_t)rows_left * pitch : 0u);
}

// Rotary positions on a row of blocks while it is still in registers (columns from a multiple of HD, so
// the blocks hold whole heads of HD = 128 or 64).  A lane owns one row, so the row's position and its angles
// are the lane's own, and the half-split partner of column c, c + HD/2, lies HD/32 blocks further in the
// same lane: the rotation needs no exchange.  trow: the row's factors, cos then sin.
template <int WN, int HD>
__device__ __forceinline__ void rope_rotate_row(f32x4 (&v)[WN], const float* trow, int g) {
  static_assert((HD == 128 || HD == 64) && 16 * WN % HD == 0, "whole heads of 64 or 128");
  constexpr int HALF = HD / 2, STEP = HD / 32;      // partner block = block + STEP
#pragma unroll
  for (int f = 0; f < HALF / 16; f++) {   // frequencies 16 f + 4 g .. +3
    const f32x4 c = *reinterpret_cast<const f32x4*>(trow + 16 * f + 4 * g);
    const f32x4 s = *reinterpret_cast<const f32x4*>(trow + HALF + 16 * f + 4 * g);
#pragma unroll
    for (int head = 0; head < 16 * WN / HD; head++) {
      f32x4& a = v[head * 2 * STEP + f];
      f32x4& b = v[head * 2 * STEP + f + STEP];
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const float x1 = a[e], x2 = b[e];
        a[e] = x1 * c[e] - x2 * s[e];
        b[e] = x2 * c[e] + x1 * s[e];
      }
    }
  }
}

// C (+)= acc (+ bias, then rotated) (+ residual): WM x WN blocks of 16 x 16 from (row0, col0).  ROPE_HD:
// head width of the rotary positions, 0 for none; sub-tiles past rope_cols (the v columns) are not rotated.
// What a call does not have is decided once, in front of the rows.
template <int WM, int WN, bool OUT_F32, int ROPE_HD = 0>
__device__ __forceinline__ void store_blocks(const GemmParams& p, const f32x4 (&acc)[WM][WN], int64_t row0, int64_t col0, int lane,
                                             uint32_t* stage) {
  constexpr int ESIZE = OUT_F32 ? 4 : 2;
  constexpr int LPR = WN * ESIZE, RPS = 64 / LPR, NS = 16 / RPS;   // a row's lanes, rows of a store, stores of a row of blocks
  const int g = lane >> 4, r = lane & 15;
  const int rows_left = (int)max((int64_t)0, min((int64_t)(16 * WM), p.M - row0));
  const int cols_left = (int)max((int64_t)0, min((int64_t)(16 * WN), p.N - col0));
  const uint32_t pitch = (uint32_t)(p.ldc * ESIZE);
  const __amdgpu_buffer_rsrc_t rc = rows_buffer(reinterpret_cast<const char*>(p.c) + (row0 * p.ldc + col0) * ESIZE, rows_left, pitch);
  const int srow = lane / LPR, scol = lane % LPR * (16 / ESIZE);    // the lane's row and columns in a store
  const uint32_t past = scol < cols_left ? 0u : OOB;                // past the last column: an offset that is never in range
  const uint32_t lane_off = (uint32_t)srow * pitch + (uint32_t)(ESIZE * scol);
  const uint32_t rpitch = (uint32_t)(p.ldres * 2), rlane_off = (uint32_t)srow * rpitch + (uint32_t)(2 * scol);
  const __amdgpu_buffer_rsrc_t rr = rows_buffer(p.res + row0 * p.ldres + col0, !OUT_F32 && p.res ? rows_left : 0, rpitch);
  auto rows = [&](auto bias_c, auto add_c, auto rope_c) __attribute__((always_inline)) {
    constexpr bool BIAS = decltype(bias_c)::value, ADD = decltype(add_c)::value, ROPE = decltype(rope_c)::value;
    constexpr bool WIDE = OUT_F32 || ADD;                            // staged in fp32, otherwise already rounded
    constexpr int PITCH = (WIDE ? 16 : 8) * WN + 4;                  // 32-bit words of a staged row
    f32x4 bias[BIAS ? WN : 1];
    if constexpr (BIAS) {
#pragma unroll
      for (int j = 0; j < WN; j++) {
        uint2 bb = make_uint2(0, 0);
        if (16 * j + 4 * g < cols_left) bb = *reinterpret_cast<const uint2*>(p.bias + col0 + 16 * j + 4 * g);
        bias[j] = f32x4{bf16lo(bb.x), bf16hi(bb.x), bf16lo(bb.y), bf16hi(bb.y)};
      }
    }
    // what is added to C's chunks (the residual, or C itself when accumulating), a row of blocks ahead
    u32x4 add[2][ADD ? NS : 1];
    auto offset = [&](int i, int q, uint32_t lo, uint32_t pt) { return (int)((lo + (uint32_t)(16 * i + RPS * q) * pt) | past); };
    auto fetch = [&](int i) {
#pragma unroll
      for (int q = 0; q < NS; q++)
        add[i & 1][q] = OUT_F32 ? __builtin_amdgcn_raw_buffer_load_b128(rc, offset(i, q, lane_off, pitch), 0, 0)
                                : __builtin_amdgcn_raw_buffer_load_b128(rr, offset(i, q, rlane_off, rpitch), 0, 0);
    };
    if constexpr (ADD) fetch(0);
#pragma unroll
    for (int i = 0; i < WM; i++) {
      if constexpr (ADD) {
        if (i + 1 < WM) fetch(i + 1);
      }
      uint32_t* const st = stage + (i & 1) * 16 * PITCH;
      f32x4 v[WN];
#pragma unroll
      for (int j = 0; j < WN; j++) {
        v[j] = acc[i][j];
        asm volatile("" : "+v"(v[j]));
        if constexpr (BIAS) {
#pragma unroll
          for (int e = 0; e < 4; e++) v[j][e] += bias[j][e];
        }
      }
      if constexpr (ROPE) {
        const int64_t row = row0 + 16 * i + r;
        const int pos = row < p.M ? p.rope_pos[row] : 0;
        rope_rotate_row<WN, ROPE_HD>(v, p.rope_table + (int64_t)pos * ROPE_HD, g);
      }
#pragma unroll
      for (int j = 0; j < WN; j++) {
        if constexpr (WIDE) *reinterpret_cast<u32x4*>(st + r * PITCH + 16 * j + 4 * g) = __builtin_bit_cast(u32x4, v[j]);
        else *reinterpret_cast<u32x2*>(st + r * PITCH + 8 * j + 2 * g) = pack4(v[j]);
      }
      asm volatile("" ::: "memory");   // a wavefront's own LDS accesses execute in order
#pragma unroll
      for (int q = 0; q < NS; q++) {
        const uint32_t* src = st + (srow + RPS * q) * PITCH + (WIDE ? scol : scol / 2);
        u32x4 c = staged_chunk(src);
        if constexpr (OUT_F32 && ADD) {
#pragma unroll
          for (int e = 0; e < 4; e++) c[e] = __float_as_uint(__uint_as_float(c[e]) + __uint_as_float(add[i & 1][q][e]));
        }
        if constexpr (!OUT_F32 && ADD) {
          const u32x4 d = staged_chunk(src + 4), x = add[i & 1][q];
          const uint32_t w0 = pack_bf16x2(__uint_as_float(c[0]) + bf16lo(x[0]), __uint_as_float(c[1]) + bf16hi(x[0]));
          const uint32_t w1 = pack_bf16x2(__uint_as_float(c[2]) + bf16lo(x[1]), __uint_as_float(c[3]) + bf16hi(x[1]));
          const uint32_t w2 = pack_bf16x2(__uint_as_float(d[0]) + bf16lo(x[2]), __uint_as_float(d[1]) + bf16hi(x[2]));
          const uint32_t w3 = pack_bf16x2(__uint_as_float(d[2]) + bf16lo(x[3]), __uint_as_float(d[3]) + bf16hi(x[3]));
          c = u32x4{w0, w1, w2, w3};
        }
        __builtin_amdgcn_raw_buffer_store_b128(c, rc, offset(i, q, lane_off, pitch), 0, 0);
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using T = std::true_type;
  using F = std::false_type;
  const bool add = OUT_F32 ? p.accumulate != 0 : p.res != nullptr;
  if constexpr (ROPE_HD != 0) {   // a forward product without residual
    if (col0 < p.rope_cols) { if (p.bias) rows(T{}, F{}, T{}); else rows(F{}, F{}, T{}); return; }
    if (p.bias) rows(T{}, F{}, F{}); else rows(F{}, F{}, F{});
  } else if (p.bias) {
    if (add) rows(T{}, T{}, F{}); else rows(T{}, F{}, F{});
  } else {
    if (add) rows(F{}, T{}, F{}); else rows(F{}, F{}, F{});
  }
}

// Epilogue of the fused SwiGLU product.  The left half of the sub-tile's blocks are gate columns
// gcol0 .., the right half the up columns of the same indices.  Writes gate and up into C = [gate | up]
// ([M, N], up at column N / 2 + gcol) and silu(gate) * up, from the fp32 accumulators, into act
// ([M, N / 2]).  The sub-tile's columns all exist (N / 2 is a multiple of the tile's gate columns).
template <int WM, int WN>
__device__ __forceinline__ void store_blocks_swiglu(const GemmParams& p, f32x4 (&acc)[WM][WN], int64_t row0, int64_t gcol0, int lane,
                                                    uint32_t* stage) {
  constexpr int LPR = WN, RPS = 64 / LPR, NS = 16 / RPS;   // a row's lanes (8 columns each), rows of a store, stores of a row of blocks
  constexpr int PART = 4 * WN, PITCH = 3 * PART + 4;       // staged row: gate, up, act, rounded to bf16
  const int g = lane >> 4, r = lane & 15, srow = lane / LPR, scol = lane % LPR * 8;
  const int64_t half = p.N >> 1;
  const int rows_left = (int)max((int64_t)0, min((int64_t)(16 * WM), p.M - row0));
  const uint32_t c_pitch = (uint32_t)(p.ldc * 2), a_pitch = (uint32_t)(half * 2);
  const __amdgpu_buffer_rsrc_t rg = rows_buffer(reinterpret_cast<const char*>(p.c) + (row0 * p.ldc + gcol0) * 2, rows_left, c_pitch);
  const __amdgpu_buffer_rsrc_t ru = rows_buffer(reinterpret_cast<const char*>(p.c) + (row0 * p.ldc + half + gcol0) * 2, rows_left, c_pitch);
  const __amdgpu_buffer_rsrc_t ra = rows_buffer(p.act + row0 * half + gcol0, rows_left, a_pitch);
  const uint32_t c_lane = (uint32_t)srow * c_pitch + (uint32_t)(2 * scol), a_lane = (uint32_t)srow * a_pitch + (uint32_t)(2 * scol);
#pragma unroll
  for (int i = 0; i < WM; i++) {
    uint32_t* const st = stage + (i & 1) * 16 * PITCH;
#pragma unroll
    for (int j = 0; j < WN / 2; j++) {
      f32x4 gt = acc[i][j], up = acc[i][WN / 2 + j], a;
#pragma unroll
      for (int e = 0; e < 4; e++)   // silu through the hardware exp2 and reciprocal (1 ulp each; the result is rounded to bf16)
        a[e] = gt[e] * up[e] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(gt[e] * -1.44269504088896340736f));
      uint32_t* const w = st + r * PITCH + 8 * j + 2 * g;
      *reinterpret_cast<u32x2*>(w) = pack4(gt);
      *reinterpret_cast<u32x2*>(w + PART) = pack4(up);
      *reinterpret_cast<u32x2*>(w + 2 * PART) = pack4(a);
    }
    asm volatile("" ::: "memory");   // a wavefront's own LDS accesses execute in order
#pragma unroll
    for (int q = 0; q < NS; q++) {
      const uint32_t* src = st + (srow + RPS * q) * PITCH + scol / 2;
      const uint32_t row = (uint32_t)(16 * i + RPS * q);
      __builtin_amdgcn_raw_buffer_store_b128(staged_chunk(src), rg, (int)(c_lane + row * c_pitch), 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(staged_chunk(src + PART), ru, (int)(c_lane + row * c_pitch), 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(staged_chunk(src + 2 * PART), ra, (int)(a_lane + row * a_pitch), 0, 0);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Epilogue of dA = dY.W_d^T with SwiGLU's gradient: dA never reaches memory.  A lane takes the gate and
// up chunks of its rows and columns from pre = [gate | up] ([M, 2N], requested a row of blocks ahead) and
// writes
//   d gate = dA * up * s * (1 + gate * (1 - s)),  d up = dA * gate * s,  s = sigmoid(gate)
// to dpre = [d gate | d up] ([M, 2N]).
template <int WM, int WN>
__device__ __forceinline__ void store_blocks_swiglu_bwd(const GemmParams& p, f32x4 (&acc)[WM][WN], int64_t row0, int64_t col0, int lane,
                                                        uint32_t* stage) {
  constexpr int LPR = 2 * WN, RPS = 64 / LPR, NS = 16 / RPS, PITCH = 16 * WN + 4;   // staged row: dA in fp32
  const int g = lane >> 4, r = lane & 15, srow = lane / LPR, scol = lane % LPR * 8;
  const int rows_left = (int)max((int64_t)0, min((int64_t)(16 * WM), p.M - row0));
  const int cols_left = (int)max((int64_t)0, min((int64_t)(16 * WN), p.N - col0));
  const uint32_t past = scol < cols_left ? 0u : OOB;
  const uint32_t pitch = (uint32_t)(p.N * 4);   // bytes: a row of [M, 2N] bf16
  const int64_t at = row0 * 2 * p.N + col0;
  const __amdgpu_buffer_rsrc_t rg = rows_buffer(p.pre + at, rows_left, pitch), ru = rows_buffer(p.pre + at + p.N, rows_left, pitch);
  const __amdgpu_buffer_rsrc_t wg = rows_buffer(p.dpre + at, rows_left, pitch), wu = rows_buffer(p.dpre + at + p.N, rows_left, pitch);
  const uint32_t lane_off = (uint32_t)srow * pitch + (uint32_t)(2 * scol);
  auto offset = [&](int i, int q) { return (int)((lane_off + (uint32_t)(16 * i + RPS * q) * pitch) | past); };
  u32x4 gq[2][NS], uq[2][NS];
  auto fetch = [&](int i) {
#pragma unroll
    for (int q = 0; q < NS; q++) {
      gq[i & 1][q] = __builtin_amdgcn_raw_buffer_load_b128(rg, offset(i, q), 0, 0);
      uq[i & 1][q] = __builtin_amdgcn_raw_buffer_load_b128(ru, offset(i, q), 0, 0);
    }
  };
  fetch(0);
#pragma unroll
  for (int i = 0; i < WM; i++) {
    if (i + 1 < WM) fetch(i + 1);
    uint32_t* const st = stage + (i & 1) * 16 * PITCH;
#pragma unroll
    for (int j = 0; j < WN; j++) {
      f32x4 v = acc[i][j];
      asm volatile("" : "+v"(v));
      *reinterpret_cast<u32x4*>(st + r * PITCH + 16 * j + 4 * g) = __builtin_bit_cast(u32x4, v);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < NS; q++) {
      const uint32_t* src = st + (srow + RPS * q) * PITCH + scol;
      const u32x4 d[2] = {staged_chunk(src), staged_chunk(src + 4)};
      u32x4 og, ou;
#pragma unroll
      for (int w = 0; w < 4; w++) {
        const uint32_t gw = gq[i & 1][q][w], uw = uq[i & 1][q][w];
        const float gt[2] = {bf16lo(gw), bf16hi(gw)}, up[2] = {bf16lo(uw), bf16hi(uw)};
        float dg[2], du[2];
#pragma unroll
        for (int e = 0; e < 2; e++) {
          const float da = __uint_as_float(d[w >> 1][2 * (w & 1) + e]);
          const float s = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(gt[e] * -1.44269504088896340736f));
          const float gs = gt[e] * s;
          dg[e] = da * up[e] * (s + gs * (1.f - s));
          du[e] = da * gs;
        }
        og[w] = pack_bf16x2(dg[0], dg[1]);
        ou[w] = pack_bf16x2(du[0], du[1]);
      }
      __builtin_amdgcn_raw_buffer_store_b128(og, wg, offset(i, q), 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(ou, wu, offset(i, q), 0, 0);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
}

}  // namespace mllm
