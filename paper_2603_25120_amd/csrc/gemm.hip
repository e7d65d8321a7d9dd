// bf16 MFMA GEMM for gfx950: C[M,N] = op(A) . op(B) (+ bias) (+ residual), fp32 accumulate.
//
// These are the linear operations of the stage, applied to the whole packed sequence at once
// (Model Profiler, "Throughput Profiling"): QKV / output / MLP projections and the connector,
// their input gradients (dX = dY.W^T) and their weight gradients (dW = X^T.dY).
//
// Four kernels.  gemm4_kernel (gemm_tile.h): 256x256, 224x256, 192x256 and 128x128 tiles on four wavefronts with a
// hand-placed k-loop, for every K that is a multiple of 64 and for any K of a weight gradient; gemm_wide_kernel
// (gemm_wide.h): all of these but 224x256 on eight wavefronts; gemm_small_kernel (gemm_small.h): quarters of the small tiles, for
// products of few tiles; plan_gemm below chooses the tile and whether the K loop is split.  A part of the K loop is summed in the
// same order in all of their tiles.
// gemm_kernel (here): a general template for what is left, K no multiple of 64 with an operand whose contiguous dimension is k.  It wants, per lane, eight
// consecutive values along the contraction index for v_mfma_f32_32x32x16_bf16: operands whose
// contraction index is contiguous in memory are staged in LDS as [row][k] and fetched with one 16-byte read;
// operands whose contraction index is the strided one are staged as they lie in memory, [k][row], and
// fetched with the LDS transposing read, so no operand is transposed in global memory or in registers.  One
// workgroup computes a BM x BN tile with (BM/WM)*(BN/WN) wavefronts, each owning a WM x WN sub-tile; the K
// loop moves BK = 64 at a time: global -> registers (prefetch of the next tile) -> LDS.
#include <algorithm>
#include <cmath>
#include <utility>

#include "gemm_common.h"

namespace mllm {

namespace {

// Row padding (elements).  LDS has 64 banks of 4 bytes.  k-contiguous tiles: rows 144 B apart put
// the 16-byte reads of any 16 consecutive rows on distinct banks.  Tiles read with the transposing
// load: 32 lanes of one read touch 4 rows x 64 B, so the row stride must be 16 dwords mod 64
// (576 B for 256 columns, 320 B for 128): the four rows then fill the 64 banks exactly (measured:
// no bank-conflict cycles in any layout).
constexpr int PAD_K = 8;
constexpr int PAD_T = 32;

// Global -> register -> LDS staging of one operand tile through buffer loads: an out-of-range
// offset returns zeros, so ragged edges need no branches.  K_ROWS: the tile's rows run along the
// contraction index (operand stored [K, rows]); otherwise its columns do (stored [rows, K]).
template <int ROWS, int COLS, int PADC, int NT, bool K_ROWS>
struct TileLoader {
  static constexpr int VEC_PER_ROW = COLS / 8;
  static constexpr int NVEC = ROWS * COLS / 8;
  static constexpr int PER_THREAD = NVEC / NT;
  static constexpr int STRIDE = COLS + PADC;
  static_assert(NVEC % NT == 0 && NT % VEC_PER_ROW == 0, "tile must divide among threads");
  u32x4 r[PER_THREAD];
  uint32_t off[PER_THREAD];   // byte offset of this thread's vectors at k0 = 0, OOB if never valid
  int klim[PER_THREAD];       // vector i is inside the matrix while k0 < klim[i]
  uint32_t kstep;             // bytes per BK step

  __device__ __forceinline__ void init(int64_t ld, int64_t fixed0, int64_t nfixed, int64_t K, int tid) {
    kstep = (uint32_t)(K_ROWS ? BK * ld * 2 : BK * 2);
#pragma unroll
    for (int i = 0; i < PER_THREAD; i++) {
      const int v = tid + i * NT, rr = v / VEC_PER_ROW, cc = (v % VEC_PER_ROW) * 8;
      const int64_t fx = fixed0 + (K_ROWS ? cc : rr);
      const int64_t lin = K_ROWS ? (int64_t)rr * ld + fx : fx * ld + cc;
      off[i] = fx < nfixed ? (uint32_t)(lin * 2) : OOB;
      klim[i] = (int)(K - (K_ROWS ? rr : cc));
    }
  }
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rsrc, int kt) { load_part<0, PER_THREAD>(rsrc, kt); }
  __device__ __forceinline__ void store(bf16_t* lds, int tid) const { store_part<0, PER_THREAD>(lds, tid); }
  template <int I0, int I1>
  __device__ __forceinline__ void load_part(__amdgpu_buffer_rsrc_t rsrc, int kt) {
    const int k0 = kt * BK;
#pragma unroll
    for (int i = I0; i < I1; i++) {
      const uint32_t o = (off[i] != OOB && k0 < klim[i]) ? off[i] + (uint32_t)kt * kstep : OOB;
      r[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)o, 0, 0);
    }
  }
  template <int I0, int I1>
  __device__ __forceinline__ void store_part(bf16_t* lds, int tid) const {
#pragma unroll
    for (int i = I0; i < I1; i++) {
      const int v = tid + i * NT, rr = v / VEC_PER_ROW, cc = (v % VEC_PER_ROW) * 8;
      *reinterpret_cast<u32x4*>(lds + rr * STRIDE + cc) = r[i];
    }
  }
};

// Fragment of 8 contraction values for row (r0 + lane%32), k = kk*16 + 8*(lane/32) ...
template <bool TRANSPOSED, int STRIDE>
__device__ __forceinline__ bf16x8 fetch_frag(const bf16_t* tile, int r0, int kk, int lane) {
  Frag8 f;
  const int h = lane >> 5;
  if constexpr (!TRANSPOSED) {
    f.u = *reinterpret_cast<const uint4*>(tile + (r0 + (lane & 31)) * STRIDE + kk * 16 + 8 * h);
  } else {
    const int n0 = r0 + 16 * ((lane >> 4) & 1);
    f.h[0] = lds_read_tr4(tile, STRIDE, kk * 16 + 8 * h, n0, lane & 15);
    f.h[1] = lds_read_tr4(tile, STRIDE, kk * 16 + 8 * h + 4, n0, lane & 15);
  }
  return f.v;
}

// Scheduling pattern of one k-step: MFMA slot M is preceded by up to PER LDS reads while any
// of the N_READS remain.
template <int PER, int N_READS, int M>
__device__ __forceinline__ void interleave_slot() {
  if constexpr (M * PER < N_READS)
    __builtin_amdgcn_sched_group_barrier(0x100, (M + 1) * PER <= N_READS ? PER : N_READS - M * PER, 0);
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
}
template <int PER, int N_READS, int... Ms>
__device__ __forceinline__ void interleave_reads(std::integer_sequence<int, Ms...>) {
  (interleave_slot<PER, N_READS, Ms>(), ...);
}

template <int BM, int BN, int WM, int WN, bool A_T, bool B_T, bool OUT_F32>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN)) void gemm_kernel(GemmParams p) {
  constexpr int NWM = BM / WM, NWN = BN / WN, NT = 64 * NWM * NWN;
  constexpr int TM = WM / 32, TN = WN / 32;
  // A tile: [BM][BK] (contraction contiguous) or [BK][BM] (as stored, transposing reads)
  constexpr int A_ROWS = A_T ? BK : BM, A_COLS = A_T ? BM : BK, A_PAD = A_T ? PAD_T : PAD_K;
  constexpr int B_ROWS = B_T ? BK : BN, B_COLS = B_T ? BN : BK, B_PAD = B_T ? PAD_T : PAD_K;
  constexpr int A_STRIDE = A_COLS + A_PAD, B_STRIDE = B_COLS + B_PAD;
  constexpr int A_SIZE = A_ROWS * A_STRIDE, B_SIZE = B_ROWS * B_STRIDE;
  // two LDS stages: tile kt+1 is written while tile kt is being multiplied
  __shared__ __attribute__((aligned(16))) bf16_t As[2 * A_SIZE];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[2 * B_SIZE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / NWN, wn = wave % NWN;
  int tm, tn;
  tile_of_block(blockIdx.x, gridDim.x, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;

  TileLoader<A_ROWS, A_COLS, A_PAD, NT, A_T> la;
  TileLoader<B_ROWS, B_COLS, B_PAD, NT, B_T> lb;
  la.init(p.lda, m0, p.M, p.K, tid);
  lb.init(p.ldb, n0, p.N, p.K, tid);
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.a, p.a_bytes), rb = make_rsrc(p.b, p.b_bytes);
  auto gload = [&](int kt) {
    la.load(ra, kt);
    lb.load(rb, kt);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  const int nk = (int)((p.K + BK - 1) / BK);
  gload(0);
  la.store(As, tid);
  lb.store(Bs, tid);
  gload(1);
  __syncthreads();

  // Fragments are double-buffered in registers: those of step kk+1 are fetched from LDS while
  // the 16 MFMAs of step kk run; step 0 of the next tile is fetched right after the barrier.
  bf16x8 af[2][TM], bfr[2][TN];
  auto fetch = [&](int buf, const bf16_t* at, const bf16_t* bt, int kk) {
#pragma unroll
    for (int i = 0; i < TM; i++) af[buf][i] = fetch_frag<A_T, A_STRIDE>(at, wm * WM + 32 * i, kk, lane);
#pragma unroll
    for (int j = 0; j < TN; j++) bfr[buf][j] = fetch_frag<B_T, B_STRIDE>(bt, wn * WN + 32 * j, kk, lane);
  };
  fetch(0, As, Bs, 0);
  constexpr int STEPS = BK / 16;
  using LA = TileLoader<A_ROWS, A_COLS, A_PAD, NT, A_T>;
  using LB = TileLoader<B_ROWS, B_COLS, B_PAD, NT, B_T>;
  // The next tile is moved in the first half of the k-steps and the barrier sits before the last
  // step's MFMAs, so that tile's first fragments are fetched under them.
  constexpr int MOVE_STEPS = STEPS / 2;
  constexpr int A_PER = LA::PER_THREAD / MOVE_STEPS, B_PER = LB::PER_THREAD / MOVE_STEPS;
  static_assert(A_PER * MOVE_STEPS == LA::PER_THREAD && B_PER * MOVE_STEPS == LB::PER_THREAD && A_PER >= 1 && B_PER >= 1,
                "the moving k-steps must split the tile evenly");
  for (int kt = 0; kt < nk; kt++) {
    const int cur = kt & 1;
    bf16_t* an = As + (cur ^ 1) * A_SIZE;
    bf16_t* bn = Bs + (cur ^ 1) * B_SIZE;
    const bf16_t* at = As + cur * A_SIZE;
    const bf16_t* bt = Bs + cur * B_SIZE;
    // Branch-free body.  The moving k-steps each put a share of tile kt+1 from the staging
    // registers into the other LDS stage and at once refill those registers with the same share
    // of tile kt+2 (every prefetch has a whole iteration to land); every step but the last
    // fetches the next step's fragments before issuing its MFMAs.  The barrier comes
    // before the last step's MFMAs: by then every fragment of this stage is in registers and
    // every store to the other stage has been issued.  Past the end the prefetch offsets are out
    // of range (zeros, no traffic) and the stored stage is never read.
    auto step = [&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      if constexpr (kk < MOVE_STEPS) {
        la.template store_part<kk * A_PER, (kk + 1) * A_PER>(an, tid);
        lb.template store_part<kk * B_PER, (kk + 1) * B_PER>(bn, tid);
        la.template load_part<kk * A_PER, (kk + 1) * A_PER>(ra, kt + 2);
        lb.template load_part<kk * B_PER, (kk + 1) * B_PER>(rb, kt + 2);
      }
      if constexpr (kk + 1 < STEPS) {
        fetch((kk + 1) & 1, at, bt, kk + 1);
      } else {
        __syncthreads();
        fetch(0, an, bn, 0);
      }
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk & 1][j], af[kk & 1][i], acc[i][j], 0, 0, 0);
      // Issue order inside the step: the LDS reads of the next fragments go out one per MFMA from
      // the step's start (left alone, the scheduler puts them after the MFMAs and the wavefront
      // then waits on LDS with nothing queued behind it).
      constexpr int N_READS = TM * (A_T ? 2 : 1) + TN * (B_T ? 2 : 1), N_MFMA = TM * TN;
      constexpr int PER = (N_READS + N_MFMA - 1) / N_MFMA;     // reads per MFMA slot
      interleave_reads<PER, N_READS>(std::make_integer_sequence<int, N_MFMA>{});
      __builtin_amdgcn_sched_barrier(0);
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
  }

  constexpr int ST_STRIDE = WN + 4;  // floats
  static_assert(NWM * NWN * 32 * ST_STRIDE * 4 <= 2 * A_SIZE * 2, "staging must fit in the A stages");
  store_tile<TM, TN, OUT_F32>(p, acc, reinterpret_cast<float*>(As) + wave * 32 * ST_STRIDE,
                              m0 + wm * WM, n0 + wn * WN, lane);
}

// The tile kernel (gemm_tile.h) takes K a positive multiple of 64, or any K when k runs along the rows of
// both operands (the weight-gradient layout).  There the rows of the last k-tile that lie past K are left to the
// buffer's range check, which sees their 32-bit byte offsets: an operand so close to 4 GiB that one of them would
// wrap round to its first rows stays with the general kernel, which compares row numbers.
bool takes_tile_kernel(const GemmArgs& g) {
  if (g.k <= 0) return false;
  if (g.k % BK == 0) return true;
  if (g.a_layout == 0 || g.b_layout != 0) return false;
  const int64_t rows = (g.k + BK - 1) / BK * BK;
  return rows * g.lda * 2 <= 0xFFFFFFFFll && rows * g.ldb * 2 <= 0xFFFFFFFFll;
}
GemmParams tile_params(const GemmArgs& g, GemmTile tile, int splits) {
  GemmParams p = make_gemm_params(g, tile_rows(tile), tile_cols(tile));
  if (splits > 1) {   // the plan has made sure that no split is empty
    p.kt_per_split = (p.kt_per_split + splits - 1) / splits;
    p.c_split_stride = g.m * g.n;
  }
  return p;
}
// Whether the kernel on eight wavefronts (gemm_wide.h) can take the operands: it loads both straight to LDS.  The rotary epilogue of
// 128 wide heads wants a head's columns in one wavefront.
bool fits_wide_form(const GemmArgs& g) {
  return (((uintptr_t)g.a | (uintptr_t)g.b) & 15) == 0 && !(g.a_layout != 0 && g.b_layout != 0) && !(g.rope_table && g.rope_head_dim == 128);
}
// Quarters of 128x128 tiles (gemm_small.h) in place of these, cut or not, as long as every quarter has a CU to itself.
// 508 products of 18 maps 192 to 4096 wide, 64 to 1728 tokens, operands from memory, in either layout: up to 256 quarters
// (439 products) 1.16x at least, geomean 1.29x, whatever the weight; beyond, where a CU takes two one after the other, 0.73 to
// 0.94x up to 340 and 0.54 to 0.98x up to 640: the larger tiles read half as much for their work.
constexpr int64_t QUARTERS_MOST = GEMM_CUS;
int64_t quarters(const GemmArgs& g, int splits) { return ((g.m + 63) / 64) * ((g.n + 63) / 64) * splits; }
bool takes_quarters(const GemmArgs& g, int splits) {
  return fits_wide_form(g) && !g.swiglu_act && !g.swiglu_dpre && !g.rope_table && quarters(g, splits) <= QUARTERS_MOST;
}
// Rows that fill as many tiles of 224 as of 256 (so at most 1568 of them) take those, on four wavefronts, in place of a plan of 256x256
// tiles, cut or not: the same tiles with an eighth less of padding (777 rows: 3.5 tile-rows of 256 in place of 4).  Products of the
// decoders' widths, 210 to 1560 tokens (us): 777 x 28672 x 4096 181 -> 170, with the SwiGLU epilogue 184 -> 169, 1340 x 28672 x 4096 280 ->
// 251, 777 x 22016 x 4096 with SwiGLU (on eight wavefronts before) 174 -> 158; both gradients, dX so: 0.98 to 1.08x, mean 1.02x (777 x 14336 x
// 4096 193 -> 184).
bool takes_224_rows(const GemmArgs& g) { return g.a_layout == 0 && (g.m + 223) / 224 == (g.m + 255) / 256; }
hipError_t launch_tiles(const GemmArgs& g, GemmTile tile, int splits, bool wide, hipStream_t s) {
  const GemmParams p = tile_params(g, tile, splits);
  const dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)splits);
  const int epi = g.swiglu_act ? EPI_SWIGLU : g.swiglu_dpre ? EPI_SWIGLU_BWD : !g.rope_table ? EPI_PLAIN : g.rope_head_dim == 128 ? EPI_ROPE128 : EPI_ROPE64;
  const bool at = g.a_layout != 0, bt = g.b_layout == 0, f32 = g.out_fp32 != 0;   // b_layout 0: stored [K, N], transposing reads
  if (tile == GemmTile::T64) return launch_gemm_small(p, at, bt, f32, grid, s);
  if (wide && fits_wide_form(g)) {
    if (at) return launch_gemm_wide<true, true>(p, tile, f32, epi, grid, s);
    return bt ? launch_gemm_wide<false, true>(p, tile, f32, epi, grid, s) : launch_gemm_wide<false, false>(p, tile, f32, epi, grid, s);
  }
  if (at) return bt ? launch_gemm_tile<true, true>(p, tile, f32, epi, grid, s) : launch_gemm_tile<true, false>(p, tile, f32, epi, grid, s);
  return bt ? launch_gemm_tile<false, true>(p, tile, f32, epi, grid, s) : launch_gemm_tile<false, false>(p, tile, f32, epi, grid, s);
}

// K no multiple of 64 with an operand whose contiguous dimension is k, or K = 0.
template <int BM, int BN, int WM, int WN>
hipError_t launch_general(const GemmArgs& g, hipStream_t s) {
  const GemmParams p = make_gemm_params(g, BM, BN);
  const dim3 grid((unsigned)(p.tiles_m * p.tiles_n)), block(64 * (BM / WM) * (BN / WN));
  const bool at = g.a_layout != 0, bt = g.b_layout == 0;
#define MLLM_GEMM_CASE(AT, BT, F32)                                                      \
  if (at == AT && bt == BT && (g.out_fp32 != 0) == F32) {                                \
    hipLaunchKernelGGL((gemm_kernel<BM, BN, WM, WN, AT, BT, F32>), grid, block, 0, s, p); \
    return hipGetLastError();                                                            \
  }
  MLLM_GEMM_CASE(false, true, false)
  MLLM_GEMM_CASE(false, false, false)
  MLLM_GEMM_CASE(true, true, true)
  MLLM_GEMM_CASE(false, true, true)
  MLLM_GEMM_CASE(false, false, true)
  MLLM_GEMM_CASE(true, true, false)
  MLLM_GEMM_CASE(true, false, false)
  MLLM_GEMM_CASE(true, false, true)
#undef MLLM_GEMM_CASE
  return hipErrorInvalidValue;
}

}  // namespace

// Tile and number of parts of the K loop.  A problem with few output tiles leaves CUs idle, one with a bit more
// than a multiple of 256 tiles an almost empty last round; cutting the K loop in `splits` parts (partial
// products in fp32 in a scratch buffer, summed in a fixed order afterwards) makes as many times more
// workgroups.  The plan is the cheapest of all choices by an estimate in microseconds: rounds of workgroups times
// (k-tiles of a part times the time of a k-tile, which grows with the number of workgroups that share power and
// memory, plus a workgroup's start and end), plus the parts' trip through memory.  The constants rank the choices and do
// not time a product (single products run up to 40 % off the estimate).  They are fitted to all tiles, parts and kernels of 1500
// random products of the layers' widths (96 to 24000 tokens), with weights (dW: the saved X) that are not in the memory-side
// cache, as a layer finds them; constants from products repeated on the same operands had sent a decoder's down projection to
// uncut 128x128 tiles (763 x 3584 x 18944: its forward pass 400 -> 468 us).  On 600 other products the plan's tile and parts lose
// 0.6 % in forward layout against the best measured (worst 22 %), 0.8 % with W stored [N, K] (worst 19 %) and 1.0 % for weight
// gradients (worst 14 %), on 200 whose operands stay in the cache 0.8, 1.0 and 1.2 %.
namespace {
struct GemmPlan { GemmTile tile; int splits; bool wide; };   // wide: on eight wavefronts, where the operands allow it
struct TileCost {
  GemmTile tile; bool wide; int bm, bn;
  int slots;              // workgroups of a round
  int few;                // up to this many, a k-tile costs k_few; from there on k_more, rising to k_full for a full round
  double k_few, k_more, k_full, fixed;   // fixed: start and end
};
// By layout: 0 forward, 1 both operands k-contiguous, 2 A stored [K, M] (weight gradients).
constexpr TileCost TILE_COSTS[3][6] = {{{GemmTile::T256, false, 256, 256, 256, 0, 0.83, 0.83, 1.35, 8.2},
                                        {GemmTile::T256, true, 256, 256, 256, 0, 1.16, 1.16, 1.25, 6.8},
                                        {GemmTile::T192, false, 192, 256, 256, 0, 0.74, 0.74, 1.06, 8.1},
                                        {GemmTile::T192, true, 192, 256, 256, 0, 0.76, 0.76, 1.12, 6.9},
                                        {GemmTile::T128, false, 128, 128, 512, 256, 0.51, 0.85, 0.95, 5.0},   // two on a CU from 257 on
                                        {GemmTile::T128, true, 128, 128, 256, 0, 0.26, 0.26, 0.49, 3.9}},
                                       {{GemmTile::T256, false, 256, 256, 256, 0, 0.91, 0.91, 1.29, 9.8},
                                        {GemmTile::T256, true, 256, 256, 256, 0, 0, 0, 0, 0},   // not for this layout
                                        {GemmTile::T192, false, 192, 256, 256, 0, 0.83, 0.83, 1.13, 6.8},
                                        {GemmTile::T192, true, 192, 256, 256, 0, 0, 0, 0, 0},   // not for this layout
                                        {GemmTile::T128, false, 128, 128, 512, 256, 0.49, 0.82, 0.98, 5.5},
                                        {GemmTile::T128, true, 128, 128, 256, 0, 0.28, 0.28, 0.49, 4.0}},
                                       {{GemmTile::T256, false, 256, 256, 256, 0, 1.04, 1.04, 1.42, 11.7},
                                        {GemmTile::T256, true, 256, 256, 256, 0, 0.88, 0.88, 1.44, 10.3},
                                        {GemmTile::T192, false, 192, 256, 256, 0, 0, 0, 0, 0},   // not for this layout
                                        {GemmTile::T192, true, 192, 256, 256, 0, 0, 0, 0, 0},   // not for this layout
                                        {GemmTile::T128, false, 128, 128, 512, 256, 0.47, 0.79, 1.00, 4.2},
                                        {GemmTile::T128, true, 128, 128, 256, 0, 0.37, 0.37, 0.48, 3.8}}};
inline int cost_row(bool a_t, bool b_t) { return a_t ? 2 : b_t ? 0 : 1; }   // b_t: B stored [K, N]
// Where a tile may go to eight wavefronts at all; below these lines the estimate decides, but for more than a round of large tiles in
// forward layout and weight gradients over more than 64 k-tiles, which then always do.  128x128: as long as every workgroup has a CU to itself (gain up to there 1.02-1.15 in every
// layout, loss of 2-10 % beyond).  The large tiles: not with both operands k-contiguous; else only for short contractions, as two
// stages do not cover the latency of weights that come from memory.  Time on four wavefronts / on eight, geomeans by k-tiles of
// a part: forward 192x256 up to 16 1.02-1.13, up to 32 0.93-1.0 below 1024 workgroups, beyond 0.79-0.99 (up to 64 with weights of up to 64 MB
// 0.83-0.96 for few workgroups, 1.0-1.04 from two rounds on); forward 256x256 up to 16
// 1.04-1.15, up to 32 0.98-1.10, up to 64 0.96-0.98 for at most a round and 1.01-1.04 for more, beyond 0.89-1.0; weight gradients
// up to 64 0.95-1.2, beyond 1.0-1.05 for a round or more of a matrix at least as wide as it is high (4096 x 28672 x 32768 5420 us and
// 5230), 0.85-1.0 for others.  Weights near the size of the memory-side cache, 256 MB, leave it before the next tile-rows
// come to them: more than a round of 256x256 tiles over 50 to 64 k-tiles 1.05 up to 192 MB, over that 0.99-1.02, but 1.07 where
// the last round is almost empty (forward pass of a decoder with 4096 x 28672 SwiGLU weights 0.94-0.995 at 300 to 28000 tokens, 1.04 at
// 1561, 784 workgroups; 4096 x 22016 1.00-1.03).  Gradients 37888 wide 0.95-0.98, 28672 1.04-1.08.
bool takes_wide_form(int row, GemmTile tile, int64_t m, int64_t n, int64_t k, int64_t k_tiles, int64_t workgroups) {
  if (tile == GemmTile::T128) return workgroups <= GEMM_CUS;
  if (row == 1) return false;
  if (row == 2) return n <= 32768 && (k_tiles <= 64 || (workgroups >= GEMM_CUS && n >= m));
  if (tile == GemmTile::T192) return k_tiles <= 24 || (k_tiles <= 64 && workgroups > 2 * GEMM_CUS && 2 * n * k <= (int64_t)64 << 20);
  return k_tiles <= 32 || (k_tiles <= 64 && workgroups > GEMM_CUS && (2 * n * k <= (int64_t)192 << 20 || workgroups % GEMM_CUS <= 16));
}
// A k-tile's time among `wgs` workgroups of at most a round.
double k_tile_time(const TileCost& c, int64_t wgs) {
  return wgs <= c.few ? c.k_few : c.k_more + (c.k_full - c.k_more) * (double)(wgs - c.few) / (c.slots - c.few);
}
// Estimate of `wgs` workgroups of k_tiles each.  Gradients of very wide matrices: the rows of 512 bytes of a 128x128 tile lie 80 KB
// and more apart (6144 x 28672 x 82 170 us with 128x128 tiles, 160 with 256x256; 14336 x 28672 x 294 632 and 473).
double workgroups_time(const TileCost& c, bool a_t, int64_t n, int64_t k_tiles, int64_t wgs) {
  const int64_t rounds = wgs / c.slots, rest = wgs % c.slots;
  const double fixed = c.fixed + (a_t && n > 20000 && c.tile == GemmTile::T128 ? 1.0 : 0.0);
  return (double)rounds * ((double)k_tiles * c.k_full + fixed) + (rest > 0 ? (double)k_tiles * k_tile_time(c, rest) + fixed : 0.0);
}
// What the parts cost besides: their trip through memory and a launch.
double parts_cost(int64_t m, int64_t n, int64_t parts) { return parts > 1 ? 3.0 + (double)m * n * (8.0 * parts + 4.0) * 1.15e-7 : 0.0; }
// split_bytes: scratch for the parts; the cheapest plan that fits it (and its estimate).  fused: only uncut 256x256 tiles, the ones that
// the fused epilogues exist for (and 224x256, which may take their place).
GemmPlan plan_gemm(int64_t m, int64_t n, int64_t k, bool a_t, bool b_t, size_t split_bytes, double* estimate = nullptr, bool fused = false) {
  const int row = cost_row(a_t, b_t);
  const int64_t nk = (k + BK - 1) / BK;
  GemmPlan best{GemmTile::T256, 1, false};
  if (m <= 0 || n <= 0 || k <= 0) return best;   // an empty product
  const int64_t most = std::min<int64_t>(16, std::min<int64_t>(nk / 8, (int64_t)(split_bytes / 4 / ((uint64_t)m * (uint64_t)n))));
  const int64_t cap = fused ? 1 : std::max<int64_t>(1, most);   // at least 8 k-tiles a part
  double best_cost = 1e300;
  for (const TileCost& c : TILE_COSTS[row]) {
    if ((c.tile == GemmTile::T192 && a_t) || (fused && c.tile != GemmTile::T256)) continue;   // T192: only for A stored [M, K]
    const int64_t tiles = ((m + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn);
    for (int64_t sp = 1; sp <= cap; sp++) {
      const int64_t per = (nk + sp - 1) / sp;
      if ((nk + per - 1) / per != sp) continue;   // would leave a part empty
      if ((sp - 1) * tiles >= 512) break;         // the chip is full without
      const bool eight = takes_wide_form(row, c.tile, m, n, k, per, tiles * sp);
      if (c.wide ? !eight : eight && row == 0 && c.tile != GemmTile::T128 && tiles * sp > GEMM_CUS) continue;
      const double cost = workgroups_time(c, a_t, n, per, tiles * sp) + parts_cost(m, n, sp);
      if (cost < best_cost * (1 - 1e-9)) { best_cost = cost; best = {c.tile, (int)sp, c.wide}; }
    }
  }
  // Long weight gradients: the estimates of the two kernels lie within 1 % of each other, the times do not (takes_wide_form).
  const int64_t per = (nk + best.splits - 1) / best.splits, wgs = ((m + 255) / 256) * ((n + 255) / 256) * best.splits;
  if (row == 2 && best.tile == GemmTile::T256 && per > 64) best.wide = takes_wide_form(row, best.tile, m, n, k, per, wgs);
  if (estimate) *estimate = best_cost;
  return best;
}
}  // namespace

namespace {
// A linear map's input gradient x = dY [T, n] . W^T [n, k] and weight gradient w = X^T [k, T] . dY [T, n] in one launch:
// neither needs the other, the second starts on the CUs that the first one's last round leaves idle, and a launch and its
// gap go.  The plan takes tiles, parts and order together, as the cheapest estimate of the whole launch: the workgroups of
// the first product, then those of the second, each on the first slot that is free.  Constants fitted to 780 maps of the layers'
// widths (64 to 30000 tokens), weights and saved X not in the memory-side cache; on 150 others the plan loses 0.7 % against the best of
// all choices (worst 40 %: 2479 x 1280 x 3840 (T, k, n) 75 us and 53), and on 442 that it pairs one launch takes
// 0.83 of the time of two with the plans of their own.  Examples (us): 576 x 1024 x 4096 26.6 -> 21.7, 256 x 256 x 768 14.2 -> 8.4,
// 2880 x 1024 x 3072 52 -> 43, 5125 x 3200 x 12800 737 -> 628.
struct PairPlan { GemmPlan x, w; bool x_first, pays; };
constexpr TileCost PAIR_COSTS[2][3] = {{{GemmTile::T256, false, 256, 256, 256, 0, 0.66, 0.66, 1.21, 9.9},
                                        {GemmTile::T192, false, 192, 256, 256, 0, 0.61, 0.61, 1.07, 6.6},
                                        {GemmTile::T128, false, 128, 128, 512, 256, 0.31, 0.41, 0.93, 4.7}},
                                       {{GemmTile::T256, false, 256, 256, 256, 0, 1.08, 1.08, 1.26, 8.3},
                                        {GemmTile::T192, false, 192, 256, 256, 0, 0, 0, 0, 0},   // not for this layout
                                        {GemmTile::T128, false, 128, 128, 512, 256, 0.41, 0.70, 0.84, 2.7}}};
constexpr double FEW_128[2] = {4.8, 3.8};       // start and end of both in 128x128 tiles on eight wavefronts (up to 256 workgroups)
constexpr double MIXED_128[2] = {0.62, 0.52};   // a k-tile of a 128x128 tile that has its CU to itself beside large tiles
constexpr double LONGEST = 0.07;                // workgroups do not all take the same time: long ones delay the end more often
constexpr int MOST_PARTS = 8;
struct PairSide {   // one choice for one of the products
  const TileCost* c; int splits; int64_t per, wgs; double fixed, parts; size_t bytes;
};
// The time after which na workgroups of da each and then nb of db each have run on `slots` slots.
double makespan(int64_t na, double da, int64_t nb, double db, int64_t slots) {
  const int64_t rounds = na / slots, rest = na % slots, early = slots - rest;   // `early` slots are free one da before the others
  const double t1 = (double)rounds * da, t2 = t1 + da;
  const double q = std::floor(da / db);                                         // workgroups that an early slot takes by then
  const double alone = std::ceil((double)nb / (double)early);
  double end;
  if (rest == 0 || alone <= q) {
    end = t1 + alone * db;
  } else {
    const double lag = q + (da > q * db * (1 + 1e-9) ? 1.0 : 0.0);
    const double i = std::max(1.0, std::ceil(((double)nb + (double)rest * lag) / (double)slots));
    const double j = std::max(1.0, std::ceil(((double)nb - (double)early * q) / (double)slots));
    end = std::min(t1 + i * db, t2 + j * db);
  }
  return std::max(end, rest > 0 ? t2 : t1);
}
int pair_sides(PairSide (&out)[3 * MOST_PARTS], int64_t m, int64_t n, int64_t k, bool a_t, bool only_256, size_t bytes) {
  const int64_t nk = (k + BK - 1) / BK;
  int count = 0;
  for (const TileCost& c : PAIR_COSTS[a_t ? 1 : 0]) {
    if ((c.tile == GemmTile::T192 && a_t) || (only_256 && c.tile != GemmTile::T256)) continue;
    const int64_t tiles = ((m + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn);
    for (int64_t sp = 1; sp <= MOST_PARTS && (sp == 1 || (!only_256 && sp <= nk / 8 && (sp - 1) * tiles < 512)); sp++) {
      const int64_t per = (nk + sp - 1) / sp;
      const size_t need = sp > 1 ? (size_t)sp * (size_t)m * (size_t)n * 4 : 0;
      if ((nk + per - 1) / per != sp || need > bytes) continue;
      out[count++] = {&c, (int)sp, per, tiles * sp, c.fixed, parts_cost(m, n, sp), need};
    }
  }
  return count;
}
PairPlan plan_pair(int64_t t, int64_t k, int64_t n, bool swiglu, size_t split_bytes) {
  PairSide xs[3 * MOST_PARTS], ws[3 * MOST_PARTS];
  const int nx = pair_sides(xs, t, k, n, false, swiglu, split_bytes), nw = pair_sides(ws, k, n, t, true, false, split_bytes);
  PairPlan best{{GemmTile::T256, 1, false}, {GemmTile::T256, 1, false}, true, true};
  double best_cost = 1e300;
  for (int i = 0; i < nx; i++)
    for (int j = 0; j < nw; j++) {
      const PairSide &x = xs[i], &w = ws[j];
      if (x.bytes + w.bytes > split_bytes) continue;
      const bool x128 = x.c->tile == GemmTile::T128, w128 = w.c->tile == GemmTile::T128, both = x128 && w128;
      const int64_t slots = both ? 512 : 256, wgs = std::min(x.wgs + w.wgs, slots);
      const bool few = both && wgs <= GEMM_CUS;
      const double dx = (double)x.per * (x128 && !both ? MIXED_128[0] : k_tile_time(*x.c, wgs)) + (few ? FEW_128[0] : x.fixed);
      const double dw = (double)w.per * (w128 && !both ? MIXED_128[1] : k_tile_time(*w.c, wgs)) + (few ? FEW_128[1] : w.fixed);
      const double besides = x.parts + w.parts + LONGEST * std::max(dx, dw);
      for (const bool x_first : {true, false}) {
        const double cost = besides + (x_first ? makespan(x.wgs, dx, w.wgs, dw, slots) : makespan(w.wgs, dw, x.wgs, dx, slots));
        if (cost < best_cost * (1 - 1e-9)) { best_cost = cost; best = {{x.c->tile, x.splits, false}, {w.c->tile, w.splits, false}, x_first, true}; }
      }
    }
  // A long launch runs at the power cap: work packed tighter lowers the clock, and two products side by side evict each
  // other's panels.  Two launches / one, by the ratio of the estimates, alone: over 540 us 1.05-1.1 below 0.86, 1.02-1.05 up to 0.92,
  // 1.0 beyond; in a layer 5125 x 3200 x 12800 (0.79) 711 -> 630, but 2999 x 3584 x 37888 (0.87) makes it 0.6-1.7 % slower and
  // 8192 x 4096 x {12288, 22016} (0.92, 0.93) 1.0 %.  From 140 to 540 us 1.05-1.2 below 0.9, 1.0-1.04 up to 1.0; a 1024-wide layer on
  // 13824 tokens (0.87-0.95) 1555 -> 1510.  Shorter ones always gain by the launch that goes.
  // The SwiGLU gradient's epilogue moves three matrices while no matrix core works; beside another product's k-loops that is
  // hidden (8192 x 11008 x 4096 1226 -> 1119 us, 32768 x 14336 x 4096 6006 -> 5790).
  if (!swiglu && best_cost > 140) {
    double x_alone, w_alone;
    plan_gemm(t, k, n, false, false, split_bytes, &x_alone);
    plan_gemm(k, n, t, true, true, split_bytes, &w_alone);
    best.pays = best_cost * (best_cost > 540 ? 1.16 : 1.0) < x_alone + w_alone + 2.5;
  }
  return best;
}
size_t part_bytes(const GemmPlan& p, int64_t m, int64_t n) { return p.splits > 1 ? (size_t)p.splits * (size_t)m * (size_t)n * 4 : 0; }
}  // namespace

size_t gemm_splitk_ws_bytes(int64_t m, int64_t n, int64_t k, bool a_t, bool b_t) {
  const GemmPlan pl = plan_gemm(m, n, k, a_t, b_t, SIZE_MAX);
  return pl.splits > 1 ? (size_t)pl.splits * (size_t)m * (size_t)n * 4 : 0;
}

// The fused epilogues exist for 256x256 and 224x256 tiles; with fewer than this many of them a plan of its own for the product and a
// pass of its own for the activation or the rotation are as good.  The line is flat: forward and backward of the three
// decoder layers at 256 to 3072 tokens, 100 instead of 200 takes 1.002x the time on average (0.989-1.021), 300 0.997x
// (0.978-1.014).
static bool fills_chip(int64_t m, int64_t n) { return ((m + 255) / 256) * ((n + 255) / 256) >= 200; }

bool gemm_swiglu_fusable(int64_t m, int64_t n, int64_t k) {
  return fills_chip(m, n) && n % 256 == 0 && k >= BK && k % BK == 0;
}

bool gemm_swiglu_bwd_fusable(int64_t m, int64_t n, int64_t k) {
  return fills_chip(m, n) && n % 8 == 0 && k >= BK && k % BK == 0;
}

bool gemm_rope_fusable(int64_t m, int64_t n, int64_t k, int32_t head_dim) {
  return fills_chip(m, n) && (head_dim == 64 || head_dim == 128) && n % 8 == 0 && k >= BK && k % BK == 0;
}

namespace {
// The plan of a product that takes the tile kernel, with the tiles that run (224 rows in place of 256, quarters in place of
// 128x128): the launch and gemm_form both go by it.  With both operands k-contiguous the large tiles are loaded straight
// into LDS, 16 bytes a lane, which is only known to work from addresses that are multiples of 16; operands that start
// elsewhere (a tensor inside a larger buffer) take 128x128 tiles, whose loads go through registers.
GemmPlan plan_of(const GemmArgs& g) {
  if (!takes_tile_kernel(g)) return {GemmTile::T256, 1, false};
  if (g.a_layout == 0 && g.b_layout == 1 && (((uintptr_t)g.a | (uintptr_t)g.b) & 15)) return {GemmTile::T128, 1, false};
  const bool fused = g.swiglu_act || g.swiglu_dpre || g.rope_table;
  const bool split_ok = g.splitk_ws && g.ldc == g.n && g.n % 8 == 0;
  GemmPlan pl = plan_gemm(g.m, g.n, g.k, g.a_layout != 0, g.b_layout == 0, split_ok ? g.splitk_ws_bytes : 0, nullptr, fused);
  if (pl.tile == GemmTile::T256 && takes_224_rows(g)) pl = {GemmTile::T224, pl.splits, false};
  if (pl.tile == GemmTile::T128 && takes_quarters(g, pl.splits)) pl.tile = GemmTile::T64;
  return pl;
}
}  // namespace

GemmForm gemm_form(const GemmArgs& g) {
  if (!takes_tile_kernel(g)) return {0, 0, 1};
  const GemmPlan pl = plan_of(g);
  return {tile_rows(pl.tile), tile_cols(pl.tile), pl.splits};
}

namespace {
// The product as its K parts: partial results to the scratch, everything that the epilogue adds left to the reduction.
GemmArgs part_of(const GemmArgs& g) {
  GemmArgs part = g;
  part.c = g.splitk_ws;
  part.out_fp32 = 1;
  part.accumulate = 0;
  part.bias = nullptr;
  part.residual = nullptr;
  return part;
}
hipError_t reduce_parts(const GemmArgs& g, int splits, hipStream_t s) {
  return launch_splitk_reduce((const float*)g.splitk_ws, g.c, splits, g.m, g.n, g.out_fp32, g.accumulate, g.bias, g.residual, g.ldres, s);
}
}  // namespace

// What no form of a product accepts.
static bool refused(const GemmArgs& g) {
  if (g.rope_table && (!g.rope_pos || !gemm_rope_fusable(g.m, g.n, g.k, g.rope_head_dim) || g.a_layout != 0 ||
                       g.b_layout != 0 || g.out_fp32 || g.residual || g.swiglu_act || g.swiglu_dpre || g.ldc != g.n ||
                       g.rope_cols % 128 != 0 || g.rope_cols > g.n))
    return true;
  if ((g.swiglu_dpre || g.swiglu_pre) &&
      (!g.swiglu_dpre || !g.swiglu_pre || g.swiglu_act || !gemm_swiglu_bwd_fusable(g.m, g.n, g.k) || g.a_layout != 0 ||
       g.b_layout != 1 || g.out_fp32 || g.bias || g.residual || g.ldc != 2 * g.n))
    return true;
  if (g.swiglu_act && (!gemm_swiglu_fusable(g.m, g.n, g.k) || g.a_layout != 0 || g.b_layout != 0 || g.out_fp32 ||
                       g.bias || g.residual || g.ldc != g.n))
    return true;
  // operands are addressed through 32-bit buffer offsets
  if ((g.a_layout ? g.k : g.m) * g.lda * 2 > GEMM_MAX_OPERAND_BYTES || (g.b_layout ? g.n : g.k) * g.ldb * 2 > GEMM_MAX_OPERAND_BYTES)
    return true;
  // the epilogue addresses a sub-tile of up to 128 rows with 32-bit offsets from its first element
  if (g.ldc * (g.out_fp32 ? 4 : 2) * 128 > 0xFFFFFFFFll || (g.residual && g.ldres * 2 * 128 > 0xFFFFFFFFll))
    return true;
  return false;
}

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
  if (g.m <= 0 || g.n <= 0) return hipSuccess;
  if (refused(g)) return hipErrorInvalidValue;
  const bool tiled = takes_tile_kernel(g);
  const GemmPlan pl = plan_of(g);
  // timing classes: the three layouts of the large tiles, the 192-row form, and the small tiles
  const bool small = tiled ? pl.tile == GemmTile::T128 || pl.tile == GemmTile::T64 : !fills_chip(g.m, g.n);
  const int cls = small ? PROF_GEMM_SMALL : pl.tile == GemmTile::T192 ? PROF_GEMM_ROWS192
                  : g.a_layout ? PROF_GEMM_DW : (g.b_layout ? PROF_GEMM_DX : PROF_GEMM_FWD);
  const double flops = 2.0 * (double)g.m * (double)g.n * (double)g.k;
  if (pl.splits == 1) {
    ProfScope prof(cls, flops, s);
    if (tiled) return launch_tiles(g, pl.tile, 1, pl.wide, s);
    // 256x256 tiles (8 wavefronts of 128x64) once they fill the chip; smaller problems keep
    // 128x128 tiles so that more workgroups exist
    return small ? launch_general<128, 128, 64, 64>(g, s) : launch_general<256, 256, 128, 64>(g, s);
  }
  hipError_t e;
  {
    ProfScope prof(cls, flops, s);
    e = launch_tiles(part_of(g), pl.tile, pl.splits, pl.wide, s);
  }
  return e != hipSuccess ? e : reduce_parts(g, pl.splits, s);
}


// Whether the two gradients may share a launch: both take the tile kernel, on operands that start on 16 bytes (they are
// loaded straight to LDS).
static bool pairable(const GemmArgs& x, const GemmArgs& w) {
  return x.m > 0 && x.n > 0 && w.m > 0 && w.n > 0 && takes_tile_kernel(x) && takes_tile_kernel(w) && (((uintptr_t)x.a | (uintptr_t)x.b | (uintptr_t)w.a | (uintptr_t)w.b) & 15) == 0;
}

// The plan of both gradients of operands that may share a launch, with the tiles that run: quarters of 128x128 tiles (takes_quarters)
// in place of a plan with both in these, and 224 rows for dX.  The launch and linear_bwd_form both go by it.
// Up to 256 quarters, the same maps and tokens as there: uncut 1.20 to 1.34x (83 maps), with a product in parts 1.13 to 1.20x (20); 257 to
// 512 0.80 to 1.37x, geomean 1.0x, and 0.80 to 1.12x with parts.
static PairPlan pair_plan_of(const GemmArgs& x, const GemmArgs& w) {
  PairPlan pl = plan_pair(x.m, x.n, x.k, x.swiglu_dpre != nullptr, x.splitk_ws ? x.splitk_ws_bytes : 0);
  if (pl.x.tile == GemmTile::T256 && takes_224_rows(x)) pl.x.tile = GemmTile::T224;
  if (pl.x.tile == GemmTile::T128 && pl.w.tile == GemmTile::T128 && !x.swiglu_dpre &&
      quarters(x, pl.x.splits) + quarters(w, pl.w.splits) <= QUARTERS_MOST)
    pl.x.tile = pl.w.tile = GemmTile::T64;
  return pl;
}

LinearBwdForm linear_bwd_form(const GemmArgs& x, const GemmArgs& w) {
  if (!pairable(x, w)) return {false, gemm_form(x), gemm_form(w), false};
  const PairPlan pl = pair_plan_of(x, w);
  if (!pl.pays) return {false, gemm_form(x), gemm_form(w), false};
  auto form = [](const GemmPlan& p) { return GemmForm{tile_rows(p.tile), tile_cols(p.tile), p.splits}; };
  return {true, form(pl.x), form(pl.w), pl.x_first};
}

// Enough for one launch and for two: which it will be also hangs on where the operands start.
size_t linear_bwd_ws_bytes(int64_t t, int64_t k, int64_t n, bool swiglu) {
  if (t <= 0) return 0;
  GemmArgs x{}, w{};
  x.m = t; x.n = k; x.k = n; x.lda = x.ldb = n; x.b_layout = 1;
  w.m = k; w.n = n; w.k = t; w.lda = k; w.ldb = n; w.a_layout = 1;
  const size_t apart = std::max(swiglu || !takes_tile_kernel(x) ? 0 : gemm_splitk_ws_bytes(t, k, n, false, false),
                                takes_tile_kernel(w) ? gemm_splitk_ws_bytes(k, n, t, true, true) : 0);
  if (!pairable(x, w)) return apart;
  const PairPlan pl = plan_pair(t, k, n, swiglu, SIZE_MAX);
  return pl.pays ? std::max(apart, part_bytes(pl.x, t, k) + part_bytes(pl.w, k, n)) : apart;
}

// Whether one of the gradients is written over something that the other product reads: as two launches, dW first, dX may take
// the place of X.
static bool gradients_over_operands(const GemmArgs& x, const GemmArgs& w) {
  const int64_t dy = x.m * x.lda * 2, act = w.k * w.lda * 2, weight = x.n * x.ldb * 2;
  const void* dx = x.swiglu_dpre ? x.swiglu_dpre : x.c;
  const int64_t dx_bytes = x.m * x.ldc * 2, dw_bytes = w.m * w.ldc * 4;
  return ranges_overlap(dx, dx_bytes, w.a, act) || ranges_overlap(dx, dx_bytes, w.b, dy) || ranges_overlap(w.c, dw_bytes, x.a, dy) ||
         ranges_overlap(w.c, dw_bytes, x.b, weight) || ranges_overlap(w.c, dw_bytes, x.swiglu_pre, x.m * 2 * x.n * 2) ||
         ranges_overlap(dx, dx_bytes, w.c, dw_bytes);
}

hipError_t launch_linear_bwd(const GemmArgs& x, const GemmArgs& w, hipStream_t s) {
  const bool pair = pairable(x, w) && !gradients_over_operands(x, w);
  const PairPlan pl = pair ? pair_plan_of(x, w) : PairPlan{};
  if (!pair || !pl.pays) {
    const hipError_t e = launch_gemm(w, s);
    return e != hipSuccess ? e : launch_gemm(x, s);
  }
  if (refused(x) || refused(w)) return hipErrorInvalidValue;
  GemmArgs xa = x, wa = w;   // the parts of both are in the scratch at the same time
  wa.splitk_ws = (char*)x.splitk_ws + part_bytes(pl.x, x.m, x.n);
  const GemmArgs xp = pl.x.splits > 1 ? part_of(xa) : xa, wp = pl.w.splits > 1 ? part_of(wa) : wa;
  GemmPairParams p;
  p.x = tile_params(xp, pl.x.tile, pl.x.splits);
  p.w = tile_params(wp, pl.w.tile, pl.w.splits);
  p.x_tiles = p.x.tiles_m * p.x.tiles_n;
  p.w_tiles = p.w.tiles_m * p.w.tiles_n;
  const int x_wgs = p.x_tiles * pl.x.splits, w_wgs = p.w_tiles * pl.w.splits;
  p.x_first = pl.x_first;
  p.first = pl.x_first ? x_wgs : w_wgs;
  hipError_t e;
  {
    const bool in_quarters = pl.x.tile == GemmTile::T64, small = in_quarters || (pl.x.tile == GemmTile::T128 && pl.w.tile == GemmTile::T128);
    ProfScope prof(small ? PROF_GEMM_SMALL : PROF_GEMM_DX, 4.0 * (double)x.m * (double)x.n * (double)x.k, s);
    e = in_quarters ? launch_gemm_pair_small(p, xp.out_fp32 != 0, x_wgs + w_wgs, s)
                    : launch_gemm_pair_tiles(p, pl.x.tile, xp.out_fp32 != 0, x.swiglu_dpre ? EPI_SWIGLU_BWD : EPI_PLAIN, pl.w.tile, x_wgs + w_wgs, s);
  }
  if (e == hipSuccess && pl.x.splits > 1) e = reduce_parts(xa, pl.x.splits, s);
  if (e == hipSuccess && pl.w.splits > 1) e = reduce_parts(wa, pl.w.splits, s);
  return e;
}

}  // namespace mllm
