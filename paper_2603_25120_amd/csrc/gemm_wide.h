// The form of the MFMA GEMM kernel with two wavefronts on a SIMD: (32 WM) x (64 WN) x 64 tiles on eight wavefronts (2 x 4), each
// owning WM x WN blocks of v_mfma_f32_16x16x32_bf16, both operands loaded straight to LDS.
#pragma once
#include "gemm_tile.h"

namespace mllm {

namespace {

// ---------------------------------------------------------------------------------------------
// Why eight wavefronts.  A wavefront alone on its SIMD issues an instruction every 5 clocks or so, whatever it is: the
// fragment reads, LDS stores, loads and scalar work of a k-tile take as long as its MFMAs, and no order of them hides
// that.  With two, one issues under the other's MFMAs, the staging registers and their LDS stores go, and direct loads of
// operands stored [K, .] are no longer late.  The price is LDS reads: 192 KB a k-tile of 256x256 where four wavefronts of
// 128x128 read 128 KB, which on long contractions at the power cap costs more than it gives; and two stages look one k-tile
// ahead, which does not cover the latency of operands that come from memory (where the line lies then: takes_wide_form in
// gemm.hip).  No SwiGLU gradient: its product has both operands k-contiguous and 256x256 tiles.
// Four wavefronts -> eight, one card, in turn, operands in the memory-side cache (us):
//   256x256, B stored [K, N]: 26496 x 4096 x 1024 206 -> 188, 5125 x 12800 x 3200 357 -> 335, 4096 x 4096 x 4096 100 -> 95, 32768 x 28672 x
//   4096 5550 -> 5330, 32768 x 4096 x 14336 2710 -> 2750; both [K, .]: 4096 x 28672 x 32768 5420 -> 5230, 3200 x 12800 x 5125
//   347 -> 332; both k-contiguous: 26496 x 4096 x 1024 187 -> 186, 32768 x 4096 x 28672 4990 -> 5400.
//   128x128 with four stages, at most one workgroup for every CU: 256 x 192 x 192 5.2 -> 4.6, 576 x 4096 x 1024 10.9 -> 9.1, 2880 x
//   1024 x 4096 30.6 -> 27.0, 777 x 4096 x 4096 34 -> 28; with more workgroups than CUs two of the four-wavefront
//   form on a CU overlap their starts and ends, 2880 x 4096 x 1024 27.5 -> 28.3, 4096 x 4096 x 576 24.3 -> 26.9.
// The k-loop is written slot by slot as in gemm_tile.h.  A tile's loads go out in the second k-step, behind the one barrier of a
// k-tile: 3 slots apart at 256x256 (1, 2, 3, 4 slots: 180.6, 181.4, 178.9, 179.6 us at 26496 x 4096 x 1024), behind the
// fragment reads at 128x128.  Loads straight to LDS want operands that start on 16 bytes.
// ---------------------------------------------------------------------------------------------
// NST: LDS stages, two (256 and 192 rows) or four (128x128; As2 .. Bs3 are not used with two).  All of them distinct
// variables of the kernel, or halves of such.
template <int WM, int WN, int NST, bool A_T, bool B_T, bool OUT_F32, int EPI>
__device__ __forceinline__ void gemm_wide_tile(GemmParams p, int pid, int nblk, int split, bf16_t* As0, bf16_t* As1, bf16_t* As2, bf16_t* As3,
                                               bf16_t* Bs0, bf16_t* Bs1, bf16_t* Bs2, bf16_t* Bs3) {
  constexpr int BM = 32 * WM, BN = 64 * WN, NU = WM + WN, NS = WM * WN;
  using TA = TileLoader16<BM, A_T, 8>;
  using TB = TileLoader16<BN, B_T, 8>;
  constexpr int NA = TA::PER_WAVE, NL = NA + TB::PER_WAVE;
  constexpr int AHEAD = NST == 2 ? 2 : NST - 1;
  constexpr int RS = NS >= 2 * NU + 4 ? 2 : 1;
  constexpr int LOAD_AT = NST == 2 ? 1 : NS - NL, LOAD_STEP = NST == 2 ? 3 : 1;
  static_assert(LOAD_AT + (NL - 1) * LOAD_STEP < NS, "the loads go out in one k-step");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  int tm, tn;
  tile_of_block(pid, nblk, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  TA la;
  TB lb;
  la.init(p.lda, m0, p.M, lane, wave);
  lb.init(p.ldb, n0, p.N, lane, wave, EPI == EPI_SWIGLU ? p.N >> 1 : 0, 8 * WN);
  const int kt0 = split * p.kt_per_split;
  const int last_tile = (int)((p.K + BK - 1) / BK) - 1;
  const int nk = min(p.kt_per_split, last_tile + 1 - kt0);
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  auto source = [&](uint32_t kstep, const bf16_t* base, uint32_t bytes, int kt) __attribute__((always_inline)) {
    const bool have = kt < nk;
    const uint32_t k = (uint32_t)(have ? kt0 + kt : 0);
    return TileSource{make_rsrc(base, have ? bytes : 0u), k * kstep};
  };
  auto a_stage = [&](auto i_c) __attribute__((always_inline)) -> bf16_t* {
    constexpr int i = decltype(i_c)::value % NST;
    return i == 0 ? As0 : i == 1 ? As1 : i == 2 ? As2 : As3;
  };
  auto b_stage = [&](auto i_c) __attribute__((always_inline)) -> bf16_t* {
    constexpr int i = decltype(i_c)::value % NST;
    return i == 0 ? Bs0 : i == 1 ? Bs1 : i == 2 ? Bs2 : Bs3;
  };
  auto load_direct = [&](auto q_c, auto st_c, const TileSource& sa, const TileSource& sb) __attribute__((always_inline)) {
    constexpr int q = decltype(q_c)::value;
    if constexpr (q < NA) la.template load_to_lds<q>(sa, a_stage(st_c), wave);
    else lb.template load_to_lds<q - NA>(sb, b_stage(st_c), wave);
  };
  bf16x8 af[2][WM], bfr[2][WN];
  auto fetch_unit = [&](auto u_c, auto kk_c, const bf16_t* at, const bf16_t* bt) __attribute__((always_inline)) {
    constexpr int u = decltype(u_c)::value, kk = decltype(kk_c)::value;
    if constexpr (u == 0) af[kk][0] = TA::frag(at, wm * 16 * WM, kk, lane);
    else if constexpr (u <= WN) bfr[kk][u - 1] = TB::frag(bt, wn * 16 * WN + 16 * (u - 1), kk, lane);
    else af[kk][u - WN] = TA::frag(at, wm * 16 * WM + 16 * (u - WN), kk, lane);
  };
  // Prologue: the first AHEAD tiles are requested together (one exposed latency for all of them).
  static_for<AHEAD>([&](auto t_c) __attribute__((always_inline)) {
    const TileSource sa = source(la.kstep, p.a, p.a_bytes, decltype(t_c)::value), sb = source(lb.kstep, p.b, p.b_bytes, decltype(t_c)::value);
    static_for<NL>([&](auto q) { load_direct(q, t_c, sa, sb); });
  });
  f32x4 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; i++)
#pragma unroll
    for (int j = 0; j < WN; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  __builtin_amdgcn_sched_barrier(0);
  constexpr int VM0 = (AHEAD - 1) * NL, VM = NST == 2 ? 0 : (NST - 3) * NL;
  __builtin_amdgcn_s_waitcnt(0x0F70 | (VM0 & 15) | ((VM0 >> 4) << 14));   // tile 0 has landed
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  static_for<NU>([&](auto u) { fetch_unit(u, C0{}, As0, Bs0); });

  auto iteration = [&](auto s_c, int kt) __attribute__((always_inline)) {
    constexpr int S = decltype(s_c)::value;
    using NEXT = std::integral_constant<int, S + 1>;
    using FREE = std::integral_constant<int, S + AHEAD>;
    const TileSource sa = source(la.kstep, p.a, p.a_bytes, kt + AHEAD), sb = source(lb.kstep, p.b, p.b_bytes, kt + AHEAD);
    auto slot = [&](auto kk_c, auto m_c) __attribute__((always_inline)) {
      constexpr int kk = decltype(kk_c)::value, m = decltype(m_c)::value;
      if constexpr (kk == 1 && m == 0) {
        // Tile kt + 1 has landed, this wavefront's share of it (with four stages those of tile kt + 2 may still be on their
        // way).  The stage that the next loads fill is free: with four it held tile kt - 1, whose fragments have long
        // been operands of MFMAs; with two it holds this tile, whose last fragments this wavefront waits for.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt((NST == 2 ? 0x0070 : 0x0F70) | (VM & 15) | ((VM >> 4) << 14));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (m % RS == 0 && m / RS < NU) {
        using U = std::integral_constant<int, m / RS>;
        if constexpr (kk == 0) fetch_unit(U{}, C1{}, a_stage(s_c), b_stage(s_c));
        else fetch_unit(U{}, C0{}, a_stage(NEXT{}), b_stage(NEXT{}));
      }
      if constexpr (kk == 1) {
        static_for<NL>([&](auto q_c) __attribute__((always_inline)) {
          if constexpr (m == LOAD_AT + decltype(q_c)::value * LOAD_STEP) load_direct(q_c, FREE{}, sa, sb);
        });
      }
      constexpr int i = m / WN, j = (i & 1) ? WN - 1 - m % WN : m % WN;
      mfma_in_place(acc[i][j], bfr[kk][j], af[kk][i]);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<NS>([&](auto m) __attribute__((always_inline)) { slot(C0{}, m); });
    static_for<NS>([&](auto m) __attribute__((always_inline)) { slot(C1{}, m); });
  };
  int kt = 0;
  for (; kt + NST - 1 < nk; kt += NST) static_for<NST>([&](auto s) __attribute__((always_inline)) { iteration(s, kt + decltype(s)::value); });
  static_for<NST - 1>([&](auto s) __attribute__((always_inline)) { if (kt + decltype(s)::value < nk) iteration(s, kt + decltype(s)::value); });
  __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0): loads past the end land where the epilogue stages its rows
  mfma_results_ready();
  int lane_out = lane;
  asm volatile("" : "+v"(lane_out));
#pragma unroll
  for (int i = 0; i < WM; i++)
#pragma unroll
    for (int j = 0; j < WN; j++) asm volatile("" : "+a"(acc[i][j]));   // no read above the wait
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  bf16_t* const part = wave < 2 ? As0 : wave < 4 ? As1 : wave < 6 ? Bs0 : Bs1;   // two wavefronts to a stage
  static_assert(2 * 2 * 16 * (16 * WN + 4) * 2 <= (TA::SIZE < TB::SIZE ? TA::SIZE : TB::SIZE), "two staged rows of blocks of two wavefronts in a tile's LDS");
  uint32_t* const out_stage = reinterpret_cast<uint32_t*>(part) + (wave & 1) * 2 * 16 * (16 * WN + 4);
  if constexpr (OUT_F32) p.c = reinterpret_cast<float*>(p.c) + split * p.c_split_stride;
  const int64_t row0 = m0 + wm * 16 * WM, col0 = n0 + wn * 16 * WN;
  if constexpr (EPI == EPI_SWIGLU) store_blocks_swiglu<WM, WN>(p, acc, row0, (n0 >> 1) + 8 * WN * wn, lane_out, out_stage);
  else store_blocks<WM, WN, OUT_F32, EPI == EPI_ROPE64 ? 64 : 0>(p, acc, row0, col0, lane_out, out_stage);
}

template <int WM, int WN, int NST, bool A_T, bool B_T, bool OUT_F32, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_wide_kernel(GemmParams p) {
  constexpr int SA = 32 * WM * BK, SB = 64 * WN * BK;
  __shared__ __attribute__((aligned(1024))) bf16_t As0[SA], As1[SA], Bs0[SB], Bs1[SB];
  if constexpr (NST == 2) {
    gemm_wide_tile<WM, WN, NST, A_T, B_T, OUT_F32, EPI>(p, blockIdx.x, gridDim.x, blockIdx.y, As0, As1, nullptr, nullptr, Bs0, Bs1, nullptr, nullptr);
  } else {
    __shared__ __attribute__((aligned(1024))) bf16_t As2[SA], As3[SA], Bs2[SB], Bs3[SB];
    gemm_wide_tile<WM, WN, NST, A_T, B_T, OUT_F32, EPI>(p, blockIdx.x, gridDim.x, blockIdx.y, As0, As1, As2, As3, Bs0, Bs1, Bs2, Bs3);
  }
}

}  // namespace

template <bool A_T, bool B_T>
hipError_t launch_gemm_wide(const GemmParams& p, GemmTile tile, bool out_f32, int epi, dim3 grid, hipStream_t s) {
  if (p.K <= 0 || (p.K % BK != 0 && !(A_T && B_T))) return hipErrorInvalidValue;
#define MLLM_WIDE(WM, WN, NST, F32, EPI)                                                                          \
  do {                                                                                                            \
    hipLaunchKernelGGL((gemm_wide_kernel<WM, WN, NST, A_T, B_T, F32, EPI>), grid, dim3(512), 0, s, p);            \
    return hipGetLastError();                                                                                     \
  } while (0)
#define MLLM_WIDE_TYPES(WM, WN, NST)                 \
  do {                                               \
    if (out_f32) MLLM_WIDE(WM, WN, NST, true, EPI_PLAIN); \
    else MLLM_WIDE(WM, WN, NST, false, EPI_PLAIN);   \
  } while (0)
  if constexpr (!A_T && B_T) {
    if (epi == EPI_SWIGLU && tile == GemmTile::T256) MLLM_WIDE(8, 4, 2, false, EPI_SWIGLU);
    if (epi == EPI_ROPE64 && tile == GemmTile::T256) MLLM_WIDE(8, 4, 2, false, EPI_ROPE64);
  }
  if (epi != EPI_PLAIN) return hipErrorInvalidValue;
  if (tile == GemmTile::T128) MLLM_WIDE_TYPES(4, 2, 4);
  if constexpr (B_T) {   // with both operands k-contiguous the four-wavefront form of the large tiles is better
    if (tile == GemmTile::T256) MLLM_WIDE_TYPES(8, 4, 2);
    if constexpr (!A_T) {
      if (tile == GemmTile::T192) MLLM_WIDE_TYPES(6, 4, 2);
    }
  }
#undef MLLM_WIDE_TYPES
#undef MLLM_WIDE
  return hipErrorInvalidValue;
}

}  // namespace mllm
