// The MFMA GEMM kernel of every product whose K is a multiple of 64 (or whose k runs along the rows of both
// operands, the weight gradients): (32 WM) x (32 WN) x 64 tiles on four wavefronts.  Instantiated by operand
// layout in gemm_fwd.hip, gemm_dx.hip and gemm_dw.hip.
#pragma once
#include <utility>

#include "gemm_common.h"

namespace mllm {

namespace {

// ---------------------------------------------------------------------------------------------
// Four wavefronts (2 x 2) own WM x WN blocks of v_mfma_f32_16x16x32_bf16 each; with 8 x 8 blocks the 256
// accumulation registers of a lane are all accumulators, and a wavefront needs half an LDS fragment read per
// 32 K multiply-adds.
//
// What bounds it: at 256x256 tiles the power cap (the chip runs the loop at 1.6-1.9 GHz of 2.4) and what the
// memory pipeline holds up.  The 16x16x32 form reads and writes an accumulator half as often per multiply-add
// as 32x32x16: on normally distributed data a loop of nothing but MFMAs runs at 2020 TFLOP/s against
// 1770 (on zeros, where power does not count, both at 2410-2430).  Whole kernel against the 32x32x16 form with
// two staging sets that it replaced, one card, in turn: 32768 x 4096 x 28672, both operands k-contiguous,
// 1421 -> 1541 TFLOP/s; 32768 x 4096 x 14336 with W stored [K, N] 1394 -> 1447; 4096 x 28672 x 32768, both
// stored [K, .], 1431 -> 1477; without its global loads and LDS stores the loop reaches 1880-1920.  128x128
// tiles (two workgroups on a CU): 777 x 4096 x 14336 128 -> 100 us, 2999 x 3584 x 18944 464 -> 390 us.
//
// With one wavefront per SIMD nothing else hides a stall, so the k-loop is written slot by slot: every MFMA
// slot names the LDS read, LDS store and global load that issue in front of it and a scheduling barrier after
// every slot keeps that order.  The loop holds no vector ALU instruction.
// ---------------------------------------------------------------------------------------------
template <class F, int... Is>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  for_each_index(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// A k-tile of an operand to be loaded; the k-advance sits in the scalar offset.  The buffer's range check
// covers the sum of lane offset and scalar offset (measured, loads to registers and to LDS alike), so rows
// past the operand's end, the tail of a ragged K among them, arrive as zeros.
struct TileSource { __amdgpu_buffer_rsrc_t rsrc; uint32_t soff; };

// One operand's tile in LDS: EXT rows (or columns) of C by 64 along k, without padding; 16-byte chunk c
// of an LDS row sits at chunk position c ^ swz(row).
//   K_ROWS = false (operand stored [EXT, K]): LDS rows are rows of C, 64 k-values each.  A fragment is one
//     16-byte read a lane, 16 consecutive rows by 4 chunks.  A load instruction covers 8 rows, 1 KiB of
//     consecutive LDS in lane order (the lane asks for the chunk that the permutation keeps at its place), so
//     the tile can also go from memory straight to LDS.
//   K_ROWS = true (stored [K, EXT]): LDS rows are k, EXT values each, read transposed, 4 rows x 32 bytes per
//     16 lanes: the eight row segments of 32 lanes (rows k .. k+3 and k+8 .. k+11) land on eight different
//     32-byte slots of the 256 bytes that LDS serves at a time.  A lane's vectors are rows that differ only
//     in bits 2, 4 and 5, which the permutation does not see, so one offset register serves them all (the
//     row steps are scalar offsets and instruction offsets).
template <int EXT, bool K_ROWS, int WAVES = 4>
struct TileLoader16 {
  static constexpr int SIZE = EXT * BK;                    // elements
  static constexpr int PER_WAVE = SIZE / 512 / WAVES;      // instructions per wavefront and tile
  static constexpr int CPR = K_ROWS ? EXT / 8 : BK / 8;    // chunks per LDS row
  static_assert(PER_WAVE * 512 * WAVES == SIZE && (!K_ROWS || EXT == 128 || EXT == 256) && (WAVES == 4 || WAVES == 8), "whole instructions per wavefront");
  uint32_t off[K_ROWS ? 1 : PER_WAVE];   // byte offset of the lane's chunks in k-tile 0, OOB if never valid
  uint32_t lds_off;                      // the lane's element of vector 0 in the LDS tile
  uint32_t kstep, pitch;                 // bytes per k-tile; bytes per row of the operand

  static __device__ __forceinline__ int swz(int r) {
    if constexpr (K_ROWS) return ((r & 3) | ((r >> 1) & 4)) << 1;
    else return (r >> 1) & 7;
  }
  static constexpr int row_step(int i) {
    return EXT == 256 ? ((i & 1) << 2) | ((i >> 1) << (WAVES == 8 ? 5 : 4)) : i << (WAVES == 8 ? 5 : 4);
  }
  static __device__ __forceinline__ int wave_row(int wave) {
    return (EXT == 256 ? ((wave & 1) << 1) | (((wave >> 1) & 1) << 3) : (((wave >> 1) & 1) << 2) | ((wave & 1) << 3)) | ((wave >> 2) << 4);
  }
  // pair_half > 0 (operands stored [K, N] only): the tile's columns alternate, in runs of `run`, between
  // the left half of the matrix and the same columns of the right half (+ pair_half), so that each
  // wavefront's columns are matching gate and up columns.
  __device__ __forceinline__ void init(int64_t ld, int64_t fixed0, int64_t nfixed, int lane, int wave, int64_t pair_half = 0,
                                       int run = 1) {
    pitch = (uint32_t)(ld * 2);
    kstep = K_ROWS ? BK * pitch : BK * 2;
    if constexpr (K_ROWS) {
      const int r = (EXT == 256 ? lane >> 5 : lane >> 4) | wave_row(wave);
      const int cc = ((lane % CPR) ^ swz(r)) * 8;
      int64_t fx = fixed0 + cc;
      if (pair_half > 0) {
        const int blk = cc / run;
        fx = (blk & 1) * pair_half + (fixed0 >> 1) + run * (blk >> 1) + cc % run;
      }
      off[0] = fx < nfixed ? (uint32_t)(((int64_t)r * ld + fx) * 2) : OOB;
      lds_off = (uint32_t)(r * EXT + (lane % CPR) * 8);
    } else {
      lds_off = (uint32_t)(wave * PER_WAVE * 512 + lane * 8);
#pragma unroll
      for (int i = 0; i < PER_WAVE; i++) {
        const int r = (wave * PER_WAVE + i) * 8 + lane / 8, cc = ((lane % 8) ^ swz(r)) * 8;
        off[i] = fixed0 + r < nfixed ? (uint32_t)(((fixed0 + r) * ld + cc) * 2) : OOB;
      }
    }
  }
  // A load instruction's 64 vectors are 1 KiB of consecutive LDS in lane order, in either layout.
  template <int I>
  __device__ __forceinline__ void load_to_lds(const TileSource& s, bf16_t* lds, int wave) const {
    if constexpr (K_ROWS) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rsrc, (MLLM_LDS void*)(lds + (wave_row(wave) + row_step(I)) * EXT), 16, (int)off[0],
                                               (int)(s.soff + (uint32_t)row_step(I) * pitch), 0, 0);
    } else {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rsrc, (MLLM_LDS void*)(lds + (wave * PER_WAVE + I) * 512), 16, (int)off[I], (int)s.soff, 0, 0);
    }
  }
  template <int I>
  __device__ __forceinline__ u32x4 load(const TileSource& s) const {
    if constexpr (K_ROWS) return __builtin_amdgcn_raw_buffer_load_b128(s.rsrc, (int)off[0], (int)(s.soff + (uint32_t)row_step(I) * pitch), 0);
    else return __builtin_amdgcn_raw_buffer_load_b128(s.rsrc, (int)off[I], (int)s.soff, 0);
  }
  template <int I>
  __device__ __forceinline__ void store(bf16_t* lds, const u32x4& v) const {
    *reinterpret_cast<u32x4*>(lds + lds_off + (K_ROWS ? row_step(I) * EXT : I * 512)) = v;
  }
  // Fragment of the 16 rows (columns) from n0: lane l holds row l%16, k = 32 kk + 8 (l/16) .. +7.
  static __device__ __forceinline__ bf16x8 frag(const bf16_t* tile, int n0, int kk, int lane) {
    Frag8 f;
    const int g = lane >> 4, i16 = lane & 15;
    if constexpr (!K_ROWS) {
      const int r = n0 + i16;
      f.u = *reinterpret_cast<const uint4*>(tile + r * BK + 8 * ((4 * kk + g) ^ swz(i16)));
    } else {
      const int k = 32 * kk + 8 * g + (i16 >> 2), n = n0 + 4 * (i16 & 3);
      const bf16_t* q = tile + k * EXT + 8 * ((n >> 3) ^ swz(8 * g + (i16 >> 2))) + (n & 7);
      f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLLM_LDS s16x4*)q);
      f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLLM_LDS s16x4*)(q + 4 * EXT));
    }
    return f.v;
  }
};

// acc += a . b^T in place.  As a builtin the accumulator's input and output are two values that the
// register allocator has to bring together again; with all 256 accumulation registers taken by accumulators
// it has no room to do so and moves hundreds of registers around in every iteration.  Written as assembly
// the accumulator is one register quadruple from the first k-tile to the last.  The compiler does not know
// the statement for an MFMA: results may be read only behind mfma_results_ready().
__device__ __forceinline__ void mfma_in_place(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// More wait states than any MFMA in flight needs until its result may be read by another instruction.
__device__ __forceinline__ void mfma_results_ready() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// K must be a multiple of 64 unless k runs along the rows of both operands (the rows of the last k-tile that lie
// past K are then past the operands' ends).
// pid of nblk workgroups of the product, each of them with part `split` of the K loop; As0 .. Bs1: the two LDS stages of
// both operands (distinct variables of the kernel, so that the compiler can tell their accesses apart).
template <int WM, int WN, bool A_T, bool B_T, bool OUT_F32, int EPI>
__device__ __forceinline__ void gemm_dma_tile(GemmParams p, int pid, int nblk, int split, bf16_t* As0, bf16_t* As1, bf16_t* Bs0, bf16_t* Bs1) {
  static_assert(EPI == EPI_PLAIN || (!OUT_F32 && !A_T && B_T == (EPI != EPI_SWIGLU_BWD)), "fused epilogues: bf16, forward layout (gradient: W stored [N, K])");
  constexpr int BM = 32 * WM, BN = 32 * WN;
  constexpr int NU = WM + WN;         // fragments per k-step
  constexpr int NS = WM * WN;         // MFMA slots per k-step
  using TA = TileLoader16<BM, A_T>;
  using TB = TileLoader16<BN, B_T>;
  static_assert(TA::PER_WAVE == WM && TB::PER_WAVE == WN, "loads per wavefront and k-tile");
  // Slots: the fragments of a k-step are read every RS slots of the step before; the barrier of a k-tile
  // stands in front of slot BAR of its first k-step, when the last of the tile's fragments is on its way
  // to the registers.
  constexpr bool DIRECT = !A_T && !B_T && NS >= 48;
  constexpr int RS = DIRECT ? (NS >= 2 * NU + 8 ? 2 : 1) : (NS >= NU + 8 ? (NS - 8) / NU : 1);
  constexpr int BAR = RS * (NU - 1) + (NS < 48 ? 4 : DIRECT ? 8 : 10);
  constexpr int BAR2 = DIRECT ? NS - 1 : -1;   // second barrier of a k-tile, direct loads only
  static_assert(BAR < NS, "the first k-step's reads are issued before the barrier");

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int tm, tn;
  tile_of_block(pid, nblk, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  TA la;
  TB lb;
  la.init(p.lda, m0, p.M, lane, wave);
  lb.init(p.ldb, n0, p.N, lane, wave, EPI == EPI_SWIGLU ? p.N >> 1 : 0, 8 * WN);

  // Split-K: part `split` owns k-tiles [kt0, kt0 + nk) and writes its own partial C.
  const int kt0 = split * p.kt_per_split;
  const int last_tile = (int)((p.K + BK - 1) / BK) - 1;
  const int nk = min(p.kt_per_split, last_tile + 1 - kt0);   // at least one: the host leaves no split empty

  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  // k-tile kt0 + kt of an operand (a tile that this workgroup does not have: an empty buffer, no traffic)
  auto source = [&](uint32_t kstep, const bf16_t* base, uint32_t bytes, int kt) __attribute__((always_inline)) {
    const bool have = kt < nk;
    const uint32_t k = (uint32_t)(have ? kt0 + kt : 0);
    return TileSource{make_rsrc(base, have ? bytes : 0u), k * kstep};
  };
  auto source_a = [&](int kt) __attribute__((always_inline)) { return source(la.kstep, p.a, p.a_bytes, kt); };
  auto source_b = [&](int kt) __attribute__((always_inline)) { return source(lb.kstep, p.b, p.b_bytes, kt); };
  auto a_stage = [&](auto i_c) __attribute__((always_inline)) -> bf16_t* { return decltype(i_c)::value ? As1 : As0; };
  auto b_stage = [&](auto i_c) __attribute__((always_inline)) -> bf16_t* { return decltype(i_c)::value ? Bs1 : Bs0; };
  // The tile traffic of one k-tile's time, from the barrier of tile kt to that of tile kt + 1 ("window kt", NW
  // slots), into the LDS stage that tile kt has left.
  //   DIRECT (both operands k-contiguous, large tiles): tile kt + 2 is requested from memory straight into LDS,
  //   LOAD_STEP slots from load to load: closer together the wavefront stands still while the memory pipeline
  //   takes them, further apart the last ones have too little time to land (32768 x 4096 x 28672: 4 slots 1481, 5
  //   1532, 6 1544 TFLOP/s).
  //   Otherwise tile kt + 2 goes from the staging registers to LDS, one vector at a time over the whole
  //   window, and each register is refilled with tile kt + 3 at once, so that every load has a whole
  //   k-tile's time to land.  Direct loads of operands stored [K, .] are late whatever their spacing (32768 x 4096 x
  //   14336: 1044-1067 TFLOP/s direct, 1404 through registers), and 128x128 tiles need their loads too close
  //   together (777 x 4096 x 28672: 525 and 763).
  constexpr int NW = 2 * NS, HEAD = NS + NS - BAR;   // slots [0, HEAD) belong to iteration kt, the rest to kt + 1
  constexpr int LOAD_STEP = NS >= 64 ? 6 : 5;   // 192x256 tiles: 5 slots 1196, 6 1137 TFLOP/s (5125 x 3200 x 12800)
  u32x4 stage[DIRECT ? 1 : NU];
  auto load_vec = [&](auto q_c, const TileSource& sa, const TileSource& sb) __attribute__((always_inline)) {
    constexpr int q = decltype(q_c)::value;
    if constexpr (q < WM) stage[q] = la.template load<q>(sa);
    else stage[q] = lb.template load<q - WM>(sb);
  };
  auto store_vec = [&](auto q_c, bf16_t* as, bf16_t* bs) __attribute__((always_inline)) {
    constexpr int q = decltype(q_c)::value;
    if constexpr (q < WM) la.template store<q>(as, stage[q]);
    else lb.template store<q - WM>(bs, stage[q]);
  };
  auto load_direct = [&](auto q_c, const TileSource& sa, const TileSource& sb, bf16_t* as, bf16_t* bs) __attribute__((always_inline)) {
    constexpr int q = decltype(q_c)::value;
    if constexpr (q < WM) la.template load_to_lds<q>(sa, as, wave);
    else lb.template load_to_lds<q - WM>(sb, bs, wave);
  };
  // sa, sb: the tile to be requested, kt + 2 (DIRECT) or kt + 3
  auto window = [&](auto w_c, auto st_c, const TileSource& sa, const TileSource& sb) __attribute__((always_inline)) {
    constexpr int w = decltype(w_c)::value;
    static_for<NU>([&](auto q_c) __attribute__((always_inline)) {
      constexpr int q = decltype(q_c)::value;
      if constexpr (DIRECT) {
        if constexpr (w == 1 + q * LOAD_STEP) load_direct(q_c, sa, sb, a_stage(st_c), b_stage(st_c));
      } else {
        constexpr int at = 1 + q * (NW - 6) / NU;
        if constexpr (w == at) store_vec(q_c, a_stage(st_c), b_stage(st_c));
        if constexpr (w == at + 1) load_vec(q_c, sa, sb);
      }
    });
  };

  // Fragments, double-buffered by k-step, in the order of first use: A0, B0.., A1..
  bf16x8 af[2][WM], bfr[2][WN];
  auto fetch_unit = [&](auto u_c, auto kk_c, const bf16_t* at, const bf16_t* bt) __attribute__((always_inline)) {
    constexpr int u = decltype(u_c)::value, kk = decltype(kk_c)::value;
    if constexpr (u == 0) af[kk][0] = TA::frag(at, wm * 16 * WM, kk, lane);
    else if constexpr (u <= WN) bfr[kk][u - 1] = TB::frag(bt, wn * 16 * WN + 16 * (u - 1), kk, lane);
    else af[kk][u - WN] = TA::frag(at, wm * 16 * WM + 16 * (u - WN), kk, lane);
  };

  // Prologue: tiles 0 and 1 are requested together (one exposed latency for both); tile 0 and the part of
  // window -1 (tile 1) that precedes iteration 0 go to LDS.
  constexpr int AHEAD = DIRECT ? 2 : 3;   // window kt requests tile kt + AHEAD
  f32x4 acc[WM][WN];
  auto clear = [&]() __attribute__((always_inline)) {   // while the first tiles are on their way
#pragma unroll
    for (int i = 0; i < WM; i++)
#pragma unroll
      for (int j = 0; j < WN; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    __builtin_amdgcn_sched_barrier(0);
  };
  {
    const TileSource a0 = source_a(0), b0 = source_b(0), a1 = source_a(1), b1 = source_b(1);
    if constexpr (DIRECT) {
      static_for<NU>([&](auto q) { load_direct(q, a0, b0, As0, Bs0); });
      static_for<HEAD>([&](auto w) { window(w, C1{}, a1, b1); });
      clear();
      constexpr int FIRST1 = (HEAD - 2) / LOAD_STEP + 1;   // loads of tile 1 issued here: slots 1 + q * LOAD_STEP < HEAD
      constexpr int VM = FIRST1 < NU ? FIRST1 : NU;
      __builtin_amdgcn_s_waitcnt(0x0F70 | (VM & 15) | ((VM >> 4) << 14));   // tile 0 has landed
    } else {
      const TileSource a2 = source_a(2), b2 = source_b(2);
      u32x4 first[NU];
      static_for<NU>([&](auto q) { load_vec(q, a0, b0); });
#pragma unroll
      for (int q = 0; q < NU; q++) first[q] = stage[q];
      static_for<NU>([&](auto q) { load_vec(q, a1, b1); });
      clear();
      static_for<NU>([&](auto q_c) {
        constexpr int q = decltype(q_c)::value;
        if constexpr (q < WM) la.template store<q>(As0, first[q]);
        else lb.template store<q - WM>(Bs0, first[q]);
      });
      static_for<HEAD>([&](auto w) { window(w, C1{}, a2, b2); });
      __builtin_amdgcn_s_waitcnt(0xC07F);   // stored
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
  static_for<NU>([&](auto u) { fetch_unit(u, C0{}, As0, Bs0); });

  // One k-tile; its LDS stage is kt % 2.
  auto iteration = [&](auto p_c, int kt) __attribute__((always_inline)) {
    using CUR = decltype(p_c);
    using OTHER = std::integral_constant<int, 1 - CUR::value>;
    // this tile's first slots finish the window of the tile before
    const TileSource a_prev = source_a(kt - 1 + AHEAD), b_prev = source_b(kt - 1 + AHEAD);
    const TileSource a_next = source_a(kt + AHEAD), b_next = source_b(kt + AHEAD);
    auto slot = [&](auto kk_c, auto m_c) __attribute__((always_inline)) {
      constexpr int kk = decltype(kk_c)::value, m = decltype(m_c)::value;
      if constexpr (kk == 0 && m == BAR) {
        // Every wavefront has read tile kt, so its stage may take tile kt + 2; global loads stay in flight.
        // Staged: this wavefront's share of tile kt + 1 has been stored, too.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (kk == 0 && m == BAR2) {
        // Direct: this wavefront's share of tile kt + 1 has landed (of tile kt + 2's loads, those issued since the
        // first barrier may be on their way).  A barrier of its own, as late as the tile's first reader allows, gives
        // the loads 27 slots more than one barrier for both would.
        constexpr int ISSUED = DIRECT ? (BAR2 - BAR - 2) / LOAD_STEP + 1 : 0, VM = ISSUED < NU ? ISSUED : NU;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70 | (VM & 15) | ((VM >> 4) << 14));   // vmcnt(VM)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (m % RS == 0 && m / RS < NU) {
        using U = std::integral_constant<int, m / RS>;
        if constexpr (kk == 0) fetch_unit(U{}, C1{}, a_stage(CUR{}), b_stage(CUR{}));
        else fetch_unit(U{}, C0{}, a_stage(OTHER{}), b_stage(OTHER{}));
      }
      if constexpr (kk == 0 && m < BAR) window(std::integral_constant<int, HEAD + m>{}, OTHER{}, a_prev, b_prev);
      else window(std::integral_constant<int, kk * NS + m - BAR>{}, CUR{}, a_next, b_next);
      constexpr int i = m / WN, j = (i & 1) ? WN - 1 - m % WN : m % WN;
      mfma_in_place(acc[i][j], bfr[kk][j], af[kk][i]);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<NS>([&](auto m) __attribute__((always_inline)) { slot(C0{}, m); });
    static_for<NS>([&](auto m) __attribute__((always_inline)) { slot(C1{}, m); });
  };
  for (int kt = 0; kt + 1 < nk; kt += 2) {
    iteration(C0{}, kt);
    iteration(C1{}, kt + 1);
  }
  if (nk & 1) iteration(C0{}, nk - 1);
  // The epilogue stages its rows where the tiles were: whatever is still on its way there (tiles past the end,
  // zeros) has to land first, of every wavefront.
  if constexpr (DIRECT) __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
  else __builtin_amdgcn_s_waitcnt(0xC07F);                    // lgkmcnt(0)
  mfma_results_ready();
  // the epilogue's addresses depend on the lane alone; hidden from the loop, they take none of its registers
  int lane_out = lane;
  asm volatile("" : "+v"(lane_out));
#pragma unroll
  for (int i = 0; i < WM; i++)
#pragma unroll
    for (int j = 0; j < WN; j++) asm volatile("" : "+a"(acc[i][j]));   // no read above the wait
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  uint32_t* const out_stage = reinterpret_cast<uint32_t*>(wave == 0 ? As0 : wave == 1 ? As1 : wave == 2 ? Bs0 : Bs1);
  static_assert(2 * 16 * (16 * WN + 4) * 4 <= 2 * (TA::SIZE < TB::SIZE ? TA::SIZE : TB::SIZE), "two staged rows of blocks in a tile's LDS");

  const int64_t row0 = m0 + wm * 16 * WM, col0 = n0 + wn * 16 * WN;
  if constexpr (OUT_F32) p.c = reinterpret_cast<float*>(p.c) + split * p.c_split_stride;
  if constexpr (EPI == EPI_SWIGLU) {
    store_blocks_swiglu<WM, WN>(p, acc, row0, (n0 >> 1) + 8 * WN * wn, lane_out, out_stage);
  } else if constexpr (EPI == EPI_SWIGLU_BWD) {
    store_blocks_swiglu_bwd<WM, WN>(p, acc, row0, col0, lane_out, out_stage);
  } else {
    store_blocks<WM, WN, OUT_F32, EPI == EPI_ROPE128 ? 128 : EPI == EPI_ROPE64 ? 64 : 0>(p, acc, row0, col0, lane_out, out_stage);
  }
}

template <int WM, int WN, bool A_T, bool B_T, bool OUT_F32, int EPI>
__global__ __launch_bounds__(256, WM * WN <= 16 ? 2 : 1) void gemm4_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) bf16_t As0[32 * WM * BK], As1[32 * WM * BK], Bs0[32 * WN * BK], Bs1[32 * WN * BK];
  gemm_dma_tile<WM, WN, A_T, B_T, OUT_F32, EPI>(p, blockIdx.x, gridDim.x, blockIdx.y, As0, As1, Bs0, Bs1);
}

}  // namespace

template <bool A_T, bool B_T>
hipError_t launch_gemm_tile(const GemmParams& p, GemmTile tile, bool out_f32, int epi, dim3 grid, hipStream_t s) {
  const dim3 block(256);
  if (p.K <= 0 || (p.K % BK != 0 && !(A_T && B_T))) return hipErrorInvalidValue;
#define MLLM_TILE(WM, WN, F32, EPI)                                                                      \
  do {                                                                                                   \
    hipLaunchKernelGGL((gemm4_kernel<WM, WN, A_T, B_T, F32, EPI>), grid, block, 0, s, p);                \
    return hipGetLastError();                                                                            \
  } while (0)
#define MLLM_TILE_TYPES(WM, WN)                \
  do {                                         \
    if (out_f32) MLLM_TILE(WM, WN, true, EPI_PLAIN);  \
    else MLLM_TILE(WM, WN, false, EPI_PLAIN);  \
  } while (0)
  if constexpr (!A_T && B_T) {
#define MLLM_TILE_FUSED(E)                                                 \
    if (epi == E) {                                                        \
      if (tile == GemmTile::T256) MLLM_TILE(8, 8, false, E);               \
      if (tile == GemmTile::T224) MLLM_TILE(7, 8, false, E);               \
      return hipErrorInvalidValue;                                         \
    }
    MLLM_TILE_FUSED(EPI_SWIGLU)
    MLLM_TILE_FUSED(EPI_ROPE128)
    MLLM_TILE_FUSED(EPI_ROPE64)
#undef MLLM_TILE_FUSED
  }
  if constexpr (!A_T && !B_T) {
    if (epi == EPI_SWIGLU_BWD) {
      if (tile == GemmTile::T256) MLLM_TILE(8, 8, false, EPI_SWIGLU_BWD);
      if (tile == GemmTile::T224) MLLM_TILE(7, 8, false, EPI_SWIGLU_BWD);
      if (tile == GemmTile::T128) MLLM_TILE(4, 4, false, EPI_SWIGLU_BWD);   // operands off 16-byte alignment
      return hipErrorInvalidValue;
    }
  }
  if (epi != EPI_PLAIN) return hipErrorInvalidValue;
  if constexpr (!A_T) {
    if (tile == GemmTile::T192) MLLM_TILE_TYPES(6, 8);
    if (tile == GemmTile::T224) MLLM_TILE_TYPES(7, 8);
  }
  if (tile == GemmTile::T256) MLLM_TILE_TYPES(8, 8);
  if (tile == GemmTile::T128) MLLM_TILE_TYPES(4, 4);
#undef MLLM_TILE_TYPES
#undef MLLM_TILE
  return hipErrorInvalidValue;
}

}  // namespace mllm
