// Varlen block-diagonal flash attention for gfx950, forward and backward.
//
// Attention depends on the length of every single sample and has to treat each packed sample
// on its own so that no sample sees another (Model Profiler, "Throughput Profiling"): a packed
// [T, heads, hd] sequence is cut into segments by cu_seqlens; each segment
// attends only to itself, bidirectionally (an image inside the ViT) or causally (a sample inside
// the LLM).  The host turns the segments into lists of (segment, tile, head) work items, one list
// per XCD, in which workgroups that share rows sit together (attn_items.h).
//
// All kernels compute score blocks TRANSPOSED so that a lane owns one column of a 16x16 MFMA result, a query (a key in the
// dK/dV pass) of its wavefront: row statistics are then per-lane scalars, summed over the four lanes of a column at the end,
// and the probability block can be fed straight back as the B operand of the next MFMA without leaving registers (the
// contraction-slot order of that operand is a fixed permutation of the key/query rows, applied identically to the A
// operand, which is fetched from LDS with the transposing read).
//
//   forward:  S^T = K.Q^T, online softmax, O^T += V^T.P^T
//   dQ pass:  delta = rowsum(dO*O); S^T, dP^T = V.dO^T, dS^T = P^T*(dP^T - delta), dQ^T += K^T.dS^T
//   dK/dV:    S = Q.K^T, dP = dO.V^T, dV^T += dO^T.P, dK^T += Q^T.dS, looping the query tiles
//             and the query heads of the GQA group, so dK/dV need no atomics.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace mllm {

namespace {

constexpr int BKV = 64;   // key rows staged per step (forward, dQ)
constexpr int BQ = 64;    // query rows staged per step (dK/dV, heads of 64)

// LDS tiles are [rows][HD] bf16 without padding; 16-byte chunk c of row r lives at chunk position c ^ swz<HD, BLOCK>(r), BLOCK the
// rows of an MFMA operand.  LDS serves 256 B per clock.  A transposing 8-byte read is processed 32 lanes at a time (8 consecutive
// rows x 32 B with operands of 16 rows, 4 x 64 B with 32), a 16-byte read 16 lanes at a time, lanes 0-3, 12-15, 20-23 and 24-27 of
// each 32, then the other 16 (operands of 16 rows: rows 0-3 and 12-15 at an even chunk and rows 4-11 at the next one, or the other
// way round; of 32: 16 rows at one chunk).  The permutations make both patterns conflict-free on the same tile: HD = 128 (256-byte
// rows), operands of 16 rows: rows 0-7 take the 8 pairs of chunks and rows 8-15 the other halves of the pairs, those of 12-15
// beside 0-3; of 32: 16 rows take 16 chunks, the 4 rows of a transposing read the 4 quarters of the row.  HD = 64 (128-byte rows,
// two rows per 256-byte window) does the same over row pairs.
template <int HD, int BLOCK = 16>
__device__ __forceinline__ int swz(int r) {
  const int t = (r >> 1) & 7;
  if constexpr (BLOCK == 32) return HD == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : ((t & 1) << 2) | (t >> 1);
  else return HD == 128 ? (((r & 7) ^ ((r >> 1) & 4)) << 1) | ((r >> 3) & 1) : (((t & 3) ^ ((t >> 1) & 2)) << 1) | (t >> 2);
}
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// v_exp_f32: flushes tiny results to zero, which is what a masked or negligible probability wants.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

struct AttnParams {
  const bf16_t* q; const bf16_t* k; const bf16_t* v; bf16_t* o; float* lse;
  const bf16_t* d_o; bf16_t* dq; bf16_t* dk; bf16_t* dv; float* delta;
  int64_t q_stride, kv_stride, o_stride;
  int32_t T, Hq, Hkv;
  const AttnItem* list;      // work list, one entry per workgroup
  float scale_log2e, scale;
  const float* rope_table;   // backward: dq, dk are rotated back by the rotary angle of their row (null: not)
  float* dkv_partial;        // dK/dV pass in gridDim.y > 1 parts: fp32 sums [part][dK, dV][T][Hkv * HD]
};

// The dK/dV pass of a key tile walks (query head of the group, query tile) pairs; with gridDim.y parts a
// workgroup walks its share of them.
struct KvRange { int n_it, head, q0; };   // iterations, and where they start: head of the group, first query row
__device__ __forceinline__ KvRange kv_range(int grp, int q_begin, int seg_len, int tile_rows, int part, int parts) {
  const int per_head = (seg_len - q_begin + tile_rows - 1) / tile_rows, total = grp * per_head;
  const int first = total * part / parts, last = total * (part + 1) / parts;
  return {last - first, first / per_head, q_begin + first % per_head * tile_rows};
}

// The work item of this workgroup (an entry of the list, by default blockIdx.x; the host has arranged the entries so
// that workgroups sharing rows run on one XCD).  Returns false, for the whole workgroup, on the empty
// items that pad the shorter XCD lists.
__device__ __forceinline__ bool work_item(const AttnItem* list, AttnItem& t, int entry) {
  const AttnItem x = list[entry];
  // the same for every lane: keep the fields in scalar registers
  t.seg_start = __builtin_amdgcn_readfirstlane(x.seg_start);
  t.seg_len = __builtin_amdgcn_readfirstlane(x.seg_len);
  t.tile0 = __builtin_amdgcn_readfirstlane(x.tile0);
  t.causal = __builtin_amdgcn_readfirstlane(x.causal);
  t.head = __builtin_amdgcn_readfirstlane(x.head);
  return t.seg_len > 0;
}

// ---- operands -----------------------------------------------------------------------------------
// All products but those of the forward pass at head_dim 64 are v_mfma_f32_16x16x32_bf16.  A wavefront owns 32 rows (queries, or
// keys in the dK/dV pass) as the columns of the results, in two groups j of 16: lane l holds column l%16 of group j, and with g = l/16 the rows 4g .. 4g+3 of each
// 16-row group i of the other side's block of 32.  The 32x32x16 form does the same work in half the MFMAs and reads and
// writes its accumulator twice as often per multiply-add, and that is power, which bounds these kernels at head_dim 128: 13255
// causal tokens, 32/8 heads of 128, MFMA busy 61 % of the cycles in the forward pass and 72 % in dQ at 1.76 and 1.66 GHz with
// it, 62 % and 69 % at 1.88 and 1.87 GHz with this form (of 2.4): 1245 -> 1121 and 1672 -> 1544 us on one card.  The order in
// which a wavefront issues its reads and vector work no longer shows there (reads one to four fragments ahead, vector work
// between the MFMAs or behind them: within 1 %, behind them where not).  At head_dim 64 the vector ALU and latency bound them, at 2.2 GHz
// (46 x 576 tokens, 16 heads: dK/dV 211 -> 187).
struct Lane {
  int lane, g, c16;
  __device__ __forceinline__ explicit Lane(int tid) : lane(tid & 63), g((tid & 63) >> 4), c16(tid & 15) {}
};
typedef MLLM_LDS const char* lds_cptr;
typedef MLLM_LDS char* lds_ptr;
__device__ __forceinline__ bf16x8 lds_b128(lds_cptr base, uint32_t off) {
  return __builtin_bit_cast(bf16x8, *(MLLM_LDS const u32x4_t*)(base + off));
}
__device__ __forceinline__ s16x4 lds_tr(lds_cptr base, uint32_t off) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLLM_LDS s16x4*)(base + off));
}
__device__ __forceinline__ f32x4 lds_f4(lds_cptr base, uint32_t off) { return *(MLLM_LDS const f32x4*)(base + off); }
// Natural-layout operand of the score-like products: row l%16 of a 16-row group, columns 32c + 8g .. +7.  Byte offset in the
// tile; 16 rows further on are 16 * HD * 2 bytes.
template <int HD>
__device__ __forceinline__ uint32_t row_offset(const Lane& L, int c) { return (uint32_t)(L.c16 * HD + 8 * ((4 * c + L.g) ^ swz<HD>(L.c16))) * 2u; }
// Transposed operand for the register-resident operand made of two 16-row groups of a result: column 16n + l%16 of the tile,
// contraction slots e = 0..7 standing for tile rows 4g + e%4 (+16 for e >= 4).  Each transposing read returns tile[k0 + e][n0 + i]
// for e = 0..3 when lane i of a 16-lane group addresses tile[k0 + i/4][n0 + 4*(i%4)].
template <int HD>
__device__ __forceinline__ uint32_t col_offset(const Lane& L, int n) {
  const int k = 4 * L.g + (L.c16 >> 2), chunk = 2 * n + ((L.c16 & 3) >> 1);
  return (uint32_t)(k * HD + 8 * (chunk ^ swz<HD>(k)) + 4 * (L.c16 & 1)) * 2u;
}
template <int HD>
__device__ __forceinline__ bf16x8 read_col(lds_cptr base, uint32_t off) {
  Frag8 f;
  f.h[0] = lds_tr(base, off);
  f.h[1] = lds_tr(base, off + 16 * HD * 2);
  return f.v;
}
__device__ __forceinline__ bf16x8 global_frag(const bf16_t* p, bool ok) {
  Frag8 f;
  f.u = ok ? *reinterpret_cast<const uint4*>(p) : make_uint4(0, 0, 0, 0);
  return f.v;
}
__device__ __forceinline__ bf16x8 negated(bf16x8 x) {
  Frag8 f;
  f.v = x;
#pragma unroll
  for (int w = 0; w < 4; w++) f.w[w] ^= 0x80008000u;
  return f.v;
}
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
// Keeps what a slot (a few MFMAs and what is to be issued beside them) holds apart from the next one's.
#define MLLM_SLOT_END __builtin_amdgcn_sched_barrier(0)

// ---- loads from memory straight into LDS (common.h) --------------------------------------------------
// Descriptor over rows [0, rows) of a row-major bf16 matrix slice of `width` columns.
__device__ __forceinline__ i32x4_t rows_rsrc(const bf16_t* base, int64_t stride, int rows, int width) {
  return raw_rsrc(base, rows > 0 ? (uint32_t)(((int64_t)(rows - 1) * stride + width) * 2) : 0u);
}
// The workgroup's barrier, in its place; LDS writes issued before it are visible behind it.
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
template <int V> using Int = std::integral_constant<int, V>;
// One such instruction moves 64 lanes x 16 bytes = RPI rows of a tile; lane l's chunk lands at position l of that 1 KiB, so the
// lane fetches the global chunk that the permutation puts there.  Byte offset of the lane's chunk, instruction `ins` of the tile.
template <int HD, int BLOCK = 16>
__device__ __forceinline__ uint32_t load_offset(const Lane& L, int ins, int64_t stride) {
  constexpr int CPR = HD / 8, RPI = 64 / CPR;
  const int r = ins * RPI + L.lane / CPR, c = (L.lane % CPR) ^ swz<HD, BLOCK>(r);
  return (uint32_t)((r * stride + 8 * c) * 2);
}

// ---- results -----------------------------------------------------------------------------------------
// acc[n][j]: columns 16n + 4g .. +3 of the head, own row 16j + l%16.
// Gradient of the rotary positions on row group j, whose lanes own row `pos` of their segment: the pair (c, c + HD/2) sits in
// groups (n, n + HD/32) of the same lane.  Forward was y1 = x1 cos - x2 sin, y2 = x2 cos + x1 sin, so
// dx1 = dy1 cos + dy2 sin, dx2 = dy2 cos - dy1 sin.  `scale` multiplies the result.
template <int HD>
__device__ __forceinline__ void rope_unrotate(f32x4 (&acc)[HD / 16][2], int j, const float* table, int pos, int g, float scale) {
  constexpr int HALF = HD / 2;
  const float* trow = table + (int64_t)pos * HD;
#pragma unroll
  for (int n = 0; n < HD / 32; n++) {
    const int f0 = 16 * n + 4 * g;
    const float4 c = *reinterpret_cast<const float4*>(trow + f0);
    const float4 sn = *reinterpret_cast<const float4*>(trow + HALF + f0);
    const float cs[4] = {c.x * scale, c.y * scale, c.z * scale, c.w * scale};
    const float ss[4] = {sn.x * scale, sn.y * scale, sn.z * scale, sn.w * scale};
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float y1 = acc[n][j][e], y2 = acc[n + HD / 32][j][e];
      acc[n][j][e] = y1 * cs[e] + y2 * ss[e];
      acc[n + HD / 32][j][e] = y2 * cs[e] - y1 * ss[e];
    }
  }
}
// Row group j in bf16, times `scale`; dst: the row's first column of the head, plus 4g.
template <int HD>
__device__ __forceinline__ void store_row(bf16_t* dst, const f32x4 (&acc)[HD / 16][2], int j, float scale) {
#pragma unroll
  for (int n = 0; n < HD / 16; n++) {
    uint2 w;
    w.x = pack_bf16x2(acc[n][j][0] * scale, acc[n][j][1] * scale);
    w.y = pack_bf16x2(acc[n][j][2] * scale, acc[n][j][3] * scale);
    *reinterpret_cast<uint2*>(dst + 16 * n) = w;
  }
}
// A part's sums of row group j, fp32 and without the softmax scale; which: 0 dK, 1 dV.
template <int HD>
__device__ __forceinline__ void store_kv_partial(const AttnParams& p, const f32x4 (&acc)[HD / 16][2], int j, int which, float sign, int64_t row, int kvh, int g,
                                                 unsigned part) {
  float* dst = p.dkv_partial + ((int64_t)(2 * part + which) * p.T + row) * ((int64_t)p.Hkv * HD) + kvh * HD + 4 * g;
#pragma unroll
  for (int n = 0; n < HD / 16; n++)
    *reinterpret_cast<float4*>(dst + 16 * n) = make_float4(sign * acc[n][j][0], sign * acc[n][j][1], sign * acc[n][j][2], sign * acc[n][j][3]);
}
// dK (negated in acc) or dV of the lane's two rows: partial sums, or bf16 with scale and rotation.
template <int HD>
__device__ __forceinline__ void store_dk(const AttnParams& p, f32x4 (&acc)[HD / 16][2], int j, int krow, int64_t gkrow, int kvh, int g, bool split, unsigned part) {
  if (split) return store_kv_partial<HD>(p, acc, j, 0, -1.f, gkrow, kvh, g, part);
  bf16_t* dst = p.dk + gkrow * p.kv_stride + kvh * HD + 4 * g;
  if (p.rope_table) rope_unrotate<HD>(acc, j, p.rope_table, krow, g, -p.scale);
  store_row<HD>(dst, acc, j, p.rope_table ? 1.f : -p.scale);
}
template <int HD>
__device__ __forceinline__ void store_dv(const AttnParams& p, const f32x4 (&acc)[HD / 16][2], int j, int64_t gkrow, int kvh, int g, bool split, unsigned part) {
  if (split) return store_kv_partial<HD>(p, acc, j, 1, 1.f, gkrow, kvh, g, part);
  store_row<HD>(p.dv + gkrow * p.kv_stride + kvh * HD + 4 * g, acc, j, 1.f);
}
// Sum and maximum over the four lanes that hold parts of one own row.
__device__ __forceinline__ float own_row_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float own_row_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}

// ---------------------------------------------------------------------------------------------
// forward, head_dim 128: one workgroup per (query tile of 128, head), looping over key tiles of 64: two blocks b of 32 keys.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void attn_fwd_kernel(AttnParams p) {
  constexpr int HD = 128, NC = HD / 32, NN = HD / 16, NS = 2 * NC, TILE_B = BKV * HD * 2, BLOCK_B = 32 * HD * 2, GROUP_B = 16 * HD * 2;
  // two stages of a K tile and a V tile
  __shared__ __attribute__((aligned(1024))) char lds[4 * TILE_B];
  AttnItem t;
  if (!work_item(p.list, t, blockIdx.x)) return;
  const int head = t.head, kvh = head / (p.Hq / p.Hkv);
  const Lane L(threadIdx.x);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_first_q = t.tile0 + 32 * wave, wave_last_q = wave_first_q + 31;
  int qrow[2];
  bf16x8 qf[2][NC];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    qrow[j] = wave_first_q + 16 * j + L.c16;
    const bf16_t* qp = p.q + (int64_t)(t.seg_start + qrow[j]) * p.q_stride + head * HD + 8 * L.g;
#pragma unroll
    for (int c = 0; c < NC; c++) qf[j][c] = global_frag(qp + 32 * c, qrow[j] < t.seg_len);
  }
  const int kv_end = t.causal ? min(t.seg_len, t.tile0 + ATTN_FWD_Q_TILE) : t.seg_len;

  f32x4 acc[NN][2];
#pragma unroll
  for (int n = 0; n < NN; n++) acc[n][0] = acc[n][1] = f32x4{0, 0, 0, 0};
  const float c2 = p.scale_log2e;
  // Reference maximum m (in units of log2: score * scale * log2(e)) and sum l = sum of exp2(... - m).  The reference is the
  // row's maximum over the first tile and stays: probabilities above 1 carry the same relative precision in fp32 sums and
  // in the bf16 operand.  Only a tile where a lane's 16 probabilities sum to more than `limit`, so that one of them is above 2^8 (or past the
  // range of fp32), has its scores formed again and moves the reference (`again`); so neither the maximum of a tile's scores, nor its
  // exchange between lanes, nor the rescaling of the accumulator is on the path.
  constexpr float LIMIT = 4096.f;
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f}, limit[2] = {-1.f, -1.f};   // -1: no reference yet

  // Rows past kv_end are outside the descriptors: zeros, no traffic.
  const i32x4_t rk = rows_rsrc(p.k + (int64_t)t.seg_start * p.kv_stride + kvh * HD, p.kv_stride, kv_end, HD);
  const i32x4_t rv = rows_rsrc(p.v + (int64_t)t.seg_start * p.kv_stride + kvh * HD, p.kv_stride, kv_end, HD);
  constexpr int PER_WAVE = BKV * HD / 8 / 64 / 4;
  uint32_t kv_off[PER_WAVE];
#pragma unroll
  for (int i = 0; i < PER_WAVE; i++) kv_off[i] = load_offset<HD>(L, wave * PER_WAVE + i, p.kv_stride);
  const uint32_t row_bytes = (uint32_t)(p.kv_stride * 2);
  const uint32_t lds_b = __builtin_amdgcn_readfirstlane(lds_address((MLLM_LDS const void*)lds) + wave * PER_WAVE * 1024);
  auto issue_part = [&](int st, int kv0, int j) {   // j even: K, odd: V
    load_to_lds_b128(j % 2 ? rv : rk, lds_b + (uint32_t)(st * 2 * TILE_B + j % 2 * TILE_B + j / 2 * 1024), kv_off[j / 2], (uint32_t)kv0 * row_bytes);
  };
  const lds_cptr M = (lds_cptr)lds;
  uint32_t rows[NC], cols[NN];
#pragma unroll
  for (int c = 0; c < NC; c++) rows[c] = row_offset<HD>(L, c);
#pragma unroll
  for (int n = 0; n < NN; n++) cols[n] = col_offset<HD>(L, n) + TILE_B;

  f32x4 s[2][2][2];      // scores, then probabilities: [block][row group][own group]
  Frag8 pb[2][2];        // probabilities as MFMA operand: [block][own group]
  auto mask = [&](int kv0) {
    if ((kv0 + BKV > t.seg_len) || (t.causal && kv0 + BKV - 1 > wave_first_q)) {   // the tile crosses the segment end or the diagonal
#pragma unroll
      for (int b = 0; b < 2; b++)
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
              const int kv = kv0 + 32 * b + 16 * i + 4 * L.g + e;
              s[b][i][j][e] = (kv < t.seg_len && (!t.causal || kv <= qrow[j])) ? s[b][i][j][e] : -INFINITY;
            }
    }
  };
  auto tile_max = [&](int j) {
    float mx = s[0][0][j][0];
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int e = 0; e < 4; e++) mx = fmaxf(mx, s[b][i][j][e]);
    return own_row_max(mx) * c2;
  };
  float mu[2] = {0.f, 0.f};   // m, or 0 where there is none yet
  auto set_reference = [&](int j, float to) {
    m[j] = to;
    mu[j] = to == -INFINITY ? 0.f : to;
    limit[j] = to == -INFINITY ? -1.f : LIMIT;
  };
  float rs[2];   // the tile's sums
  auto probs = [&]() {
    rs[0] = rs[1] = 0.f;
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
#pragma unroll
          for (int e = 0; e < 4; e++) {
            s[b][i][j][e] = fast_exp2(fmaf(s[b][i][j][e], c2, -mu[j]));
            rs[j] += s[b][i][j][e];
          }
          pb[b][j].w[2 * i] = pack_bf16x2(s[b][i][j][0], s[b][i][j][1]);
          pb[b][j].w[2 * i + 1] = pack_bf16x2(s[b][i][j][2], s[b][i][j][3]);
        }
  };
  auto again = [&](int st, int kv0) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; b++) {
      const uint32_t at = (uint32_t)(st * 2 * TILE_B + b * BLOCK_B);
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) s[b][i][j] = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int c = 0; c < NC; c++)
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++) s[b][i][j] = mfma(lds_b128(M, rows[c] + at + i * GROUP_B), qf[j][c], s[b][i][j]);
    }
    mask(kv0);
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const float mx = tile_max(j), old = m[j];
      if (mx > old + 8.f) set_reference(j, mx);
      const float alpha = fast_exp2(old - mu[j]);
      l[j] *= alpha;
#pragma unroll
      for (int n = 0; n < NN; n++) acc[n][j] *= alpha;
    }
    probs();
  };

  constexpr int AHEAD = 4;    // natural-layout fragments read ahead of their MFMAs
  constexpr int VAHEAD = 2;   // transposed fragments
  auto tile = [&](auto STt, int kv0, bool live) {
    constexpr int ST = decltype(STt)::value;
    constexpr uint32_t AT = ST * 2 * TILE_B;
    wait_loads<0>();
    phase_barrier();   // the tile has landed, and every wavefront is done with the other stage
    bf16x8 fr[2 * NS], fv[2 * NN];
    // fragment x: block x / NS, column chunk x % NS / 2, row group x % 2
    auto read_row = [&](int x) { fr[x] = lds_b128(M, rows[x % NS / 2] + AT + x / NS * BLOCK_B + x % 2 * GROUP_B); };
    auto read_v = [&](int x) { fv[x] = read_col<HD>(M, cols[x % NN] + AT + x / NN * BLOCK_B); };
    // A tile past the end, or wholly above the diagonal of this wavefront's rows, or a wavefront without a row (uniform over
    // the wavefront): only the next tile's loads are wanted.
    if (!live || (t.causal && kv0 > wave_last_q) || wave_first_q >= t.seg_len) {
#pragma unroll
      for (int x = 0; x < 2 * PER_WAVE; x++) issue_part(1 - ST, kv0 + BKV, x);
      return;
    }
#pragma unroll
    for (int x = 0; x < AHEAD; x++) read_row(x);
    // Scores; the next tile's loads go out one behind each of the first slots, so the wavefront does not stand still while the
    // memory pipeline takes them.
#pragma unroll
    for (int x = 0; x < 2 * NS; x++) {
      if (x + AHEAD < 2 * NS) read_row(x + AHEAD);
      const int b = x / NS, c = x % NS / 2, i = x % 2;
#pragma unroll
      for (int j = 0; j < 2; j++) s[b][i][j] = mfma(fr[x], qf[j][c], c == 0 ? f32x4{0, 0, 0, 0} : s[b][i][j]);
      if (x < 2 * PER_WAVE) issue_part(1 - ST, kv0 + BKV, x);
      MLLM_SLOT_END;
    }
#pragma unroll
    for (int x = 0; x < VAHEAD; x++) read_v(x);   // their latency runs under the vector work
    MLLM_SLOT_END;
    mask(kv0);
    if (kv0 == 0) {
#pragma unroll
      for (int j = 0; j < 2; j++) set_reference(j, tile_max(j));
    }
    probs();
    if (__any(rs[0] > limit[0] || rs[1] > limit[1])) again(ST, kv0);
    l[0] += rs[0];
    l[1] += rs[1];
    MLLM_SLOT_END;
#pragma unroll
    for (int x = 0; x < 2 * NN; x++) {
      if (x + VAHEAD < 2 * NN) read_v(x + VAHEAD);
#pragma unroll
      for (int j = 0; j < 2; j++) acc[x % NN][j] = mfma(fv[x], pb[x / NN][j].v, acc[x % NN][j]);
      MLLM_SLOT_END;
    }
  };

#pragma unroll
  for (int j = 0; j < 2 * PER_WAVE; j++) issue_part(0, 0, j);
  for (int kv0 = 0; kv0 < kv_end; kv0 += 2 * BKV) {
    tile(Int<0>{}, kv0, true);
    tile(Int<1>{}, kv0 + BKV, kv0 + BKV < kv_end);
  }
  // the last enqueued loads (rows past the end: zeros) must have landed before this workgroup's
  // LDS can be handed to another one
  wait_loads<0>();
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const float sum = own_row_sum(l[j]);
    if (qrow[j] >= t.seg_len) continue;
    const int64_t row = t.seg_start + qrow[j];
    store_row<HD>(p.o + row * p.o_stride + head * HD + 4 * L.g, acc, j, 1.f / sum);
    if (L.g == 0) p.lse[(int64_t)head * p.T + row] = (m[j] + log2f(sum)) * LN2;
  }
}

// ---------------------------------------------------------------------------------------------
// forward, head_dim 64: the same walk with v_mfma_f32_32x32x16_bf16: lane l owns query l%32, and with h = l/32 the keys
// 8i + 4h .. +3 of a block.  Here the vector ALU is the bound and the clock 2.2 GHz, so the 16x16x32 form gives little (46 x 576 tokens, 16
// heads: 109 us at first, 95 with the maximum off the path and without the wavefronts that have no row (130 and 112 on another card), 92
// with that form as well),
// and it adds up in another order: through the roundings of a stage of 24 encoder and 8 decoder layers that moves the gradients by
// 0.044 of their norm, as much as they are from exact ones, where this order leaves the encoder's outputs to the bit (0.020 with the
// other kernels' orders alone).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void attn_fwd_64_kernel(AttnParams p) {
  constexpr int HD = 64, NC = HD / 16, ND = HD / 32, NB = BKV / 32, TILE_B = BKV * HD * 2, BLOCK_B = 32 * HD * 2, HALF_B = 16 * HD * 2;
  // two stages of a K tile and a V tile
  __shared__ __attribute__((aligned(1024))) char lds[4 * TILE_B];
  AttnItem t;
  if (!work_item(p.list, t, blockIdx.x)) return;
  const int head = t.head, kvh = head / (p.Hq / p.Hkv);
  const Lane L(threadIdx.x);
  const int h = L.lane >> 5, c32 = L.lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_first_q = t.tile0 + 32 * wave, wave_last_q = wave_first_q + 31;
  const int qrow = wave_first_q + c32;
  const bool qok = qrow < t.seg_len;
  const bf16_t* qp = p.q + (int64_t)(t.seg_start + qrow) * p.q_stride + head * HD + 8 * h;
  bf16x8 qf[NC];
#pragma unroll
  for (int c = 0; c < NC; c++) qf[c] = global_frag(qp + 16 * c, qok);
  const int kv_end = t.causal ? min(t.seg_len, t.tile0 + ATTN_FWD_Q_TILE) : t.seg_len;

  f32x16 oacc[ND];
#pragma unroll
  for (int d = 0; d < ND; d++)
#pragma unroll
    for (int v = 0; v < 16; v++) oacc[d][v] = 0.f;
  const float c2 = p.scale_log2e;
  // Reference maximum m (in units of log2: score * scale * log2(e)) and sum l of exp2(... - m).  The reference is the row's maximum
  // over the first tile and moves when a later tile exceeds it by more than 8: probabilities reach 2^8 at most, at the same relative
  // precision in fp32 sums and in the bf16 operand.  A tile that exceeds it shows in its sum: only where one comes out above 2^8 (or past
  // the range of fp32) is the largest probability looked for, and only where that is above 2^8 are the scores formed again, their
  // maximum taken and the accumulator rescaled (`again`); so neither the maximum of a tile's scores nor its exchange between the
  // halves is on the path, and a tile formed again moves the reference.  (On the sum alone 32 probabilities of 8 were enough to form
  // every tile again: 4 x 1500 tokens, 16 heads, keys behind the first 64 scoring 2.5 to 5 nats higher 79 to 83 us and now 55 to 57; other keys 54.)
  constexpr float LIMIT = 256.f;
  float m = -INFINITY, mu = 0.f, l = 0.f, limit = -1.f;   // mu: m, or 0 where there is none yet; limit -1: no reference yet

  // Rows past kv_end are outside the descriptors: zeros, no traffic.
  const i32x4_t rk = rows_rsrc(p.k + (int64_t)t.seg_start * p.kv_stride + kvh * HD, p.kv_stride, kv_end, HD);
  const i32x4_t rv = rows_rsrc(p.v + (int64_t)t.seg_start * p.kv_stride + kvh * HD, p.kv_stride, kv_end, HD);
  constexpr int PER_WAVE = BKV * HD / 8 / 64 / 4;
  uint32_t kv_off[PER_WAVE];
#pragma unroll
  for (int i = 0; i < PER_WAVE; i++) kv_off[i] = load_offset<HD, 32>(L, wave * PER_WAVE + i, p.kv_stride);
  const uint32_t row_bytes = (uint32_t)(p.kv_stride * 2);
  const uint32_t lds_b = __builtin_amdgcn_readfirstlane(lds_address((MLLM_LDS const void*)lds) + wave * PER_WAVE * 1024);
  auto issue_part = [&](int st, int kv0, int j) {   // j even: K, odd: V
    load_to_lds_b128(j % 2 ? rv : rk, lds_b + (uint32_t)(st * 2 * TILE_B + j % 2 * TILE_B + j / 2 * 1024), kv_off[j / 2], (uint32_t)kv0 * row_bytes);
  };
  const lds_cptr M = (lds_cptr)lds;
  // natural-layout operand: row l%32 of a block, columns 16c + 8h .. +7; transposed operand: column 32d + l%32 of the tile, contraction
  // slots e = 0..7 standing for rows 4h + e%4 (+8 for e >= 4) of half a block
  uint32_t rows[NC], cols[ND][2];
#pragma unroll
  for (int c = 0; c < NC; c++) rows[c] = (uint32_t)(c32 * HD + 8 * ((2 * c + h) ^ swz<HD, 32>(c32))) * 2u;
#pragma unroll
  for (int d = 0; d < ND; d++)
#pragma unroll
    for (int e = 0; e < 2; e++) {
      const int k = 4 * h + (L.c16 >> 2) + 8 * e, n = 32 * d + 16 * (L.g & 1) + 4 * (L.c16 & 3);
      cols[d][e] = (uint32_t)(k * HD + 8 * ((n >> 3) ^ swz<HD, 32>(k)) + (n & 7)) * 2u + TILE_B;
    }
  auto mfma32 = [](bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); };

  f32x16 s[NB];          // scores, then probabilities
  Frag8 pf[NB][2];       // probabilities as MFMA operand
  float rs;              // the tile's sum over the lane's keys
  auto mask = [&](int kv0) {
    if ((kv0 + BKV > t.seg_len) || (t.causal && kv0 + BKV - 1 > wave_first_q)) {   // the tile crosses the segment end or the diagonal
#pragma unroll
      for (int b = 0; b < NB; b++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int kv = kv0 + 32 * b + 8 * (v >> 2) + 4 * h + (v & 3);
          s[b][v] = (kv < t.seg_len && (!t.causal || kv <= qrow)) ? s[b][v] : -INFINITY;
        }
    }
  };
  auto tile_max = [&]() {
    float mx = s[0][0];
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int v = 0; v < 16; v++) mx = fmaxf(mx, s[b][v]);
    return fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;
  };
  auto set_reference = [&](float to) {
    m = to;
    mu = to == -INFINITY ? 0.f : to;
    limit = to == -INFINITY ? -1.f : LIMIT;
  };
  auto largest = [&]() {   // probability of the lane's keys
    float mx = s[0][0];
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int v = 0; v < 16; v++) mx = fmaxf(mx, s[b][v]);
    return mx;
  };
  auto probs = [&]() {
    rs = 0.f;
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        s[b][v] = fast_exp2(fmaf(s[b][v], c2, -mu));
        rs += s[b][v];
      }
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int w = 0; w < 8; w++) pf[b][w >> 2].w[w & 3] = pack_bf16x2(s[b][2 * w], s[b][2 * w + 1]);
  };
  auto again = [&](int st, int kv0) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < NB; b++) {
#pragma unroll
      for (int v = 0; v < 16; v++) s[b][v] = 0.f;
#pragma unroll
      for (int c = 0; c < NC; c++) s[b] = mfma32(lds_b128(M, rows[c] + (uint32_t)(st * 2 * TILE_B + b * BLOCK_B)), qf[c], s[b]);
    }
    mask(kv0);
    const float mx = tile_max(), old = m;
    if (mx > old + 8.f) set_reference(mx);
    const float alpha = fast_exp2(old - mu);
    l *= alpha;
#pragma unroll
    for (int d = 0; d < ND; d++)
#pragma unroll
      for (int v = 0; v < 16; v++) oacc[d][v] *= alpha;
    probs();
  };

  constexpr int AHEAD = 4, VAHEAD = 1;   // natural-layout and transposed fragments read ahead of their MFMAs
  auto tile = [&](auto STt, int kv0, bool live) {
    constexpr int ST = decltype(STt)::value;
    constexpr uint32_t AT = ST * 2 * TILE_B;
    wait_loads<0>();
    phase_barrier();   // the tile has landed, and every wavefront is done with the other stage
    // A tile past the end, or wholly above the diagonal of this wavefront's rows, or a wavefront without a row (uniform over
    // the wavefront): only the next tile's loads are wanted.
    if (!live || (t.causal && kv0 > wave_last_q) || wave_first_q >= t.seg_len) {
#pragma unroll
      for (int x = 0; x < 2 * PER_WAVE; x++) issue_part(1 - ST, kv0 + BKV, x);
      return;
    }
    constexpr int NSC = NC * NB, NPV = NB * 2 * ND;
    bf16x8 fr[NSC];        // fragment x: column chunk x / NB, block x % NB
    Frag8 fv[NPV];         // fragment x: half block x / ND, columns x % ND
    auto read_row = [&](int x) { fr[x] = lds_b128(M, rows[x / NB] + AT + x % NB * BLOCK_B); };
    auto read_v = [&](int x) {
#pragma unroll
      for (int e = 0; e < 2; e++) fv[x].h[e] = lds_tr(M, cols[x % ND][e] + AT + x / ND * HALF_B);
    };
#pragma unroll
    for (int x = 0; x < AHEAD; x++) read_row(x);
    // Scores; the next tile's loads go out one behind each of the first slots, so the wavefront does not stand still while the
    // memory pipeline takes them.
#pragma unroll
    for (int x = 0; x < NSC; x++) {
      if (x + AHEAD < NSC) read_row(x + AHEAD);
      if (x < NB) {
#pragma unroll
        for (int v = 0; v < 16; v++) s[x][v] = 0.f;
      }
      s[x % NB] = mfma32(fr[x], qf[x / NB], s[x % NB]);
      static_assert(2 * PER_WAVE <= NSC, "a slot for every load");
      if (x < 2 * PER_WAVE) issue_part(1 - ST, kv0 + BKV, x);
      MLLM_SLOT_END;
    }
#pragma unroll
    for (int x = 0; x < VAHEAD; x++) read_v(x);   // their latency runs under the vector work
    MLLM_SLOT_END;
    mask(kv0);
    if (kv0 == 0) set_reference(tile_max());
    probs();
    if (__any(rs > limit) && __any(largest() > limit - 0.01f)) again(ST, kv0);   // 0.01: more than the exponential's rounding
    l += rs;
    MLLM_SLOT_END;
#pragma unroll
    for (int x = 0; x < NPV; x++) {
      if (x + VAHEAD < NPV) read_v(x + VAHEAD);
      oacc[x % ND] = mfma32(fv[x].v, pf[x / ND / 2][x / ND % 2].v, oacc[x % ND]);
      MLLM_SLOT_END;
    }
  };

#pragma unroll
  for (int j = 0; j < 2 * PER_WAVE; j++) issue_part(0, 0, j);
  for (int kv0 = 0; kv0 < kv_end; kv0 += 2 * BKV) {
    tile(Int<0>{}, kv0, true);
    tile(Int<1>{}, kv0 + BKV, kv0 + BKV < kv_end);
  }
  // the last enqueued loads (rows past the end: zeros) must have landed before this workgroup's
  // LDS can be handed to another one
  wait_loads<0>();
  l += __shfl_xor(l, 32, 64);
  if (!qok) return;
  const float inv = 1.f / l;
  bf16_t* op = p.o + (int64_t)(t.seg_start + qrow) * p.o_stride + head * HD;
#pragma unroll
  for (int d = 0; d < ND; d++)
#pragma unroll
    for (int g4 = 0; g4 < 4; g4++) {
      uint2 w;
      w.x = pack_bf16x2(oacc[d][4 * g4] * inv, oacc[d][4 * g4 + 1] * inv);
      w.y = pack_bf16x2(oacc[d][4 * g4 + 2] * inv, oacc[d][4 * g4 + 3] * inv);
      *reinterpret_cast<uint2*>(op + 32 * d + 8 * g4 + 4 * h) = w;
    }
  if (h == 0) p.lse[(int64_t)head * p.T + t.seg_start + qrow] = (m + log2f(l)) * LN2;
}

// ---------------------------------------------------------------------------------------------
// dQ pass: one workgroup per (query tile of 128, head), looping over key tiles.  It runs first in
// the backward pass and also produces delta[h][t] = sum_d dO[t,h,d] * O[t,h,d] for the dK/dV pass.
// dO enters negated and the dP products start from delta, so that they end as delta - dP: the subtraction costs no
// instruction, and dQ, which comes out negated, takes its sign back with the softmax scale.
// ---------------------------------------------------------------------------------------------
template <int HD>
__device__ __forceinline__ void attn_bwd_dq(const AttnParams& p, const AttnItem* list, int entry, char* lds) {
  constexpr int NC = HD / 32, NN = HD / 16, NS = 2 * NC, TILE_B = BKV * HD * 2, BLOCK_B = 32 * HD * 2, GROUP_B = 16 * HD * 2;
  AttnItem t;
  if (!work_item(list, t, entry)) return;
  const int head = t.head, kvh = head / (p.Hq / p.Hkv);
  const Lane L(threadIdx.x);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_first_q = t.tile0 + 32 * wave, wave_last_q = wave_first_q + 31;
  int qrow[2];
  bf16x8 qf[2][NC], dof[2][NC];
  Frag8 of[2][NC];
  float lse[2];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    qrow[j] = wave_first_q + 16 * j + L.c16;
    const bool ok = qrow[j] < t.seg_len;
    const int64_t row = t.seg_start + (ok ? qrow[j] : 0);
    const bf16_t* qp = p.q + row * p.q_stride + head * HD + 8 * L.g;
    const bf16_t* dop = p.d_o + row * p.o_stride + head * HD + 8 * L.g;
    const bf16_t* op = p.o + row * p.o_stride + head * HD + 8 * L.g;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      qf[j][c] = global_frag(qp + 32 * c, ok);
      of[j][c].v = global_frag(op + 32 * c, ok);
      dof[j][c] = global_frag(dop + 32 * c, ok);
    }
    lse[j] = p.lse[(int64_t)head * p.T + row];
  }
  const int kv_end = t.causal ? min(t.seg_len, t.tile0 + ATTN_FWD_Q_TILE) : t.seg_len;
  const i32x4_t rk = rows_rsrc(p.k + (int64_t)t.seg_start * p.kv_stride + kvh * HD, p.kv_stride, kv_end, HD);
  const i32x4_t rv = rows_rsrc(p.v + (int64_t)t.seg_start * p.kv_stride + kvh * HD, p.kv_stride, kv_end, HD);
  constexpr int PER_WAVE = BKV * HD / 8 / 64 / 4;
  uint32_t kv_off[PER_WAVE];
#pragma unroll
  for (int i = 0; i < PER_WAVE; i++) kv_off[i] = load_offset<HD>(L, wave * PER_WAVE + i, p.kv_stride);
  const uint32_t row_bytes = (uint32_t)(p.kv_stride * 2);
  const uint32_t lds_b = __builtin_amdgcn_readfirstlane(lds_address((MLLM_LDS const void*)lds) + wave * PER_WAVE * 1024);
  auto issue_part = [&](int st, int kv0, int j) {   // j even: K, odd: V; rows past kv_end: zeros, no traffic
    load_to_lds_b128(j % 2 ? rv : rk, lds_b + (uint32_t)(st * 2 * TILE_B + j % 2 * TILE_B + j / 2 * 1024), kv_off[j / 2], (uint32_t)kv0 * row_bytes);
  };
#pragma unroll
  for (int j = 0; j < 2 * PER_WAVE; j++) issue_part(0, 0, j);   // before anything waits for the rows above (5 x 576 tokens, 16 heads, both passes: 43.8 -> 42.9 us)

  float lse2[2], delta[2];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const bool ok = qrow[j] < t.seg_len;
    float d = 0.f;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      Frag8 fd;
      fd.v = dof[j][c];
#pragma unroll
      for (int w = 0; w < 4; w++) d += bf16lo(of[j][c].w[w]) * bf16lo(fd.w[w]) + bf16hi(of[j][c].w[w]) * bf16hi(fd.w[w]);
      dof[j][c] = negated(fd.v);
    }
    delta[j] = own_row_sum(d);
    // Rows beyond the segment get lse = +inf, so their probabilities are exp2(-inf) = 0.
    lse2[j] = ok ? lse[j] * LOG2E : INFINITY;
    if (ok && L.g == 0) p.delta[(int64_t)head * p.T + t.seg_start + qrow[j]] = delta[j];
  }
  const float c2 = p.scale_log2e;

  f32x4 acc[NN][2], start[2];
#pragma unroll
  for (int n = 0; n < NN; n++) acc[n][0] = acc[n][1] = f32x4{0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 2; j++) start[j] = f32x4{delta[j], delta[j], delta[j], delta[j]};

  const lds_cptr M = (lds_cptr)lds;
  uint32_t rows[NC], cols[NN];
#pragma unroll
  for (int c = 0; c < NC; c++) rows[c] = row_offset<HD>(L, c);
#pragma unroll
  for (int n = 0; n < NN; n++) cols[n] = col_offset<HD>(L, n);

  f32x4 s[2][2], dp[2][2];   // a block's scores and delta - dP: [row group][own group]
  constexpr int AHEAD = HD == 128 ? 2 : 4, CAHEAD = 2;   // fragments (pairs of them in the score stage) read ahead of their MFMAs
  auto tile = [&](auto STt, int kv0, bool live) {
    constexpr int ST = decltype(STt)::value;
    wait_loads<0>();
    phase_barrier();
    if (!live || (t.causal && kv0 > wave_last_q) || wave_first_q >= t.seg_len) {   // only the loads are wanted (see the forward kernel)
#pragma unroll
      for (int x = 0; x < 2 * PER_WAVE; x++) issue_part(1 - ST, kv0 + BKV, x);
      return;
    }
#pragma unroll
    for (int b = 0; b < 2; b++) {
      constexpr uint32_t AT0 = ST * 2 * TILE_B;
      const uint32_t AT = AT0 + b * BLOCK_B;
      bf16x8 fk[NS], fv[NS], fc[NN];
      auto read_row = [&](int x) {
        const uint32_t o = rows[x / 2] + AT + x % 2 * GROUP_B;
        fk[x] = lds_b128(M, o);
        fv[x] = lds_b128(M, o + TILE_B);
      };
      auto read_c = [&](int x) { fc[x] = read_col<HD>(M, cols[x] + AT); };
#pragma unroll
      for (int x = 0; x < AHEAD; x++) read_row(x);
#pragma unroll
      for (int x = 0; x < NS; x++) {
        if (x + AHEAD < NS) read_row(x + AHEAD);
#pragma unroll
        for (int j = 0; j < 2; j++) {
          s[x % 2][j] = mfma(fk[x], qf[j][x / 2], x < 2 ? f32x4{0, 0, 0, 0} : s[x % 2][j]);
          dp[x % 2][j] = mfma(fv[x], dof[j][x / 2], x < 2 ? start[j] : dp[x % 2][j]);
        }
        static_assert(2 * PER_WAVE == NS, "one load a slot");
        if (b == 0) issue_part(1 - ST, kv0 + BKV, x);   // the next tile's loads, one a slot (see the forward kernel)
        MLLM_SLOT_END;
      }
#pragma unroll
      for (int x = 0; x < CAHEAD; x++) read_c(x);   // their latency runs under the vector work
      MLLM_SLOT_END;
      const int k0 = kv0 + 32 * b;
      if ((k0 + 32 > t.seg_len) || (t.causal && k0 + 31 > wave_first_q)) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
              const int kv = k0 + 16 * i + 4 * L.g + e;
              s[i][j][e] = (kv < t.seg_len && (!t.causal || kv <= qrow[j])) ? s[i][j][e] : -INFINITY;
            }
      }
      Frag8 db[2];   // dS negated as MFMA operand
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
          float ds[4];
#pragma unroll
          for (int e = 0; e < 4; e++) ds[e] = fast_exp2(fmaf(s[i][j][e], c2, -lse2[j])) * dp[i][j][e];
          db[j].w[2 * i] = pack_bf16x2(ds[0], ds[1]);
          db[j].w[2 * i + 1] = pack_bf16x2(ds[2], ds[3]);
        }
      MLLM_SLOT_END;
#pragma unroll
      for (int x = 0; x < NN; x++) {
        if (x + CAHEAD < NN) read_c(x + CAHEAD);
#pragma unroll
        for (int j = 0; j < 2; j++) acc[x][j] = mfma(fc[x], db[j].v, acc[x][j]);
        MLLM_SLOT_END;
      }
    }
  };
  for (int kv0 = 0; kv0 < kv_end; kv0 += 2 * BKV) {
    tile(Int<0>{}, kv0, true);
    tile(Int<1>{}, kv0 + BKV, kv0 + BKV < kv_end);
  }
  wait_loads<0>();   // the last enqueued tile (zeros) has landed
#pragma unroll
  for (int j = 0; j < 2; j++) {
    if (qrow[j] >= t.seg_len) continue;
    if (p.rope_table) rope_unrotate<HD>(acc, j, p.rope_table, qrow[j], L.g, -p.scale);   // the scale rides on the rotation's factors
    store_row<HD>(p.dq + (int64_t)(t.seg_start + qrow[j]) * p.q_stride + head * HD + 4 * L.g, acc, j, p.rope_table ? 1.f : -p.scale);
  }
}

template <int HD>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[4 * BKV * HD * 2];
  attn_bwd_dq<HD>(p, p.list, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------------------------
// dK/dV pass at head_dim 64: one workgroup per (key tile of 128, kv head); each wavefront owns 32 key rows and
// loops over the query heads of the group and the query tiles of 64 that can see its keys, in the same four steps of two
// blocks.  The query-side tiles (Q, dO) have two stages in LDS, the row statistics beside them: lse times log2(e), delta.
// V enters negated (see the dQ pass).
// SELF_DELTA: delta is formed here, four threads a query row of the tile, instead of read from the dQ pass.
// ---------------------------------------------------------------------------------------------
constexpr int DKV_STAT_AT = 4 * BQ * 64 * 2, DKV_LDS_B = DKV_STAT_AT + 4 * BQ * 4;
template <bool SELF_DELTA>
__device__ __forceinline__ void attn_bwd_dkv(const AttnParams& p, const AttnItem* list, int entry, int part, int parts, char* lds) {
  constexpr int HD = 64, NC = HD / 32, NN = HD / 16, NS = 2 * NC, TILE_B = BQ * HD * 2, BLOCK_B = 32 * HD * 2, GROUP_B = 16 * HD * 2;
  AttnItem t;
  if (!work_item(list, t, entry)) return;
  const int kvh = t.head, grp = p.Hq / p.Hkv;
  const int tid = threadIdx.x;
  const Lane L(tid);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_first_k = t.tile0 + 32 * wave;
  int krow[2];
  bf16x8 kf[2][NC], vf[2][NC];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    krow[j] = wave_first_k + 16 * j + L.c16;
    const bool ok = krow[j] < t.seg_len;
    const int64_t at = (int64_t)(t.seg_start + (ok ? krow[j] : 0)) * p.kv_stride + kvh * HD + 8 * L.g;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      kf[j][c] = global_frag(p.k + at + 32 * c, ok);
      vf[j][c] = global_frag(p.v + at + 32 * c, ok);
    }
  }
  f32x4 dk[NN][2], dv[NN][2];
#pragma unroll
  for (int n = 0; n < NN; n++) dk[n][0] = dk[n][1] = dv[n][0] = dv[n][1] = f32x4{0, 0, 0, 0};

  const int q_begin = t.causal ? (t.tile0 / BQ) * BQ : 0;
  const KvRange range = kv_range(grp, q_begin, t.seg_len, BQ, part, parts);
  const int n_it = range.n_it;
  const float c2 = p.scale_log2e;

  constexpr int PER_WAVE = BQ * HD / 8 / 64 / 4;
  uint32_t q_off[PER_WAVE], do_off[PER_WAVE];
#pragma unroll
  for (int i = 0; i < PER_WAVE; i++) {
    q_off[i] = load_offset<HD>(L, wave * PER_WAVE + i, p.q_stride);
    do_off[i] = load_offset<HD>(L, wave * PER_WAVE + i, p.o_stride);
  }
  const uint32_t q_bytes = (uint32_t)(((int64_t)(t.seg_len - 1) * p.q_stride + HD) * 2);
  const uint32_t do_bytes = (uint32_t)(((int64_t)(t.seg_len - 1) * p.o_stride + HD) * 2);
  const uint32_t lds_b = __builtin_amdgcn_readfirstlane(lds_address((MLLM_LDS const void*)lds) + wave * PER_WAVE * 1024);

  // The tile to be loaded next: query head nj of the group, query rows from nq0.  Past the last
  // tile the descriptors are empty and the loads write zeros.
  int nj = range.head, nq0 = range.q0;
  float r_lse = 0.f, r_delta = 0.f;   // statistics of the tile in flight, one row per thread (tid < BQ)
  bool r_ok = false;
  u32x4_t r_o[2], r_do[2];             // SELF_DELTA: the thread's 16 columns of O and dO
  auto issue = [&](int st) {
    const bool valid = nj < grp;
    const int head = kvh * grp + (valid ? nj : 0);
    const bf16_t* dos = p.d_o + (int64_t)t.seg_start * p.o_stride + head * HD;
    const i32x4_t rq = raw_rsrc(p.q + (int64_t)t.seg_start * p.q_stride + head * HD, valid ? q_bytes : 0u);
    const i32x4_t rdo = raw_rsrc(dos, valid ? do_bytes : 0u);
    const uint32_t qrow = (uint32_t)nq0 * (uint32_t)(p.q_stride * 2), dorow = (uint32_t)nq0 * (uint32_t)(p.o_stride * 2);
    const uint32_t so = tid < BQ ? (uint32_t)(nq0 + tid) * 4u : 0xFFFFFFFFu;
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(p.lse + (int64_t)head * p.T + t.seg_start), 0, valid ? t.seg_len * 4 : 0, 0x00020000);
    r_lse = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rl, (int)so, 0, 0));
    if constexpr (SELF_DELTA) {
      const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(dos), 0, valid ? (int)do_bytes : 0, 0x00020000);
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
          p.o + (int64_t)t.seg_start * p.o_stride + head * HD, 0, valid ? (int)do_bytes : 0, 0x00020000);
      const uint32_t at = dorow + (uint32_t)(tid >> 2) * (uint32_t)(p.o_stride * 2) + (uint32_t)(tid & 3) * 32u;
#pragma unroll
      for (int w = 0; w < 2; w++) {
        r_o[w] = __builtin_amdgcn_raw_buffer_load_b128(ro, (int)(at + 16u * w), 0, 0);
        r_do[w] = __builtin_amdgcn_raw_buffer_load_b128(rd, (int)(at + 16u * w), 0, 0);
      }
    } else {
      const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(p.delta + (int64_t)head * p.T + t.seg_start), 0, valid ? t.seg_len * 4 : 0, 0x00020000);
      r_delta = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rd, (int)so, 0, 0));
    }
#pragma unroll
    for (int i = 0; i < PER_WAVE; i++) {
      load_to_lds_b128(rq, lds_b + (uint32_t)(st * 2 * TILE_B + i * 1024), q_off[i], qrow);
      load_to_lds_b128(rdo, lds_b + (uint32_t)(st * 2 * TILE_B + TILE_B + i * 1024), do_off[i], dorow);
    }
    r_ok = valid && tid < BQ && nq0 + tid < t.seg_len;
    nq0 += BQ;
    if (nq0 >= t.seg_len) { nq0 = q_begin; nj++; }
  };
  const lds_cptr M = (lds_cptr)lds;
  float* const stats = (float*)(lds + DKV_STAT_AT);   // [stage][lse * log2(e), delta][BQ]
  uint32_t rows[NC], cols[NN];
#pragma unroll
  for (int c = 0; c < NC; c++) rows[c] = row_offset<HD>(L, c);
#pragma unroll
  for (int n = 0; n < NN; n++) cols[n] = col_offset<HD>(L, n);
  const uint32_t stat_rows = DKV_STAT_AT + 16u * L.g;

  f32x4 s[2][2][2], dp[2][2][2];   // [block][row group][own group]: scores, delta - dP
  f32x4 ls[2][2], de[2][2];        // [block][row group]: statistics of the lane's rows
  Frag8 pb[2][2], db[2][2];        // P and dS (negated) as MFMA operands: [block][own group]
  auto mask = [&](int b, int q0) {
    const int r0 = q0 + 32 * b;
    if (t.causal && r0 <= wave_first_k + 31) {   // block touches the diagonal
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
          for (int e = 0; e < 4; e++) s[b][i][j][e] = (krow[j] <= r0 + 16 * i + 4 * L.g + e) ? s[b][i][j][e] : -INFINITY;
    }
  };
  auto grad = [&](int b, int v) {   // elements v, v+1 of a block
    const int i = v >> 3, j = (v >> 2) & 1, e = v & 3;
    const float x = fast_exp2(fmaf(s[b][i][j][e], c2, -ls[b][i][e])), y = fast_exp2(fmaf(s[b][i][j][e + 1], c2, -ls[b][i][e + 1]));
    pb[b][j].w[2 * i + (e >> 1)] = pack_bf16x2(x, y);
    db[b][j].w[2 * i + (e >> 1)] = pack_bf16x2(x * dp[b][i][j][e], y * dp[b][i][j][e + 1]);
  };
  constexpr int AHEAD = 2, CAHEAD = 1;
  constexpr int EPS = 16 / NS, EPV = 16 / NN;

  // One tile: publish the statistics of the tile whose loads were enqueued a tile ago, wait for
  // those loads, barrier (every wavefront is now done with the other stage), enqueue the next
  // tile into the other stage, multiply.
  auto tile = [&](auto STt, int q0, bool live) {
    constexpr int ST = decltype(STt)::value;
    constexpr uint32_t AT = ST * 2 * TILE_B;
    if (tid < BQ) {
      stats[ST * 2 * BQ + tid] = r_ok ? r_lse * LOG2E : INFINITY;   // +inf: probabilities of rows past the segment are 0
      if constexpr (!SELF_DELTA) stats[ST * 2 * BQ + BQ + tid] = r_ok ? r_delta : 0.f;
    }
    if constexpr (SELF_DELTA) {   // rows past the segment, and the tile past the last one, have come as zeros
      float d = 0.f;
#pragma unroll
      for (int w = 0; w < 2; w++)
#pragma unroll
        for (int e = 0; e < 4; e++) d += bf16lo(r_o[w][e]) * bf16lo(r_do[w][e]) + bf16hi(r_o[w][e]) * bf16hi(r_do[w][e]);
      d += __shfl_xor(d, 1, 64);
      d += __shfl_xor(d, 2, 64);
      if ((tid & 3) == 0) stats[ST * 2 * BQ + BQ + (tid >> 2)] = d;
    }
    wait_loads<0>();
    phase_barrier();
    issue(1 - ST);
    MLLM_SLOT_END;
    if (!live || (t.causal && q0 + BQ - 1 < wave_first_k) || wave_first_k >= t.seg_len) return;   // no query here sees this wavefront's keys, or it has none
    bf16x8 fq[2 * NS], fo[2 * NS], cq[2 * NN], co[2 * NN];
    auto read_row = [&](int x) {
      const uint32_t o = rows[x % NS / 2] + AT + x / NS * BLOCK_B + x % 2 * GROUP_B;
      fq[x] = lds_b128(M, o);
      fo[x] = lds_b128(M, o + TILE_B);
    };
    auto read_c = [&](int x) {
      const uint32_t o = cols[x % NN] + AT + x / NN * BLOCK_B;
      cq[x] = read_col<HD>(M, o);
      co[x] = read_col<HD>(M, o + TILE_B);
    };
    auto read_stats = [&](int b) {
#pragma unroll
      for (int i = 0; i < 2; i++) {
        de[b][i] = lds_f4(M, stat_rows + (uint32_t)((ST * 2 * BQ + BQ + 32 * b + 16 * i) * 4));
        ls[b][i] = lds_f4(M, stat_rows + (uint32_t)((ST * 2 * BQ + 32 * b + 16 * i) * 4));
      }
    };
    auto score = [&](int x) {
      const int b = x / NS, c = x % NS / 2, i = x % 2;
#pragma unroll
      for (int j = 0; j < 2; j++) {
        s[b][i][j] = mfma(fq[x], kf[j][c], c == 0 ? f32x4{0, 0, 0, 0} : s[b][i][j]);
        dp[b][i][j] = mfma(fo[x], vf[j][c], c == 0 ? de[b][i] : dp[b][i][j]);
      }
    };
    auto output = [&](int x) {
#pragma unroll
      for (int j = 0; j < 2; j++) {
        dv[x % NN][j] = mfma(co[x], pb[x / NN][j].v, dv[x % NN][j]);
        dk[x % NN][j] = mfma(cq[x], db[x / NN][j].v, dk[x % NN][j]);
      }
    };
    read_stats(0);
#pragma unroll
    for (int x = 0; x < AHEAD; x++) read_row(x);
#pragma unroll
    for (int x = 0; x < NS; x++) {
      read_row(x + AHEAD);
      if (x == NS - 1) read_stats(1);
      score(x);
      MLLM_SLOT_END;
    }
    mask(0, q0);
    MLLM_SLOT_END;
#pragma unroll
    for (int x = NS; x < 2 * NS; x++) {
      if (x + AHEAD < 2 * NS) read_row(x + AHEAD);
      else if (x - (2 * NS - AHEAD) < CAHEAD) read_c(x - (2 * NS - AHEAD));
      score(x);
#pragma unroll
      for (int v = (x - NS) * EPS; v < (x - NS + 1) * EPS; v += 2) grad(0, v);
      MLLM_SLOT_END;
    }
    mask(1, q0);
    MLLM_SLOT_END;
#pragma unroll
    for (int x = 0; x < NN; x++) {
      read_c(x + CAHEAD);
      output(x);
#pragma unroll
      for (int v = x * EPV; v < (x + 1) * EPV; v += 2) grad(1, v);
      MLLM_SLOT_END;
    }
#pragma unroll
    for (int x = NN; x < 2 * NN; x++) {
      if (x + CAHEAD < 2 * NN) read_c(x + CAHEAD);
      output(x);
      MLLM_SLOT_END;
    }
  };

  issue(0);
#pragma unroll
  for (int j = 0; j < 2; j++)
#pragma unroll
    for (int c = 0; c < NC; c++) vf[j][c] = negated(vf[j][c]);   // once the first tile is on its way
  int q0 = range.q0;
  auto advance = [&]() { q0 += BQ; if (q0 >= t.seg_len) q0 = q_begin; };
  for (int it = 0; it < n_it; it += 2) {
    tile(Int<0>{}, q0, true);
    advance();
    tile(Int<1>{}, q0, it + 1 < n_it);
    advance();
  }
  // the last enqueued loads (an empty tile: zeros) must have landed before this workgroup's LDS
  // can be handed to another one
  wait_loads<0>();
#pragma unroll
  for (int j = 0; j < 2; j++) {
    if (krow[j] >= t.seg_len) continue;
    const int64_t row = t.seg_start + krow[j];
    store_dk<HD>(p, dk, j, krow[j], row, kvh, L.g, parts > 1, (unsigned)part);
    store_dv<HD>(p, dv, j, row, kvh, L.g, parts > 1, (unsigned)part);
  }
}

__global__ __launch_bounds__(256, 2) void attn_bwd_dkv_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[DKV_LDS_B];
  attn_bwd_dkv<false>(p, p.list, blockIdx.x, blockIdx.y, gridDim.y, lds);
}
// Both passes in one launch, the dK/dV pass first.
__global__ __launch_bounds__(256, 2) void attn_bwd_both_kernel(AttnParams p, const AttnItem* kv_list, int kv_grid, int kv_parts) {
  __shared__ __attribute__((aligned(1024))) char lds[DKV_LDS_B];
  const int kv = kv_grid * kv_parts, pid = blockIdx.x;
  if (pid < kv) attn_bwd_dkv<true>(p, kv_list, pid % kv_grid, pid / kv_grid, kv_parts, lds);
  else attn_bwd_dq<64>(p, p.list, pid - kv, lds);
}

// ---------------------------------------------------------------------------------------------
// dK/dV pass at head_dim 128: one workgroup of eight wavefronts per (key tile of 128, kv head), two wavefronts on a
// SIMD.  The work of a block of 32 query rows falls into two halves that hold one accumulator each, so that two
// wavefronts fit where one that does all of it needs the whole register file:
//   wavefronts 0..3 (keys 32 w ..):  S = Q.K^T, P = exp2(S scale log2 e - lse log2 e), dV^T += dO^T.P
//   wavefronts 4..7 (the same keys): dP = dO.V^T - delta, dS = P * dP, dK^T += Q^T.dS
// P goes from the one to the other through LDS in fp32, lane for lane.  Both are pipelined over phases of one block, a
// barrier each; in phase n
//   the first:  dV of block n-1 (exponents of n formed under it), then S of n+1 (P of n formed and written under it)
//   the second: dK of block n-2 (P of n-1 read under it), then dP of n (dS of n-1 formed under it)
// so every product is formed from operands that have been at hand since the phase before, and a block passes through in
// three phases.  Q blocks rotate through 8 stages of LDS (n-2 .. n+1 are read, n+2 .. n+4 on their way), dO blocks through 4
// (n-1 and n, n+1 and n+2); eight phases are unrolled, so that a stage is an offset in the instruction.
// One wavefront per SIMD that did both halves was bound by its own instruction issue, 11 instructions a 32x32x16 MFMA at one
// every 4 to 6 clocks: 13255 causal tokens, 32/8 heads, 5.93 M cycles with the MFMAs busy 47 %, now 5.10 M and 55 %, 2915 -> 2467
// us on one card.  What is left is spread evenly: without the exchange of P 9 % less time, without the loads 9 %, without the
// natural reads 7 %, the transposing ones 15 %, the exponentials 5 %, without all of them 25 %.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(512, 2) void attn_bwd_dkv_duo_kernel(AttnParams p) {
  constexpr int HD = 128, NC = HD / 32, NN = HD / 16, NS = 2 * NC, QB = 32;   // QB: query rows of a block
  constexpr int BLOCK_B = QB * HD * 2, GROUP_B = 16 * HD * 2;
  constexpr int NQ = 8, NO = 4;                                  // stages of Q and of dO
  constexpr int DO_AT = NQ * BLOCK_B, P_AT = DO_AT + NO * BLOCK_B, P_SLOT = 4 * 4096, STAT_AT = P_AT + 2 * P_SLOT;
  constexpr int STAT_B = 256, WAVE_STAT_B = NQ * STAT_B;         // a wavefront's own row statistics, a stage each
  // One array on purpose: the compiler tags LDS accesses with the variable they belong to, and with a single one there is
  // nothing to tag.
  __shared__ __attribute__((aligned(1024))) char lds[STAT_AT + 8 * WAVE_STAT_B];
  AttnItem t;
  if (!work_item(p.list, t, blockIdx.x)) return;
  const int kvh = t.head, grp = p.Hq / p.Hkv;
  const int tid = threadIdx.x;
  const Lane L(tid);
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave8 & 3;
  const bool second = wave8 >= 4;
  const int wave_first_k = t.tile0 + 32 * wave;
  int krow[2];
  // The wavefront's K, or V negated: dP products that start from delta end as delta - dP, and dK takes its sign back with the scale.
  bf16x8 kvf[2][NC];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    krow[j] = wave_first_k + 16 * j + L.c16;
    const bool ok = krow[j] < t.seg_len;
    const bf16_t* kvp = (second ? p.v : p.k) + (int64_t)(t.seg_start + (ok ? krow[j] : 0)) * p.kv_stride + kvh * HD + 8 * L.g;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      kvf[j][c] = global_frag(kvp + 32 * c, ok);
    }
  }
  f32x4 acc[NN][2];   // dV, or dK negated
#pragma unroll
  for (int n = 0; n < NN; n++) acc[n][0] = acc[n][1] = f32x4{0, 0, 0, 0};

  const int q_begin = t.causal ? (t.tile0 / BQ) * BQ : 0;
  const KvRange range = kv_range(grp, q_begin, t.seg_len, QB, blockIdx.y, gridDim.y);
  const int n_it = range.n_it;
  const float c2 = p.scale_log2e;

  // ---- loads: the first wavefronts bring Q and lse, the second dO and delta, 8 rows each -----------
  constexpr int PER_WAVE = QB * HD / 8 / 64 / 4, PT = PER_WAVE + 1;   // PT: instructions per wavefront and block
  const int64_t in_stride = second ? p.o_stride : p.q_stride;
  const bf16_t* const in = (second ? p.d_o : p.q) + (int64_t)t.seg_start * in_stride;
  const float* const in_stat = (second ? p.delta : p.lse) + t.seg_start;
  uint32_t in_off[PER_WAVE];
#pragma unroll
  for (int i = 0; i < PER_WAVE; i++) in_off[i] = load_offset<HD>(L, wave * PER_WAVE + i, in_stride);
  const uint32_t in_bytes = (uint32_t)(((int64_t)(t.seg_len - 1) * in_stride + HD) * 2);
  const uint32_t in_row = (uint32_t)(in_stride * 2);
  int nj = range.head, nq0 = range.q0, to_load = n_it;   // the block to be loaded next: query head nj of the group, rows from nq0
  const uint32_t lds_b = lds_address((MLLM_LDS const void*)lds);
  const uint32_t load_at = __builtin_amdgcn_readfirstlane(lds_b + (second ? DO_AT : 0) + wave * PER_WAVE * 1024);
  const uint32_t stat_off = STAT_AT + (uint32_t)wave8 * WAVE_STAT_B;
  const uint32_t stat_at = __builtin_amdgcn_readfirstlane(lds_b + stat_off);
  // Past the last block the descriptors are empty and the loads write zeros.  Rows past the segment read as zero as well
  // (their lse and delta too): they add nothing, as their dO rows are zero.
  i32x4_t rin, rst;
  auto set_head = [&]() {
    const bool valid = to_load > 0;
    const int head = kvh * grp + (valid ? nj : 0);
    rin = raw_rsrc(in + head * HD, valid ? in_bytes : 0u);
    rst = raw_rsrc(in_stat + (int64_t)head * p.T, valid ? (uint32_t)t.seg_len * 4u : 0u);
  };
  set_head();
  auto issue_part = [&](int stage, int j) {
    if (j < PER_WAVE) load_to_lds_b128(rin, load_at + (uint32_t)(stage * BLOCK_B + j * 1024), in_off[j], (uint32_t)nq0 * in_row);
    else load_to_lds_b32(rst, stat_at + (uint32_t)(stage * STAT_B), (uint32_t)L.lane * 4u, (uint32_t)nq0 * 4u);
  };
  auto issue_end = [&]() {
    nq0 += QB;
    to_load--;
    if (nq0 >= t.seg_len || to_load == 0) {
      if (nq0 >= t.seg_len) { nq0 = q_begin; nj++; }
      set_head();
    }
  };
  auto issue = [&](int stage) {
#pragma unroll
    for (int j = 0; j < PT; j++) issue_part(stage, j);
    issue_end();
  };

  // ---- lane parts of the LDS offsets; stage, block half and operand ride in the instructions' offset fields ----
  // rows: of the block that the score-like product reads; cols: of the block that the accumulating product reads
  uint32_t rows[NC], cols[NN];
#pragma unroll
  for (int c = 0; c < NC; c++) rows[c] = row_offset<HD>(L, c) + (second ? DO_AT : 0);
#pragma unroll
  for (int n = 0; n < NN; n++) cols[n] = col_offset<HD>(L, n) + (second ? 0 : DO_AT);
  const uint32_t p_at = P_AT + (uint32_t)(wave * 4096 + L.lane * 16), stat_rows = stat_off + 16u * L.g;
  const lds_cptr M = (lds_cptr)lds;
  const lds_ptr Mw = (lds_ptr)lds;

  // What phases 0 and 1 read of blocks -2 and -1 is zero: the last two stages of Q, the last of dO, the second slot of P.
  for (int i = tid * 16; i < 2 * BLOCK_B; i += 512 * 16) *(MLLM_LDS u32x4_t*)(Mw + (NQ - 2) * BLOCK_B + i) = u32x4_t{0, 0, 0, 0};
  *(MLLM_LDS u32x4_t*)(Mw + DO_AT + (NO - 1) * BLOCK_B + tid * 16) = u32x4_t{0, 0, 0, 0};
  for (int i = tid * 16; i < P_SLOT; i += 512 * 16) *(MLLM_LDS u32x4_t*)(Mw + P_AT + P_SLOT + i) = u32x4_t{0, 0, 0, 0};

  constexpr int RD = 4, CD = 4;   // fragments read ahead of their MFMAs
  Frag8 pb[2];            // P, or dS negated, of a block as MFMA operand, an own group each
#pragma unroll
  for (int j = 0; j < 2; j++)
#pragma unroll
    for (int w = 0; w < 4; w++) pb[j].w[w] = 0;
  bf16x8 fc[NN], fr[NS];   // transposed and natural-layout fragments
  auto read_cols = [&](int stage, int n) { fc[n] = read_col<HD>(M, cols[n] + (uint32_t)(stage * BLOCK_B)); };
  auto read_rows = [&](int stage, int x) { fr[x] = lds_b128(M, rows[x / 2] + (uint32_t)(stage * BLOCK_B + x % 2 * GROUP_B)); };
  auto accumulate = [&](int n) {
#pragma unroll
    for (int j = 0; j < 2; j++) acc[n][j] = mfma(fc[n], pb[j].v, acc[n][j]);
  };
  // elements 2x, 2x+1 of a block: row group i, own group j, rows e, e+1
  struct El { int i, j, e; };
  auto element = [](int v) { return El{v >> 3, (v >> 2) & 1, v & 3}; };

  const bool idle = wave_first_k >= t.seg_len;   // a wavefront without a key: only its share of the loads is wanted
  if (!second) {
    f32x4 s[2][2];          // scores of the block after the current one: [row group][own group]
    f32x4 xs[2][2];         // exponents of the current block
    auto scale_lse = [&](int stage) {   // the lse rows of a stage times log2(e), in place (they are this wavefront's own)
      const uint32_t at = stat_off + (uint32_t)(stage * STAT_B + 4 * L.lane);
      *(MLLM_LDS float*)(Mw + at) = *(MLLM_LDS const float*)(M + at) * LOG2E;
    };
    int q0 = range.q0;
#pragma unroll
    for (int st = 0; st < 4; st++) issue(st);
    wait_loads<3 * PT>();
    phase_barrier();
#pragma unroll
    for (int x = 0; x < NS; x++) {
      read_rows(0, x);
#pragma unroll
      for (int j = 0; j < 2; j++) s[x % 2][j] = mfma(fr[x], kvf[j][x / 2], x < 2 ? f32x4{0, 0, 0, 0} : s[x % 2][j]);
    }
    scale_lse(0);
#pragma unroll
    for (int n = 0; n < CD; n++) read_cols(NO - 1, n);
    auto phase = [&](auto Ut) {
      constexpr int U = decltype(Ut)::value;   // phase number modulo 8
      wait_loads<2 * PT>();
      phase_barrier();
      if (idle) return issue((U + 4) & 7);
      f32x4 ls[2];
      // dV of block n-1; exponents of block n; the first fragments of Q of block n+1; the loads of Q of block n+4
#pragma unroll
      for (int n = 0; n < NN; n++) {
        if (n + CD < NN) read_cols((U + 3) & 3, n + CD);
        else if (n - (NN - CD) < RD) read_rows((U + 1) & 7, n - (NN - CD));
        if (n < 2) ls[n] = lds_f4(M, stat_rows + (uint32_t)(U * STAT_B + 64 * n));
        if (n >= 1 && n - 1 < PT) issue_part((U + 4) & 7, n - 1);
        accumulate(n);
        if (n >= 2) {
#pragma unroll
          for (int v = (n - 2) * 16 / (NN - 2); v < (n - 1) * 16 / (NN - 2); v++) {
            const El x = element(v);
            xs[x.i][x.j][x.e] = fmaf(s[x.i][x.j][x.e], c2, -ls[x.i][x.e]);
          }
        }
        MLLM_SLOT_END;
      }
      issue_end();
      if (t.causal && q0 <= wave_first_k + 31) {   // the block touches the diagonal: masked pairs get probability zero
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const El x = element(v);
          xs[x.i][x.j][x.e] = (krow[x.j] <= q0 + 16 * x.i + 4 * L.g + x.e) ? xs[x.i][x.j][x.e] : -INFINITY;
        }
      }
      q0 += QB;
      if (q0 >= t.seg_len) q0 = q_begin;
      // S of block n+1; P of block n, written for the partner; the first fragments of dO of block n
      f32x4 pr;
      MLLM_SLOT_END;
#pragma unroll
      for (int x = 0; x < NS; x++) {
        if (x + RD < NS) read_rows((U + 1) & 7, x + RD);
        else read_cols(U & 3, x - (NS - RD));
        if (x == 1) scale_lse((U + 1) & 7);
#pragma unroll
        for (int j = 0; j < 2; j++) s[x % 2][j] = mfma(fr[x], kvf[j][x / 2], x < 2 ? f32x4{0, 0, 0, 0} : s[x % 2][j]);
        constexpr int SL = 6;   // slots that the 16 exponentials are spread over
#pragma unroll
        for (int v = x * 16 / SL; v < (x + 1) * 16 / SL && v < 16; v++) {
          const El y = element(v);
          pr[y.e] = fast_exp2(xs[y.i][y.j][y.e]);
          if (v & 1) pb[y.j].w[2 * y.i + (y.e >> 1)] = pack_bf16x2(pr[y.e - 1], pr[y.e]);
          if (y.e == 3) *(MLLM_LDS f32x4*)(Mw + p_at + (U & 1) * P_SLOT + (v >> 2) * 1024) = pr;
        }
        MLLM_SLOT_END;
      }
    };
    for (int n = 0;;) {
      phase(Int<0>{}); if (++n == n_it + 2) break;
      phase(Int<1>{}); if (++n == n_it + 2) break;
      phase(Int<2>{}); if (++n == n_it + 2) break;
      phase(Int<3>{}); if (++n == n_it + 2) break;
      phase(Int<4>{}); if (++n == n_it + 2) break;
      phase(Int<5>{}); if (++n == n_it + 2) break;
      phase(Int<6>{}); if (++n == n_it + 2) break;
      phase(Int<7>{}); if (++n == n_it + 2) break;
    }
  } else {
    f32x4 dp[2][2][2];      // delta - dP of even and odd blocks: [row group][own group]
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++) dp[0][i][j] = dp[1][i][j] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int st = 0; st < 2; st++) issue(st);
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int c = 0; c < NC; c++) kvf[j][c] = negated(kvf[j][c]);
    phase_barrier();
#pragma unroll
    for (int n = 0; n < CD; n++) read_cols(NQ - 2, n);
    auto phase = [&](auto Ut) {
      constexpr int U = decltype(Ut)::value;
      wait_loads<PT>();
      phase_barrier();
      if (idle) return issue((U + 2) & 3);
      f32x4 pq[4], de[2];
      // dK of block n-2; P of block n-1; delta and the first fragments of dO of block n; the loads of dO of block n+2
#pragma unroll
      for (int n = 0; n < NN; n++) {
        if (n + CD < NN) read_cols((U + 6) & 7, n + CD);
        else if (n - (NN - CD) < RD) read_rows(U & 3, n - (NN - CD));
        if (n < 4) pq[n] = lds_f4(M, p_at + (uint32_t)(((U + 1) & 1) * P_SLOT + n * 1024));
        else if (n < 6) de[n - 4] = lds_f4(M, stat_rows + (uint32_t)((U & 3) * STAT_B + 64 * (n - 4)));
        if (n >= 1 && n - 1 < PT) issue_part((U + 2) & 3, n - 1);
        accumulate(n);
        MLLM_SLOT_END;
      }
      issue_end();
      // dP of block n; dS of block n-1; the first fragments of Q of block n-1
      MLLM_SLOT_END;
#pragma unroll
      for (int x = 0; x < NS; x++) {
        if (x + RD < NS) read_rows(U & 3, x + RD);
        else read_cols((U + 7) & 7, x - (NS - RD));
#pragma unroll
        for (int j = 0; j < 2; j++) dp[U & 1][x % 2][j] = mfma(fr[x], kvf[j][x / 2], x < 2 ? de[x % 2] : dp[U & 1][x % 2][j]);
        const El y = element(2 * x);
        const f32x4& dc = dp[(U + 1) & 1][y.i][y.j];
        pb[y.j].w[2 * y.i + (y.e >> 1)] = pack_bf16x2(pq[x >> 1][y.e] * dc[y.e], pq[x >> 1][y.e + 1] * dc[y.e + 1]);
        MLLM_SLOT_END;
      }
    };
    for (int n = 0;;) {
      phase(Int<0>{}); if (++n == n_it + 2) break;
      phase(Int<1>{}); if (++n == n_it + 2) break;
      phase(Int<2>{}); if (++n == n_it + 2) break;
      phase(Int<3>{}); if (++n == n_it + 2) break;
      phase(Int<4>{}); if (++n == n_it + 2) break;
      phase(Int<5>{}); if (++n == n_it + 2) break;
      phase(Int<6>{}); if (++n == n_it + 2) break;
      phase(Int<7>{}); if (++n == n_it + 2) break;
    }
  }
  // the loads enqueued last (blocks past the end: zeros) must have landed before this workgroup's LDS
  // can be handed to another one
  wait_loads<0>();
#pragma unroll
  for (int j = 0; j < 2; j++) {
    if (krow[j] >= t.seg_len) continue;
    const int64_t row = t.seg_start + krow[j];
    if (second) store_dk<HD>(p, acc, j, krow[j], row, kvh, L.g, gridDim.y > 1, blockIdx.y);
    else store_dv<HD>(p, acc, j, row, kvh, L.g, gridDim.y > 1, blockIdx.y);
  }
}

// dK and dV from the parts' sums, added in their order; dK scaled and rotated back.  A thread takes eight
// columns of the left and of the right half of a row of one kv head.
__global__ __launch_bounds__(256) void attn_dkv_reduce_kernel(const float* __restrict__ partial, bf16_t* __restrict__ dk,
                                                              bf16_t* __restrict__ dv, int parts, int64_t T, int hkv, int hd,
                                                              int64_t kv_stride, float scale, const float* __restrict__ rope_table,
                                                              const int32_t* __restrict__ pos) {
  const int per_head = hd >> 4, half = hd >> 1;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int c0 = (int)(gid % per_head) * 8, head = (int)(gid / per_head % hkv);
  const int64_t row = gid / ((int64_t)per_head * hkv);
  if (row >= T) return;
  const int64_t width = (int64_t)hkv * hd, set = T * width;
  const float* src = partial + row * width + head * hd + c0;
  float s[2][2][8];   // [dK, dV][half][column]
#pragma unroll
  for (int w = 0; w < 2; w++)
#pragma unroll
    for (int x = 0; x < 2; x++)
#pragma unroll
      for (int e = 0; e < 8; e++) s[w][x][e] = 0.f;
#pragma unroll 2
  for (int p = 0; p < parts; p++)
#pragma unroll
    for (int w = 0; w < 2; w++)
#pragma unroll
      for (int x = 0; x < 2; x++) {
        const float4* f = reinterpret_cast<const float4*>(src + (2 * p + w) * set + x * half);
        const float4 a = f[0], b = f[1];
        s[w][x][0] += a.x; s[w][x][1] += a.y; s[w][x][2] += a.z; s[w][x][3] += a.w;
        s[w][x][4] += b.x; s[w][x][5] += b.y; s[w][x][6] += b.z; s[w][x][7] += b.w;
      }
  if (rope_table) {   // dx1 = dy1 cos + dy2 sin, dx2 = dy2 cos - dy1 sin
    const float* trow = rope_table + (int64_t)pos[row] * hd + c0;
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const float c = trow[e] * scale, sn = trow[half + e] * scale, y1 = s[0][0][e], y2 = s[0][1][e];
      s[0][0][e] = y1 * c + y2 * sn;
      s[0][1][e] = y2 * c - y1 * sn;
    }
  } else {
#pragma unroll
    for (int x = 0; x < 2; x++)
#pragma unroll
      for (int e = 0; e < 8; e++) s[0][x][e] *= scale;
  }
#pragma unroll
  for (int w = 0; w < 2; w++)
#pragma unroll
    for (int x = 0; x < 2; x++) {
      bf16_t* dst = (w ? dv : dk) + row * kv_stride + head * hd + c0 + x * half;
      const float* v = s[w][x];
      *reinterpret_cast<uint4*>(dst) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
    }
}

AttnParams make_params(const AttnArgs& a) {
  AttnParams p;
  p.q = (const bf16_t*)a.q; p.k = (const bf16_t*)a.k; p.v = (const bf16_t*)a.v;
  p.o = (bf16_t*)a.o; p.lse = a.lse; p.d_o = (const bf16_t*)a.d_o;
  p.dq = (bf16_t*)a.dq; p.dk = (bf16_t*)a.dk; p.dv = (bf16_t*)a.dv; p.delta = a.delta;
  p.q_stride = a.q_stride; p.kv_stride = a.kv_stride; p.o_stride = a.o_stride;
  p.T = a.total_tokens; p.Hq = a.n_q_heads; p.Hkv = a.n_kv_heads;
  p.list = nullptr;
  p.scale = 1.0f / sqrtf((float)a.head_dim);
  p.scale_log2e = p.scale * LOG2E;
  p.rope_table = a.rope_table;
  p.dkv_partial = a.dkv_partial;
  return p;
}

}  // namespace

// The kernels address K, V, Q and dO rows through 32-bit byte offsets from the segment start
// (buffer descriptors whose range ends at the last wanted row); a tile may run up to 255 rows
// past the end before the range check rejects it, so those offsets must not wrap either.
static bool offsets_fit(const AttnArgs& a) {
  const int64_t widest = std::max(a.q_stride, std::max(a.kv_stride, a.o_stride));
  return ((int64_t)a.total_tokens + 256) * widest * 2 < (int64_t)0xFFFFFFFFll;
}

// Whether a gradient is written over something that the passes read.  One launch for both passes may then write what the other
// pass still wants; one after the other, dk may take the place of k, dv that of v and dq that of o.  First to last element, so
// matrices that are only interleaved count as well: they are served in order, a little slower.
static bool gradients_over_inputs(const AttnArgs& a) {
  const auto bytes = [&](int64_t stride, int heads) { return ((a.total_tokens - 1) * stride + (int64_t)heads * a.head_dim) * 2; };
  const int64_t q = bytes(a.q_stride, a.n_q_heads), kv = bytes(a.kv_stride, a.n_kv_heads), o = bytes(a.o_stride, a.n_q_heads);
  const struct { const void* p; int64_t n; } out[3] = {{a.dq, q}, {a.dk, kv}, {a.dv, kv}}, in[5] = {{a.q, q}, {a.k, kv}, {a.v, kv}, {a.o, o}, {a.d_o, o}};
  for (const auto& w : out)
    for (const auto& r : in)
      if (ranges_overlap(w.p, w.n, r.p, r.n)) return true;
  return false;
}

hipError_t launch_attn_fwd(const AttnArgs& a, hipStream_t s) {
  if (a.q_grid == 0) return hipSuccess;
  if (!offsets_fit(a)) return hipErrorInvalidValue;
  ProfScope prof(PROF_ATTN_FWD, a.fwd_flops, s);
  AttnParams p = make_params(a);
  p.list = (const AttnItem*)a.q_list;
  const dim3 grid((unsigned)a.q_grid), block(256);
  if (a.head_dim == 128) hipLaunchKernelGGL(attn_fwd_kernel, grid, block, 0, s, p);
  else if (a.head_dim == 64) hipLaunchKernelGGL(attn_fwd_64_kernel, grid, block, 0, s, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

int attn_kv_parts(int64_t heaviest, int64_t total, int64_t rows, int head_dim) {
  const int64_t resident = head_dim == 64 ? 512 : 256;
  const double per_it = head_dim == 64 ? 1.1 : 2.2;
  int best = 1;
  double best_cost = 1e300;
  for (int parts = 1; parts <= 8 && (parts == 1 || heaviest / parts >= 4); parts++) {
    const double chain = (double)((heaviest + parts - 1) / parts), fill = (double)total / (double)resident;
    double cost = std::max(chain, fill) * per_it;
    if (parts > 1) cost += 6.0 + (double)rows * head_dim * 16.0 * parts / 4.0e6;   // fp32 dK and dV, written and read
    if (cost < 0.97 * best_cost) { best_cost = cost; best = parts; }
  }
  return best;
}

// Heads of 64: up to this many workgroups the dQ and the dK/dV pass share a launch.  The dK/dV pass then forms delta itself,
// some 6 % more instructions a query tile; for that neither waits for the other's last workgroups, and with few
// workgroups both run side by side.  Whole layers and stages, apart and together (us; workgroups): toy stage 495 and 469,
// one 576-token image (160) 218.6 and 207.8, five (800) 427 and 421, eight (1280) 662 and 653, 13 (2080) 874 and 868, 20 (3200)
// 1267 and 1265, 46 (7360) 2548 and 2571.  With more than four query heads a kv head a few long dK/dV workgroups set the time, and those
// of dQ beside them slow them down (causal, backward alone: 16 / 2 heads, 577 tokens 140 and 143, 2048 413 and 429, 4134 821 and
// 868; 28 / 4, 4134 775 and 790; with four, 16 / 4 454 and 450, 32 / 8 513 and 486), other than for a few tokens, where a launch
// counts for more (forward and backward of 16 / 2: 110 tokens 46.5 and 43.3, 342 47.6 and 43.9).
constexpr int64_t BOTH_MOST = 3072;
constexpr int BOTH_GROUP = 4, BOTH_FEW_TOKENS = 512;
hipError_t launch_attn_bwd(const AttnArgs& a, hipStream_t s) {
  if (a.q_grid == 0) return hipSuccess;
  if (!offsets_fit(a)) return hipErrorInvalidValue;
  const bool split = a.kv_parts > 1 && a.dkv_partial;
  if (split && a.rope_table && !a.pos) return hipErrorInvalidValue;
  ProfScope prof(PROF_ATTN_BWD, 2.0 * a.fwd_flops, s);
  AttnParams p = make_params(a);
  const dim3 block(256), qgrid((unsigned)a.q_grid), kgrid((unsigned)a.kv_grid, split ? (unsigned)a.kv_parts : 1u);
  // dQ first: it writes delta, which the dK/dV pass of a launch of its own reads
  if (a.head_dim == 128) {
    p.list = (const AttnItem*)a.q_list;
    hipLaunchKernelGGL(attn_bwd_dq_kernel<128>, qgrid, block, 0, s, p);
    p.list = (const AttnItem*)a.kv_list;
    hipLaunchKernelGGL(attn_bwd_dkv_duo_kernel, kgrid, dim3(512), 0, s, p);
  } else if (a.head_dim == 64 && a.q_grid + (int64_t)kgrid.x * kgrid.y <= BOTH_MOST && (a.n_q_heads <= BOTH_GROUP * a.n_kv_heads || a.total_tokens <= BOTH_FEW_TOKENS) &&
             !gradients_over_inputs(a)) {
    p.list = (const AttnItem*)a.q_list;
    hipLaunchKernelGGL(attn_bwd_both_kernel, dim3((unsigned)a.q_grid + kgrid.x * kgrid.y), block, 0, s, p, (const AttnItem*)a.kv_list,
                       (int)kgrid.x, (int)kgrid.y);
  } else if (a.head_dim == 64) {
    p.list = (const AttnItem*)a.q_list;
    hipLaunchKernelGGL(attn_bwd_dq_kernel<64>, qgrid, block, 0, s, p);
    p.list = (const AttnItem*)a.kv_list;
    hipLaunchKernelGGL(attn_bwd_dkv_kernel, kgrid, block, 0, s, p);
  } else {
    return hipErrorInvalidValue;
  }
  if (split) {
    const int64_t n = (int64_t)a.total_tokens * a.n_kv_heads * (a.head_dim / 16);
    hipLaunchKernelGGL(attn_dkv_reduce_kernel, dim3((unsigned)((n + 255) / 256)), block, 0, s, a.dkv_partial, (bf16_t*)a.dk, (bf16_t*)a.dv,
                       a.kv_parts, (int64_t)a.total_tokens, a.n_kv_heads, a.head_dim, a.kv_stride, p.scale, a.rope_table, a.pos);
  }
  return hipGetLastError();
}

}  // namespace mllm
