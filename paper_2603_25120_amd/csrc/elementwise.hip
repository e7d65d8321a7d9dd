// HBM-bound kernels of the stage: LayerNorm / RMSNorm forward and backward (one wavefront per
// row, wavefront reductions), rotary positions, GELU / SwiGLU forward and backward, bias-gradient
// column sums, row scatter / gather for the connector.  All math in fp32 on bf16 storage, 16-byte
// accesses, no atomics: every cross-row reduction is two deterministic stages.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace mllm {

namespace {

constexpr int ROWS_PER_BLOCK = 4;  // 4 wavefronts, one row each

__device__ __forceinline__ void unpack8(const uint4& u, float* f) {
  f[0] = bf16lo(u.x); f[1] = bf16hi(u.x); f[2] = bf16lo(u.y); f[3] = bf16hi(u.y);
  f[4] = bf16lo(u.z); f[5] = bf16hi(u.z); f[6] = bf16lo(u.w); f[7] = bf16hi(u.w);
}
__device__ __forceinline__ uint4 pack8(const float* f) {
  return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]),
                    pack_bf16x2(f[6], f[7]));
}

// ---------------------------------------------------------------------------------------------
// normalisation forward: y = (x - mean) * rstd * gamma + beta   (LayerNorm, KIND 0)
//                        y = x * rstd * gamma                   (RMSNorm,   KIND 1)
// NV = 16-byte vectors per lane; the row lives in registers between the passes.  Rows of x and y
// are ld elements apart (ld = d for a dense matrix, more for a column slice of a wider one).
// x_copy (may be null) receives x as well: the stage keeps its input for the backward pass, and a copy of its
// own would read it a second time (26496 x 1024: copy 20 us + norm 20 us).
// ---------------------------------------------------------------------------------------------
template <int KIND, int NV>
__global__ __launch_bounds__(256) void norm_fwd_kernel(const bf16_t* __restrict__ x,
                                                       const bf16_t* __restrict__ gamma,
                                                       const bf16_t* __restrict__ beta,
                                                       bf16_t* __restrict__ y, float* __restrict__ stats,
                                                       int64_t T, int d, int64_t ld, float eps,
                                                       bf16_t* __restrict__ x_copy) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * ROWS_PER_BLOCK + (threadIdx.x >> 6);
  if (row >= T) return;
  const int nvec = d >> 3;
  // The row, gamma and beta are requested before any of them is used (with load and use of a vector in one conditional block they came
  // one after the other: 576 x 1024 3.19 -> 2.93 us, 26496 x 1024 23.8 -> 22.7, 24000 x 1280 29.5 -> 25.6, 3000 x 3584 RMSNorm 12.5 -> 10.5).
  uint4 u[NV];
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = lane + 64 * j;
    u[j] = c < nvec ? *reinterpret_cast<const uint4*>(x + row * ld + 8 * c) : make_uint4(0, 0, 0, 0);
  }
  uint4 g4[NV], b4[NV];
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = lane + 64 * j;
    g4[j] = c < nvec ? *reinterpret_cast<const uint4*>(gamma + 8 * c) : make_uint4(0, 0, 0, 0);
    b4[j] = KIND == 0 && c < nvec ? *reinterpret_cast<const uint4*>(beta + 8 * c) : make_uint4(0, 0, 0, 0);
  }
  float v[NV][8];
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = lane + 64 * j;
    if (x_copy && c < nvec) *reinterpret_cast<uint4*>(x_copy + row * ld + 8 * c) = u[j];
    unpack8(u[j], v[j]);
#pragma unroll
    for (int e = 0; e < 8; e++) sum += v[j][e];
  }
  float mean = 0.f;
  if (KIND == 0) mean = wave_sum(sum) / (float)d;
  float sq = 0.f;
#pragma unroll
  for (int j = 0; j < NV; j++) {
    int c = lane + 64 * j;
    if (c < nvec) {
#pragma unroll
      for (int e = 0; e < 8; e++) {
        float t = v[j][e] - mean;
        sq += t * t;
      }
    }
  }
  const float rstd = rsqrtf(wave_sum(sq) / (float)d + eps);
  if (lane == 0) {
    stats[row] = rstd;
    stats[T + row] = mean;
  }
#pragma unroll
  for (int j = 0; j < NV; j++) {
    int c = lane + 64 * j;
    if (c < nvec) {
      float g[8], b[8], o[8];
      unpack8(g4[j], g);
      if (KIND == 0) unpack8(b4[j], b);
#pragma unroll
      for (int e = 0; e < 8; e++) {
        o[e] = (v[j][e] - mean) * rstd * g[e];
        if (KIND == 0) o[e] += b[e];
      }
      *reinterpret_cast<uint4*>(y + row * ld + 8 * c) = pack8(o);
    }
  }
}

// The other form for rows wider than 1024 (norm_fwd_row_form chooses): a workgroup owns a row, NV 16-byte vectors a thread.  With
// a wavefront a row, few rows leave most of the chip idle behind one wavefront's loads and stores, and many rows over 2048 wide do not
// keep enough loads in flight (us, in a layer: 5125 x 3200 LayerNorm 23.9 -> 19.1; alone: 32768 x 4096 RMSNorm 109 -> 91, LayerNorm
// 120 -> 97).
// RMSNorm: the row passes through LDS and every wavefront forms the sum of all of it by itself, in the order of norm_fwd_kernel, so that a
// row's statistics have the same bits as with a wavefront a row (sums of quarters 91.7 us at 32768 x 4096, this 94.1).
// LayerNorm, with two such sums, adds the quarters' (5125 x 3200 13.2 and 18.5 us; rstd's largest error against float64 1.41e-7 and
// 1.47e-7, at 32768 x 4096 1.42e-7 and 2.83e-7).
template <int KIND, int NV>
__global__ __launch_bounds__(256) void norm_fwd_row_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ gamma,
                                                           const bf16_t* __restrict__ beta, bf16_t* __restrict__ y,
                                                           float* __restrict__ stats, int64_t T, int d, int64_t ld, float eps,
                                                           bf16_t* __restrict__ x_copy) {
  __shared__ uint4 whole[KIND == 1 ? 256 * NV : 1];
  __shared__ float red[2][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (row >= T) return;
  const int nvec = d >> 3;
  uint4 u[NV], g4[NV], b4[NV];
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = tid + 256 * j;
    u[j] = g4[j] = b4[j] = make_uint4(0, 0, 0, 0);
    if (c < nvec) u[j] = *reinterpret_cast<const uint4*>(x + row * ld + 8 * c);
  }
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = tid + 256 * j;
    if (c < nvec) {
      g4[j] = *reinterpret_cast<const uint4*>(gamma + 8 * c);
      if (KIND == 0) b4[j] = *reinterpret_cast<const uint4*>(beta + 8 * c);
    }
  }
  float v[NV][8];
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = tid + 256 * j;
    if (KIND == 1) whole[c] = u[j];
    if (x_copy && c < nvec) *reinterpret_cast<uint4*>(x_copy + row * ld + 8 * c) = u[j];
    unpack8(u[j], v[j]);
  }
  float mean = 0.f, sq = 0.f, rstd;
  if (KIND == 1) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4 * NV; j++) {
      float w[8];
      unpack8(whole[lane + 64 * j], w);   // zeros beyond the row
#pragma unroll
      for (int e = 0; e < 8; e++) sq += w[e] * w[e];
    }
    rstd = rsqrtf(wave_sum(sq) / (float)d + eps);
  } else {
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++)
#pragma unroll
      for (int e = 0; e < 8; e++) sum += v[j][e];
    sum = wave_sum(sum);
    if (lane == 0) red[0][wave] = sum;
    __syncthreads();
    mean = (red[0][0] + red[0][1] + red[0][2] + red[0][3]) / (float)d;
#pragma unroll
    for (int j = 0; j < NV; j++)
      if (tid + 256 * j < nvec) {
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float t = v[j][e] - mean;
          sq += t * t;
        }
      }
    sq = wave_sum(sq);
    if (lane == 0) red[1][wave] = sq;
    __syncthreads();
    rstd = rsqrtf((red[1][0] + red[1][1] + red[1][2] + red[1][3]) / (float)d + eps);
  }
  if (tid == 0) {
    stats[row] = rstd;
    stats[T + row] = mean;
  }
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = tid + 256 * j;
    if (c < nvec) {
      float g[8], b[8], o[8];
      unpack8(g4[j], g);
      unpack8(b4[j], b);
#pragma unroll
      for (int e = 0; e < 8; e++) {
        o[e] = (v[j][e] - mean) * rstd * g[e];
        if (KIND == 0) o[e] += b[e];
      }
      *reinterpret_cast<uint4*>(y + row * ld + 8 * c) = pack8(o);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// normalisation backward.  With xhat = (x - mean) * rstd and dxh = dy * gamma:
//   LayerNorm: dx = (dxh - mean(dxh) - xhat * mean(dxh * xhat)) * rstd
//   RMSNorm:   dx = (dxh - xhat * mean(dxh * xhat)) * rstd
// plus the residual branch's gradient dres.  Rows of dy, x, dres and dx are ld elements apart.
// A workgroup of 256 threads owns one row at a time
// (rows b, b + B, ...); a thread keeps NV 16-byte vectors of the row and its own column sums of
// dy * xhat (and of dy) in registers; they go to partial[b][*] at the end.
// ---------------------------------------------------------------------------------------------
template <int KIND, int NV>
__global__ __launch_bounds__(256) void norm_bwd_kernel(
    const bf16_t* __restrict__ dy, const bf16_t* __restrict__ x, const bf16_t* __restrict__ gamma,
    const float* __restrict__ stats, const bf16_t* __restrict__ dres, bf16_t* __restrict__ dx,
    float* __restrict__ partial, int64_t T, int d, int64_t ld) {
  __shared__ float red[2][2][4];  // [row parity][which sum][wavefront]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int B = gridDim.x, b = blockIdx.x;
  const int nvec = d >> 3;
  float g[NV][8], dg[NV][8], db[NV][8];
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = tid + 256 * j;
    if (c < nvec) unpack8(*reinterpret_cast<const uint4*>(gamma + 8 * c), g[j]);
#pragma unroll
    for (int e = 0; e < 8; e++) { dg[j][e] = 0.f; db[j][e] = 0.f; if (c >= nvec) g[j][e] = 0.f; }
  }
  int parity = 0;
  uint4 xq[NV], dq[NV], rq[NV];
  float rstd_n = 0.f;
  auto fetch = [&](int64_t row) __attribute__((always_inline)) {   // AHEAD only: a row's operands, while the row before is worked on
    if (row >= T) return;
    rstd_n = stats[row];
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int c = tid + 256 * j;
      if (c < nvec) {
        xq[j] = *reinterpret_cast<const uint4*>(x + row * ld + 8 * c);
        dq[j] = *reinterpret_cast<const uint4*>(dy + row * ld + 8 * c);
        if (dres) rq[j] = *reinterpret_cast<const uint4*>(dres + row * ld + 8 * c);
      }
    }
  };
  // RMSNorm: one row ahead (777 x 4096 14.4 -> 10.8 us, 2999 x 3584 23.4 -> 18.6; 32768 x 4096 187 -> 191, of which
  // the second stage gives back 15).  LayerNorm's second set of sums takes the registers, so it loads each operand where it is
  // used (both stages: 32768 x 3200 126 us, all three loaded in front of the row's work 172; 32768 x 5120 280 and 428).
  constexpr bool AHEAD = KIND == 1;
  if constexpr (AHEAD) fetch(b);
  for (int64_t row = b; row < T; row += B, parity ^= 1) {
    const float rstd = AHEAD ? rstd_n : stats[row];
    const float mean = KIND == 0 ? stats[T + row] : 0.f;
    float xh[NV][8], dxh[NV][8];
    uint4 res[NV];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int c = tid + 256 * j;
      if (c < nvec) {
        float xv[8], dv[8];
        unpack8(AHEAD ? xq[j] : *reinterpret_cast<const uint4*>(x + row * ld + 8 * c), xv);
        unpack8(AHEAD ? dq[j] : *reinterpret_cast<const uint4*>(dy + row * ld + 8 * c), dv);
        if constexpr (AHEAD) res[j] = rq[j];
#pragma unroll
        for (int e = 0; e < 8; e++) {
          xh[j][e] = (xv[e] - mean) * rstd;
          dxh[j][e] = dv[e] * g[j][e];
          s1 += dxh[j][e];
          s2 += dxh[j][e] * xh[j][e];
          dg[j][e] += dv[e] * xh[j][e];
          db[j][e] += dv[e];
        }
      }
    }
    if constexpr (AHEAD) fetch(row + B);
    s2 = wave_sum(s2);
    if (KIND == 0) s1 = wave_sum(s1);
    if (lane == 0) { red[parity][0][wave] = s1; red[parity][1][wave] = s2; }
    __syncthreads();  // one barrier per row: the two parities alternate, so a slot is rewritten
                      // only after every wavefront has passed the barrier of the row in between
    const float m2 = (red[parity][1][0] + red[parity][1][1] + red[parity][1][2] + red[parity][1][3]) / (float)d;
    const float m1 = KIND == 0 ? (red[parity][0][0] + red[parity][0][1] + red[parity][0][2] + red[parity][0][3]) / (float)d : 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int c = tid + 256 * j;
      if (c < nvec) {
        float o[8], r[8];
        if (dres) unpack8(AHEAD ? res[j] : *reinterpret_cast<const uint4*>(dres + row * ld + 8 * c), r);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          o[e] = (dxh[j][e] - m1 - xh[j][e] * m2) * rstd;
          if (dres) o[e] += r[e];
        }
        *reinterpret_cast<uint4*>(dx + row * ld + 8 * c) = pack8(o);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = tid + 256 * j;
    if (c < nvec) {
      float* pg = partial + (int64_t)b * d + 8 * c;
      *reinterpret_cast<float4*>(pg) = make_float4(dg[j][0], dg[j][1], dg[j][2], dg[j][3]);
      *reinterpret_cast<float4*>(pg + 4) = make_float4(dg[j][4], dg[j][5], dg[j][6], dg[j][7]);
      if (KIND == 0) {
        float* pb = partial + (int64_t)(B + b) * d + 8 * c;
        *reinterpret_cast<float4*>(pb) = make_float4(db[j][0], db[j][1], db[j][2], db[j][3]);
        *reinterpret_cast<float4*>(pb + 4) = make_float4(db[j][4], db[j][5], db[j][6], db[j][7]);
      }
    }
  }
}

// out[c] (+)= sum_p partial[p][c], for every job of a list.  A workgroup owns 32 columns of one job: 32 row
// slices x 8 float4 column groups; slice s adds rows s, s+32, ... in order (eight loads in flight), then the
// slice sums are added pairwise (s with s+16, then s with s+8, ...): a fixed association, so the result is
// bitwise reproducible.  A row's 32 columns are a whole line of 128 bytes: with 8 columns a workgroup, neighbours on
// different XCDs each fetched it (8 sums of 320 to 1024 rows, 89 MB: 53 us, now
// 24; 1024 rows of 4096: 22.5 and 7.1).  With a quarter of the slices a slice has four times the rows, so the last few are requested
// four at a time too (94 rows of 1024, both stages of a column sum: 5.34 us one at a time, now 4.82; with 128 slices 5.03).
constexpr int RED_COLS = 32, RED_SLICES = 32;
// JOBS: room in the list, which travels as the kernel's argument.  A list of 32 costs each workgroup a walk over 32
// entries before it knows its job, 0.7 us of a launch of 2-5; one norm or bias (at most 3 jobs) takes the short form.
template <int JOBS>
struct ReduceList {
  const float* partial[JOBS];
  float* out[JOBS];
  int rows[JOBS], n[JOBS];
  unsigned first[JOBS];   // first workgroup of a job; past the list: never reached
};
template <int JOBS>
__global__ __launch_bounds__(256) void reduce_partials_kernel(ReduceList<JOBS> list, int accumulate) {
  __shared__ float4 part[RED_SLICES][RED_COLS / 4];
  int job = 0;
#pragma unroll
  for (int j = 1; j < JOBS; j++) job += blockIdx.x >= list.first[j] ? 1 : 0;
  const float* __restrict__ partial = list.partial[job];
  float* __restrict__ out = list.out[job];
  const int P = list.rows[job];
  const int64_t n = list.n[job];
  const int cg = threadIdx.x & 7, slice = threadIdx.x >> 3;
  const int64_t c = ((int64_t)(blockIdx.x - list.first[job]) * (RED_COLS / 4) + cg) * 4;
  const bool valid = c < n;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (valid) {
    const float* col = partial + c;
    int p = slice;
    for (; p + 7 * RED_SLICES < P; p += 8 * RED_SLICES) {
      float4 v[8];
#pragma unroll
      for (int q = 0; q < 8; q++) v[q] = *reinterpret_cast<const float4*>(col + (int64_t)(p + q * RED_SLICES) * n);
#pragma unroll
      for (int q = 0; q < 8; q += 4) {
        s.x += (v[q].x + v[q + 1].x) + (v[q + 2].x + v[q + 3].x); s.y += (v[q].y + v[q + 1].y) + (v[q + 2].y + v[q + 3].y);
        s.z += (v[q].z + v[q + 1].z) + (v[q + 2].z + v[q + 3].z); s.w += (v[q].w + v[q + 1].w) + (v[q + 2].w + v[q + 3].w);
      }
    }
#pragma unroll 1
    for (; p < P; p += 4 * RED_SLICES) {   // what is left, four rows requested together
      float4 v[4];
#pragma unroll
      for (int q = 0; q < 4; q++) {
        v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p + q * RED_SLICES < P) v[q] = *reinterpret_cast<const float4*>(col + (int64_t)(p + q * RED_SLICES) * n);
      }
#pragma unroll
      for (int q = 0; q < 4; q++) { s.x += v[q].x; s.y += v[q].y; s.z += v[q].z; s.w += v[q].w; }
    }
  }
  part[slice][cg] = s;
  __syncthreads();
#pragma unroll
  for (int half = RED_SLICES / 2; half >= 1; half >>= 1) {
    if (slice < half) {
      const float4 a = part[slice][cg], b = part[slice + half][cg];
      part[slice][cg] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
    }
    __syncthreads();
  }
  if (slice == 0 && valid) {
    float4 t = part[0][cg];
    float4* o = reinterpret_cast<float4*>(out + c);
    if (accumulate) {
      const float4 old = *o;
      t.x += old.x; t.y += old.y; t.z += old.z; t.w += old.w;
    }
    *o = t;
  }
}

// ---------------------------------------------------------------------------------------------
// rotary positions, in place, half-split pairs (i, i + hd/2); angle = pos * base^(-2i/hd).
// One thread: one token, eight consecutive i, all heads.  Angles in fp64 so that positions in
// the ten-thousands keep full fp32-accurate sines.
// ---------------------------------------------------------------------------------------------
__global__ void rope_kernel(bf16_t* __restrict__ qk, const int32_t* __restrict__ pos, int64_t T,
                            int64_t row_stride, int64_t col0, int n_heads, int hd, double log2_base,
                            int inverse) {
  const int per_tok = hd >> 4;  // threads per token
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t t = gid / per_tok;
  if (t >= T) return;
  const int i0 = (int)(gid % per_tok) * 8;
  const double p = (double)pos[t];
  float cs[8], sn[8];
#pragma unroll
  for (int e = 0; e < 8; e++) {
    double inv = exp2(-2.0 * (double)(i0 + e) / (double)hd * log2_base);
    double s, c;
    sincos(p * inv, &s, &c);
    cs[e] = (float)c;
    sn[e] = inverse ? -(float)s : (float)s;
  }
  bf16_t* base = qk + t * row_stride + col0 + i0;
  const int half = hd >> 1;
  for (int h = 0; h < n_heads; h++) {
    bf16_t* p1 = base + h * hd;
    float a[8], b[8], oa[8], ob[8];
    unpack8(*reinterpret_cast<const uint4*>(p1), a);
    unpack8(*reinterpret_cast<const uint4*>(p1 + half), b);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      oa[e] = a[e] * cs[e] - b[e] * sn[e];
      ob[e] = b[e] * cs[e] + a[e] * sn[e];
    }
    *reinterpret_cast<uint4*>(p1) = pack8(oa);
    *reinterpret_cast<uint4*>(p1 + half) = pack8(ob);
  }
}

// Table of the rotary angles for the kernels that rotate in their own epilogue: row `pos` holds
// cos(pos * base^(-2i/hd)) for i < hd/2, then the sines (fp32; angles and sincos in fp64, as in
// rope_kernel, so both forms of the rotation use the same factors).
__device__ __forceinline__ void rope_table_entry(float* __restrict__ table, int64_t n_pos, int hd, double log2_base, int64_t gid) {
  const int half = hd >> 1;
  if (gid >= n_pos * half) return;
  const int64_t pos = gid / half;
  const int i = (int)(gid % half);
  const double inv = exp2(-2.0 * (double)i / (double)hd * log2_base);
  double sn, cs;
  sincos((double)pos * inv, &sn, &cs);
  table[pos * hd + i] = (float)cs;
  table[pos * hd + half + i] = (float)sn;
}
__global__ void rope_table_kernel(float* __restrict__ table, int64_t n_pos, int hd, double log2_base) {
  rope_table_entry(table, n_pos, hd, log2_base, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}
// The beginning of a stage's pass (launch_begin): workgroups of the metadata, then of each table, then of the copied rows.  A
// launch of its own for each cost 4 us of a small stage's pass, of which 1.5 to 2.5 are the kernel: launches are what bounds it.
struct BeginArgs {
  const uint4* meta_src; uint4* meta; int64_t meta_vec;
  struct { float* table; double log2_base; int hd; int first; } table[BEGIN_TABLES];   // first workgroup of each
  int64_t n_pos;
  const uint4* copy_src; uint4* copy_dst; int64_t copy_vec;
  int n_tables, copy_first;
};
__global__ __launch_bounds__(256) void begin_kernel(BeginArgs a) {
  const int b = blockIdx.x;
  if (b >= a.copy_first) {
    const int64_t i = (int64_t)(b - a.copy_first) * 256 + threadIdx.x;
    if (i < a.copy_vec) a.copy_dst[i] = a.copy_src[i];
    return;
  }
  for (int t = a.n_tables - 1; t >= 0; t--)
    if (b >= a.table[t].first) {
      rope_table_entry(a.table[t].table, a.n_pos, a.table[t].hd, a.table[t].log2_base, (int64_t)(b - a.table[t].first) * 256 + threadIdx.x);
      return;
    }
  const int64_t i = (int64_t)b * 256 + threadIdx.x;
  if (i < a.meta_vec) a.meta[i] = a.meta_src[i];
}

// The same rotation from the table (forward only): a thread takes eight pairs of one head of one token, so that a
// small microbatch still fills the chip (777 tokens, 40 heads of 128: rope_kernel 25 us on 25 workgroups that each
// form their angles in fp64, this one 4 us).
__global__ __launch_bounds__(256) void rope_from_table_kernel(bf16_t* __restrict__ qk, const int32_t* __restrict__ pos,
                                                              const float* __restrict__ table, int64_t T, int64_t row_stride,
                                                              int n_heads, int hd) {
  const int per_head = hd >> 4;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int i0 = (int)(gid % per_head) * 8, h = (int)(gid / per_head % n_heads), half = hd >> 1;
  const int64_t t = gid / ((int64_t)per_head * n_heads);
  if (t >= T) return;
  const float* trow = table + (int64_t)pos[t] * hd + i0;
  bf16_t* p1 = qk + t * row_stride + (int64_t)h * hd + i0;
  float a[8], b[8], oa[8], ob[8];
  unpack8(*reinterpret_cast<const uint4*>(p1), a);
  unpack8(*reinterpret_cast<const uint4*>(p1 + half), b);
#pragma unroll
  for (int q = 0; q < 2; q++) {
    const float4 c = *reinterpret_cast<const float4*>(trow + 4 * q), s = *reinterpret_cast<const float4*>(trow + half + 4 * q);
    const float cs[4] = {c.x, c.y, c.z, c.w}, sn[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
    for (int e = 0; e < 4; e++) {
      oa[4 * q + e] = a[4 * q + e] * cs[e] - b[4 * q + e] * sn[e];
      ob[4 * q + e] = b[4 * q + e] * cs[e] + a[4 * q + e] * sn[e];
    }
  }
  *reinterpret_cast<uint4*>(p1) = pack8(oa);
  *reinterpret_cast<uint4*>(p1 + half) = pack8(ob);
}

// ---------------------------------------------------------------------------------------------
// activations
// ---------------------------------------------------------------------------------------------
__global__ void gelu_fwd_kernel(int act, const bf16_t* __restrict__ h, bf16_t* __restrict__ a, int64_t nvec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvec) return;
  float z[8], o[8];
  unpack8(reinterpret_cast<const uint4*>(h)[i], z);
#pragma unroll
  for (int e = 0; e < 8; e++) o[e] = gelu_f(act, z[e]);
  reinterpret_cast<uint4*>(a)[i] = pack8(o);
}
__global__ void gelu_bwd_kernel(int act, const bf16_t* __restrict__ da, const bf16_t* __restrict__ h,
                                bf16_t* __restrict__ dh, int64_t nvec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvec) return;
  float z[8], g[8], o[8];
  unpack8(reinterpret_cast<const uint4*>(h)[i], z);
  unpack8(reinterpret_cast<const uint4*>(da)[i], g);
#pragma unroll
  for (int e = 0; e < 8; e++) o[e] = g[e] * gelu_grad_f(act, z[e]);
  reinterpret_cast<uint4*>(dh)[i] = pack8(o);
}
// The same with the column sums of dh (the gradient of the bias in front of the activation) formed
// on the way: workgroup (bx, by) owns columns [512 bx, 512 bx + 512) and rows by*4 + wave + k*4*gridDim.y;
// a lane keeps eight columns, the four wavefronts' sums are added through LDS in a fixed order and
// land in row by of `partial` ([gridDim.y, f] fp32), which reduce_partials_kernel then sums.
// da and dh may be the same buffer (a lane reads its eight values of a row before it writes them).
__global__ __launch_bounds__(256) void gelu_bwd_colsum_kernel(int act, const bf16_t* da,
                                                              const bf16_t* __restrict__ h, bf16_t* dh,
                                                              float* __restrict__ partial, int64_t T, int64_t f) {
  __shared__ float red[3][64][8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c = ((int64_t)blockIdx.x * 64 + lane) * 8;
  const bool valid = c < f;
  const int64_t step = (int64_t)gridDim.y * 4;
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (valid) {
    int64_t r = (int64_t)blockIdx.y * 4 + wave;
    uint4 zq, gq;
    if (r < T) { zq = *reinterpret_cast<const uint4*>(h + r * f + c); gq = *reinterpret_cast<const uint4*>(da + r * f + c); }
    for (; r < T; r += step) {
      float z[8], g[8], o[8];
      unpack8(zq, z);
      unpack8(gq, g);
      if (r + step < T) {   // the next row's loads go out before this row's arithmetic
        zq = *reinterpret_cast<const uint4*>(h + (r + step) * f + c);
        gq = *reinterpret_cast<const uint4*>(da + (r + step) * f + c);
      }
#pragma unroll
      for (int e = 0; e < 8; e++) { o[e] = g[e] * gelu_grad_f(act, z[e]); s[e] += o[e]; }
      *reinterpret_cast<uint4*>(dh + r * f + c) = pack8(o);
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int e = 0; e < 8; e++) red[wave - 1][lane][e] = s[e];
  }
  __syncthreads();
  if (wave == 0 && valid) {
#pragma unroll
    for (int e = 0; e < 8; e++) s[e] = (s[e] + red[0][lane][e]) + (red[1][lane][e] + red[2][lane][e]);
    float* p = partial + (int64_t)blockIdx.y * f + c;
    *reinterpret_cast<float4*>(p) = make_float4(s[0], s[1], s[2], s[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(s[4], s[5], s[6], s[7]);
  }
}
// gu = [g | u], [T, 2f];  a = g * sigmoid(g) * u
__global__ void swiglu_fwd_kernel(const bf16_t* __restrict__ gu, bf16_t* __restrict__ a, int64_t T, int64_t f) {
  const int64_t vec_per_row = f >> 3;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T * vec_per_row) return;
  const int64_t t = i / vec_per_row, c = (i % vec_per_row) * 8;
  float g[8], u[8], o[8];
  unpack8(*reinterpret_cast<const uint4*>(gu + t * 2 * f + c), g);
  unpack8(*reinterpret_cast<const uint4*>(gu + t * 2 * f + f + c), u);
#pragma unroll
  for (int e = 0; e < 8; e++) o[e] = g[e] / (1.f + expf(-g[e])) * u[e];
  *reinterpret_cast<uint4*>(a + t * f + c) = pack8(o);
}
__global__ void swiglu_bwd_kernel(const bf16_t* __restrict__ da, const bf16_t* __restrict__ gu,
                                  bf16_t* __restrict__ dgu, int64_t T, int64_t f) {
  const int64_t vec_per_row = f >> 3;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T * vec_per_row) return;
  const int64_t t = i / vec_per_row, c = (i % vec_per_row) * 8;
  float g[8], u[8], d[8], og[8], ou[8];
  unpack8(*reinterpret_cast<const uint4*>(gu + t * 2 * f + c), g);
  unpack8(*reinterpret_cast<const uint4*>(gu + t * 2 * f + f + c), u);
  unpack8(*reinterpret_cast<const uint4*>(da + t * f + c), d);
#pragma unroll
  for (int e = 0; e < 8; e++) {
    float s = 1.f / (1.f + expf(-g[e]));
    og[e] = d[e] * u[e] * (s + g[e] * s * (1.f - s));
    ou[e] = d[e] * g[e] * s;
  }
  *reinterpret_cast<uint4*>(dgu + t * 2 * f + c) = pack8(og);
  *reinterpret_cast<uint4*>(dgu + t * 2 * f + f + c) = pack8(ou);
}

// ---------------------------------------------------------------------------------------------
// column sums (bias gradients), stage 1: a workgroup owns 512 columns (8 per lane) and row chunk
// blockIdx.y; its four wavefronts take every fourth row of the chunk, four loads in flight each,
// and their sums are added through LDS in a fixed order.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void colsum_partial_kernel(const bf16_t* __restrict__ x, int64_t ldx,
                                                             float* __restrict__ partial, int64_t T,
                                                             int64_t n) {
  __shared__ float red[3][64][8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c = ((int64_t)blockIdx.x * 64 + lane) * 8;
  const bool valid = c < n;
  const int64_t step = (int64_t)gridDim.y * 4;
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (valid) {
    const bf16_t* col = x + c;
    int64_t r = (int64_t)blockIdx.y * 4 + wave;
    for (; r + 3 * step < T; r += 4 * step) {
      const uint4 u0 = *reinterpret_cast<const uint4*>(col + r * ldx);
      const uint4 u1 = *reinterpret_cast<const uint4*>(col + (r + step) * ldx);
      const uint4 u2 = *reinterpret_cast<const uint4*>(col + (r + 2 * step) * ldx);
      const uint4 u3 = *reinterpret_cast<const uint4*>(col + (r + 3 * step) * ldx);
      float v0[8], v1[8], v2[8], v3[8];
      unpack8(u0, v0); unpack8(u1, v1); unpack8(u2, v2); unpack8(u3, v3);
#pragma unroll
      for (int e = 0; e < 8; e++) s[e] += (v0[e] + v1[e]) + (v2[e] + v3[e]);
    }
    for (; r < T; r += step) {
      float v[8];
      unpack8(*reinterpret_cast<const uint4*>(col + r * ldx), v);
#pragma unroll
      for (int e = 0; e < 8; e++) s[e] += v[e];
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int e = 0; e < 8; e++) red[wave - 1][lane][e] = s[e];
  }
  __syncthreads();
  if (wave == 0 && valid) {
#pragma unroll
    for (int e = 0; e < 8; e++) s[e] = (s[e] + red[0][lane][e]) + (red[1][lane][e] + red[2][lane][e]);
    float* p = partial + (int64_t)blockIdx.y * n + c;
    *reinterpret_cast<float4*>(p) = make_float4(s[0], s[1], s[2], s[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(s[4], s[5], s[6], s[7]);
  }
}

__global__ void scatter_rows_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst,
                                    const int32_t* __restrict__ rows, int64_t n_rows, int64_t vec_per_row,
                                    int gather) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_rows * vec_per_row) return;
  const int64_t r = i / vec_per_row, c = i % vec_per_row;
  const int64_t other = rows[r];
  if (gather) reinterpret_cast<uint4*>(dst)[r * vec_per_row + c] = reinterpret_cast<const uint4*>(src)[other * vec_per_row + c];
  else reinterpret_cast<uint4*>(dst)[other * vec_per_row + c] = reinterpret_cast<const uint4*>(src)[r * vec_per_row + c];
}
// Average pooling at the end of the encoder (Evaluation, audio modality) and its gradient.
__global__ void pool_rows_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst,
                                 const int32_t* __restrict__ first, const int32_t* __restrict__ count,
                                 int64_t n_out, int64_t vec_per_row) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_out * vec_per_row) return;
  const int64_t j = i / vec_per_row, c = i % vec_per_row;
  const int64_t r0 = first[j];
  const int n = count[j];
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int r = 0; r < n; r++) {
    float v[8];
    unpack8(reinterpret_cast<const uint4*>(src)[(r0 + r) * vec_per_row + c], v);
#pragma unroll
    for (int e = 0; e < 8; e++) acc[e] += v[e];
  }
  const float inv = 1.f / (float)n;
#pragma unroll
  for (int e = 0; e < 8; e++) acc[e] *= inv;
  reinterpret_cast<uint4*>(dst)[j * vec_per_row + c] = pack8(acc);
}
__global__ void unpool_rows_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst,
                                   const int32_t* __restrict__ window, const int32_t* __restrict__ count,
                                   int64_t n_rows, int64_t vec_per_row) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_rows * vec_per_row) return;
  const int64_t r = i / vec_per_row, c = i % vec_per_row;
  const int64_t j = window[r];
  float v[8];
  unpack8(reinterpret_cast<const uint4*>(src)[j * vec_per_row + c], v);
  const float inv = 1.f / (float)count[j];
#pragma unroll
  for (int e = 0; e < 8; e++) v[e] *= inv;
  reinterpret_cast<uint4*>(dst)[r * vec_per_row + c] = pack8(v);
}
// Gradient of the connector's scatter (launch_connector_grad).  The workgroups of the scattered rows take a row's gradient and
// leave zeros in its place, both in one thread, so that dx_seq may be dy; the others copy the rows in between.
__global__ __launch_bounds__(256) void connector_grad_kernel(const uint4* dy, uint4* __restrict__ dproj, uint4* dx_seq, const int32_t* __restrict__ rows,
                                                             const uint32_t* __restrict__ scattered, int64_t n_rows, int64_t n_seq, int64_t vec_per_row,
                                                             int copy_first) {
  const int b = blockIdx.x;
  if (b < copy_first) {
    const int64_t i = (int64_t)b * 256 + threadIdx.x;
    if (i >= n_rows * vec_per_row) return;
    const int64_t at = (int64_t)rows[i / vec_per_row] * vec_per_row + i % vec_per_row;
    dproj[i] = dy[at];
    dx_seq[at] = make_uint4(0, 0, 0, 0);
    return;
  }
  const int64_t i = (int64_t)(b - copy_first) * 256 + threadIdx.x;
  if (i >= n_seq * vec_per_row) return;
  const int64_t r = i / vec_per_row;
  if (!((scattered[r >> 5] >> (r & 31)) & 1)) dx_seq[i] = dy[i];
}
// Sum of the partial products of a split K loop, in their order, four of their loads in flight at a time; then
// the epilogue terms of the product.  A thread takes eight consecutive columns of a row.
template <bool OUT_F32>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float4* __restrict__ partial, void* __restrict__ c, int splits,
                                                            int64_t nvec, int64_t vec_per_row, int accumulate,
                                                            const bf16_t* __restrict__ bias, const bf16_t* __restrict__ residual,
                                                            int64_t ldres) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvec) return;
  const int64_t row = i / vec_per_row, col = (i % vec_per_row) * 8;
  float t[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  auto add = [&](const float4& a, const float4& b) {
    t[0] += a.x; t[1] += a.y; t[2] += a.z; t[3] += a.w; t[4] += b.x; t[5] += b.y; t[6] += b.z; t[7] += b.w;
  };
  const float4* src = partial + 2 * i;
  const int64_t step = 2 * nvec;
  int sp = 0;
  for (; sp + 3 < splits; sp += 4) {
    float4 a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; q++) { a[q] = src[(sp + q) * step]; b[q] = src[(sp + q) * step + 1]; }
#pragma unroll
    for (int q = 0; q < 4; q++) add(a[q], b[q]);
  }
  for (; sp < splits; sp++) add(src[sp * step], src[sp * step + 1]);
  if (bias) {
    float v[8];
    unpack8(*reinterpret_cast<const uint4*>(bias + col), v);
#pragma unroll
    for (int e = 0; e < 8; e++) t[e] += v[e];
  }
  if constexpr (OUT_F32) {
    float4* o = reinterpret_cast<float4*>(c) + 2 * i;
    if (accumulate) add(o[0], o[1]);
    o[0] = make_float4(t[0], t[1], t[2], t[3]);
    o[1] = make_float4(t[4], t[5], t[6], t[7]);
  } else {
    if (residual) {
      float v[8];
      unpack8(*reinterpret_cast<const uint4*>(residual + row * ldres + col), v);
#pragma unroll
      for (int e = 0; e < 8; e++) t[e] += v[e];
    }
    reinterpret_cast<uint4*>(c)[i] = pack8(t);
  }
}
__global__ void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t nvec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nvec) dst[i] = src[i];
}

inline unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// Whether a workgroup owns a row (norm_fwd_row_kernel) or a wavefront does (us with a wavefront a row and a workgroup a row, rows
// from memory).  Up to 2048 columns the workgroup's threads have a vector each at most, and many rows are better off with more loads in
// flight a thread: 400 x 1280 LayerNorm 3.18 and 3.02, 1500 x 1280 4.32 and 4.29, 2048 x 1280 4.89 and 4.95, 2999 x 1280 5.72 and 6.39,
// 32768 x 1280 32.8 and 46, 32768 x 2048 48 and 55.  Wider rows always gain in LayerNorm (32768 x 4096 120 and 97); in RMSNorm not
// between 3/4 d rows and the 3072 (five vectors a lane and fewer: 5120) that a wavefront a row has resident at once: 600 x 4096 4.56 and 4.58,
// 2999 x 2560 7.5 and 8.4, 3072 x 4096 12.4 and 12.8, 3800 x 2560 10.2 and 11.3, 3300 x 3584 12.9 and 12.3, 4200 x 3072 13.9 and 13.3,
// 6000 x 3072 17.3 and 16.8.
static bool norm_fwd_row_form(int kind, int64_t t, int64_t d) {
  if (d <= 1024) return false;
  if (d <= 2048) return t <= 1536;
  return kind == 0 || d > 4096 || 4 * t <= 3 * d || t > (d > 2560 ? 3072 : 5120);
}
// A grid's x dimension holds fewer than 2^32 threads, 2^24 rows of the row form: beyond this many they go to y.
constexpr int64_t ROW_FORM_GRID = (int64_t)1 << 20;

hipError_t launch_norm_fwd(int kind, const void* x, const void* gamma, const void* beta, void* y,
                           float* stats, int64_t t, int64_t d, int64_t ld, float eps, hipStream_t s, void* x_copy) {
  if (t == 0) return hipSuccess;
  if (d % 8 != 0 || d > 8192 || ld < d || ld % 8 != 0) return hipErrorInvalidValue;
  ProfScope prof(PROF_ELEMENTWISE, (x_copy ? 6.0 : 4.0) * (double)t * (double)d, s);
  const int64_t nvec = d / 8;
  const bool row = norm_fwd_row_form(kind, t, d);
  const dim3 grid = row ? dim3((unsigned)std::min(t, ROW_FORM_GRID), (unsigned)((t + ROW_FORM_GRID - 1) / ROW_FORM_GRID))
                        : dim3(blocks_for(t, ROWS_PER_BLOCK)), block(256);
#define CALL(K, NV)                                                                                  \
  if (kind == 0) hipLaunchKernelGGL((K<0, NV>), grid, block, 0, s, (const bf16_t*)x, (const bf16_t*)gamma, \
      (const bf16_t*)beta, (bf16_t*)y, stats, t, (int)d, ld, eps, (bf16_t*)x_copy);                     \
  else hipLaunchKernelGGL((K<1, NV>), grid, block, 0, s, (const bf16_t*)x, (const bf16_t*)gamma,       \
      (const bf16_t*)beta, (bf16_t*)y, stats, t, (int)d, ld, eps, (bf16_t*)x_copy);
  if (nvec <= 64) { CALL(norm_fwd_kernel, 1) }
  else if (nvec <= 128) { CALL(norm_fwd_kernel, 2) }
  else if (nvec <= 256) { if (row) { CALL(norm_fwd_row_kernel, 1) } else { CALL(norm_fwd_kernel, 4) } }
  else if (nvec <= 512) {
    if (row) { CALL(norm_fwd_row_kernel, 2) }
    else { hipLaunchKernelGGL((norm_fwd_kernel<1, 8>), grid, block, 0, s, (const bf16_t*)x, (const bf16_t*)gamma, (const bf16_t*)beta,
                              (bf16_t*)y, stats, t, (int)d, ld, eps, (bf16_t*)x_copy); }
  }
  else { CALL(norm_fwd_row_kernel, 4) }
#undef CALL
  return hipGetLastError();
}

// Narrow rows (d <= 1024): a wavefront owns a row, so there is no barrier per row and all 256
// threads have data; the four wavefronts' column sums are added through LDS once at the end.
// CS: the column sums of dx (as computed, before rounding to bf16) come out as a third set of
// partial sums: dx is the gradient of a linear map's output whenever the layer below or the
// attention block above the norm ends in one, and those sums are that map's bias gradient.
template <int KIND, int NV, bool CS>
__global__ __launch_bounds__(256, 3) void norm_bwd_wave_kernel(
    const bf16_t* __restrict__ dy, const bf16_t* __restrict__ x, const bf16_t* __restrict__ gamma,
    const float* __restrict__ stats, const bf16_t* __restrict__ dres, bf16_t* __restrict__ dx,
    float* __restrict__ partial, int64_t T, int d, int64_t ld) {
  __shared__ float red[CS ? 3 : 2][4][1024];  // [d gamma | d beta | column sums of dx][wavefront][column]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int B = gridDim.x, b = blockIdx.x;
  const int nvec = d >> 3;
  float g[NV][8], dg[NV][8], db[NV][8], dc[CS ? NV : 1][8];
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = lane + 64 * j;
    if (c < nvec) unpack8(*reinterpret_cast<const uint4*>(gamma + 8 * c), g[j]);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      dg[j][e] = 0.f; db[j][e] = 0.f; if (c >= nvec) g[j][e] = 0.f;
      if (CS) dc[j][e] = 0.f;
    }
  }
  // The next row's loads are issued before this row's arithmetic: two rows in flight per wavefront.
  uint4 nx[NV], ndy[NV], nres[NV];
  auto fetch = [&](int64_t row) {
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int c = lane + 64 * j;
      if (c < nvec) {
        nx[j] = *reinterpret_cast<const uint4*>(x + row * ld + 8 * c);
        ndy[j] = *reinterpret_cast<const uint4*>(dy + row * ld + 8 * c);
        if (dres) nres[j] = *reinterpret_cast<const uint4*>(dres + row * ld + 8 * c);
      }
    }
  };
  const int64_t row0 = (int64_t)b * 4 + wave, row_step = (int64_t)4 * B;
  if (row0 < T) fetch(row0);
  for (int64_t row = row0; row < T; row += row_step) {
    const float rstd = stats[row];
    const float mean = KIND == 0 ? stats[T + row] : 0.f;
    float xh[NV][8], dxh[NV][8], r[NV][8];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int c = lane + 64 * j;
#pragma unroll
      for (int e = 0; e < 8; e++) { xh[j][e] = 0.f; dxh[j][e] = 0.f; r[j][e] = 0.f; }
      if (c < nvec) {
        float xv[8], dv[8];
        unpack8(nx[j], xv);
        unpack8(ndy[j], dv);
        if (dres) unpack8(nres[j], r[j]);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          xh[j][e] = (xv[e] - mean) * rstd;
          dxh[j][e] = dv[e] * g[j][e];
          s1 += dxh[j][e];
          s2 += dxh[j][e] * xh[j][e];
          dg[j][e] += dv[e] * xh[j][e];
          db[j][e] += dv[e];
        }
      }
    }
    if (row + row_step < T) fetch(row + row_step);
    const float m2 = wave_sum(s2) / (float)d;
    const float m1 = KIND == 0 ? wave_sum(s1) / (float)d : 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int c = lane + 64 * j;
      if (c < nvec) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
          o[e] = (dxh[j][e] - m1 - xh[j][e] * m2) * rstd + r[j][e];
          if (CS) dc[j][e] += o[e];
        }
        *reinterpret_cast<uint4*>(dx + row * ld + 8 * c) = pack8(o);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int c = lane + 64 * j;
    if (c < nvec) {
#pragma unroll
      for (int e = 0; e < 8; e++) {
        red[0][wave][8 * c + e] = dg[j][e];
        red[1][wave][8 * c + e] = db[j][e];
        if (CS) red[2][wave][8 * c + e] = dc[j][e];
      }
    }
  }
  __syncthreads();
  for (int col = tid; col < d; col += 256) {
    partial[(int64_t)b * d + col] = (red[0][0][col] + red[0][1][col]) + (red[0][2][col] + red[0][3][col]);
    if (KIND == 0)
      partial[(int64_t)(B + b) * d + col] = (red[1][0][col] + red[1][1][col]) + (red[1][2][col] + red[1][3][col]);
    if (CS)
      partial[(int64_t)(2 * B + b) * d + col] = (red[2][0][col] + red[2][1][col]) + (red[2][2][col] + red[2][3][col]);
  }
}

bool norm_bwd_colsum_fusable(int64_t d) { return d % 8 == 0 && d / 8 <= 128; }

int64_t norm_bwd_partial_rows(int64_t t) {
  return t < 1 ? 1 : (t > 1024 ? 1024 : t);
}

hipError_t PartialSums::take(int64_t rows, int64_t n, std::initializer_list<float*> outs, hipStream_t s, float** partial) {
  const size_t need = (size_t)rows * (size_t)n * outs.size();
  bool full = used + need > capacity || count + (int)outs.size() > MAX_JOBS;
  for (float* out : outs)
    for (int j = 0; out && j < count; j++) full = full || (out < jobs[j].out + jobs[j].n && jobs[j].out < out + n);
  if (full) {
    hipError_t e = flush(s);
    if (e != hipSuccess) return e;
  }
  if (need > capacity || (int)outs.size() > MAX_JOBS) return hipErrorInvalidValue;
  float* p = base + used;
  *partial = p;
  used += need;
  for (float* out : outs) {
    if (out) jobs[count++] = {p, out, (int)rows, n};
    p += rows * n;
  }
  return hipSuccess;
}

namespace {
template <int JOBS>
hipError_t launch_reduce(const PartialSums::Job* jobs, int count, int accumulate, hipStream_t s) {
  ReduceList<JOBS> list;
  unsigned blocks = 0;
  for (int j = 0; j < JOBS; j++) {
    const bool there = j < count;
    list.partial[j] = there ? jobs[j].partial : nullptr;
    list.out[j] = there ? jobs[j].out : nullptr;
    list.rows[j] = there ? jobs[j].rows : 0;
    list.n[j] = there ? (int)jobs[j].n : 0;
    list.first[j] = there ? blocks : ~0u;
    if (there) blocks += blocks_for(jobs[j].n, RED_COLS);
  }
  if (blocks == 0) return hipSuccess;
  ProfScope prof(PROF_ELEMENTWISE, 0.0, s);   // the bytes of a sum are counted with its first stage
  hipLaunchKernelGGL(reduce_partials_kernel<JOBS>, dim3(blocks), dim3(256), 0, s, list, accumulate);
  return hipGetLastError();
}
}  // namespace

hipError_t PartialSums::flush(hipStream_t s) {
  const int waiting = count;
  count = 0;
  used = 0;
  return waiting <= 3 ? launch_reduce<3>(jobs, waiting, accumulate, s) : launch_reduce<MAX_JOBS>(jobs, waiting, accumulate, s);
}

// Workgroups (= rows of partial sums) of the norm backward, at most.  The wavefront-per-row kernel with two vectors per lane
// keeps three workgroups per CU resident: a grid of 768 runs in one round.
// For few rows the second stage (W x d floats a set) weighs more than the occupancy of the first, so a workgroup
// then takes several rows: two a wavefront in the wavefront-per-row kernel, three in the other one (777 x 4096: 10.8 + 10.2 us
// with a row a workgroup, 13.9 + 5.6 with three; 2880 x 1024, three sets: 10.4 + 8.1 and 11.8 + 4.8).
int64_t norm_bwd_workgroups(int64_t t, int64_t d) {
  const int64_t nvec = d / 8, rows_per_wg = nvec <= 128 ? 4 * 2 : 3;
  int64_t W = std::min<int64_t>(norm_bwd_partial_rows(t), std::max<int64_t>(std::min<int64_t>(t, 256), t / rows_per_wg));
  W = std::max<int64_t>(1, W);
  if (nvec > 64 && nvec <= 128) W = std::min<int64_t>(W, 768);
  return W;
}

hipError_t launch_norm_bwd(int kind, const void* dy, const void* x, const void* gamma,
                           const float* stats, const void* dres, void* dx, float* dgamma,
                           float* dbeta, PartialSums& sums, int64_t t, int64_t d,
                           int64_t ld, hipStream_t s, float* dx_colsum) {
  if (d % 8 != 0 || d > 8192 || ld < d || ld % 8 != 0) return hipErrorInvalidValue;
  if (dx_colsum && !norm_bwd_colsum_fusable(d)) return hipErrorInvalidValue;
  const int64_t nvec = d / 8;
  // RMSNorm on rows over 2048 wide keeps the next row's operands in registers, and three workgroups per CU (two with four vectors).
  // Narrower rows leave room for four: 32768 x 1280 47.9 us, with three 53.5.
  const int64_t W = std::min<int64_t>(norm_bwd_workgroups(t, d), kind == 1 && nvec > 256 ? (nvec <= 512 ? 768 : 512) : 1024);
  float* partial = nullptr;
  float* beta_out = kind == 0 ? dbeta : nullptr;
  hipError_t e = dx_colsum ? sums.take(W, d, {dgamma, beta_out, dx_colsum}, s, &partial)
               : kind == 0 ? sums.take(W, d, {dgamma, beta_out}, s, &partial) : sums.take(W, d, {dgamma}, s, &partial);
  if (e != hipSuccess) return e;
  ProfScope prof(PROF_ELEMENTWISE, (dres ? 8.0 : 6.0) * (double)t * (double)d, s);
  dim3 grid((unsigned)W), block(256);
#define CALL(NV)                                                                                   \
  if (kind == 0) hipLaunchKernelGGL((norm_bwd_kernel<0, NV>), grid, block, 0, s, (const bf16_t*)dy, \
      (const bf16_t*)x, (const bf16_t*)gamma, stats, (const bf16_t*)dres, (bf16_t*)dx, partial, t, (int)d, ld); \
  else hipLaunchKernelGGL((norm_bwd_kernel<1, NV>), grid, block, 0, s, (const bf16_t*)dy,           \
      (const bf16_t*)x, (const bf16_t*)gamma, stats, (const bf16_t*)dres, (bf16_t*)dx, partial, t, (int)d, ld);
#define CALL_WAVE_CS(KIND, NV, CS)                                                                          \
  hipLaunchKernelGGL((norm_bwd_wave_kernel<KIND, NV, CS>), grid, block, 0, s, (const bf16_t*)dy,             \
      (const bf16_t*)x, (const bf16_t*)gamma, stats, (const bf16_t*)dres, (bf16_t*)dx, partial, t, (int)d, ld);
#define CALL_WAVE(NV)                                                                       \
  if (kind == 0) { if (dx_colsum) { CALL_WAVE_CS(0, NV, true) } else { CALL_WAVE_CS(0, NV, false) } } \
  else { if (dx_colsum) { CALL_WAVE_CS(1, NV, true) } else { CALL_WAVE_CS(1, NV, false) } }
  if (nvec <= 64) { CALL_WAVE(1) } else if (nvec <= 128) { CALL_WAVE(2) }
  else if (nvec <= 256) { CALL(1) } else if (nvec <= 512) { CALL(2) } else { CALL(4) }
#undef CALL_WAVE
#undef CALL_WAVE_CS
#undef CALL
  return hipGetLastError();
}

hipError_t launch_rope(void* qk, const int32_t* pos, int64_t t, int64_t row_stride, int64_t col0,
                       int32_t n_heads, int32_t head_dim, float rope_base, int inverse,
                       hipStream_t s) {
  if (t == 0 || n_heads == 0) return hipSuccess;
  if (head_dim % 16 != 0 || row_stride % 8 != 0 || col0 % 8 != 0) return hipErrorInvalidValue;
  const int64_t n = t * (head_dim / 16);
  ProfScope prof(PROF_ELEMENTWISE, 4.0 * (double)t * (double)n_heads * (double)head_dim, s);
  hipLaunchKernelGGL(rope_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, (bf16_t*)qk, pos, t,
                     row_stride, col0, (int)n_heads, (int)head_dim, log2((double)rope_base), inverse);
  return hipGetLastError();
}

hipError_t launch_rope_from_table(void* qk, const int32_t* pos, const float* table, int64_t t, int64_t row_stride,
                                  int32_t n_heads, int32_t head_dim, hipStream_t s) {
  if (t == 0 || n_heads == 0) return hipSuccess;
  if (head_dim % 16 != 0 || row_stride % 8 != 0) return hipErrorInvalidValue;
  const int64_t n = t * n_heads * (head_dim / 16);
  ProfScope prof(PROF_ELEMENTWISE, 4.0 * (double)t * (double)n_heads * (double)head_dim, s);
  hipLaunchKernelGGL(rope_from_table_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, (bf16_t*)qk, pos, table, t, row_stride,
                     (int)n_heads, (int)head_dim);
  return hipGetLastError();
}

hipError_t launch_rope_table(float* table, int64_t n_pos, int32_t head_dim, float rope_base, hipStream_t s) {
  if (n_pos == 0) return hipSuccess;
  if (head_dim % 16 != 0) return hipErrorInvalidValue;
  const int64_t n = n_pos * (head_dim / 2);
  ProfScope prof(PROF_ELEMENTWISE, 4.0 * (double)n_pos * (double)head_dim, s);
  hipLaunchKernelGGL(rope_table_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, table, n_pos, (int)head_dim,
                     log2((double)rope_base));
  return hipGetLastError();
}

hipError_t launch_begin(const void* meta_src, void* meta, size_t meta_bytes, const RopeTableSpec* tables, int n_tables, int64_t n_pos,
                        const void* copy_src, void* copy_dst, size_t copy_bytes, hipStream_t s) {
  if (meta_bytes % 16 != 0 || copy_bytes % 16 != 0) return hipErrorInvalidValue;
  BeginArgs a;
  a.meta_src = (const uint4*)meta_src; a.meta = (uint4*)meta; a.meta_vec = (int64_t)(meta_bytes / 16);
  a.copy_src = (const uint4*)copy_src; a.copy_dst = (uint4*)copy_dst; a.copy_vec = (int64_t)(copy_bytes / 16);
  a.n_pos = n_pos;
  a.n_tables = std::min(n_tables, BEGIN_TABLES);
  unsigned blocks = blocks_for(a.meta_vec, 256);
  double bytes = 2.0 * (double)(meta_bytes + copy_bytes);
  for (int t = 0; t < a.n_tables; t++) {
    if (tables[t].head_dim % 16 != 0) return hipErrorInvalidValue;
    a.table[t] = {tables[t].table, log2((double)tables[t].base), tables[t].head_dim, (int)blocks};
    blocks += blocks_for(n_pos * (tables[t].head_dim / 2), 256);
    bytes += 4.0 * (double)n_pos * (double)tables[t].head_dim;
  }
  a.copy_first = (int)blocks;
  blocks += blocks_for(a.copy_vec, 256);
  if (blocks > 0) {
    ProfScope prof(PROF_ELEMENTWISE, bytes, s);
    hipLaunchKernelGGL(begin_kernel, dim3(blocks), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  for (int t = a.n_tables; t < n_tables; t++) {
    const hipError_t e = launch_rope_table(tables[t].table, n_pos, tables[t].head_dim, tables[t].base, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_act_fwd(int act, const void* pre, void* a, int64_t t, int64_t f, hipStream_t s) {
  if (t == 0) return hipSuccess;
  if (f % 8 != 0) return hipErrorInvalidValue;
  const int64_t nvec = t * f / 8;
  ProfScope prof(PROF_ELEMENTWISE, (act == 2 ? 6.0 : 4.0) * (double)t * (double)f, s);
  if (act == 2)
    hipLaunchKernelGGL(swiglu_fwd_kernel, dim3(blocks_for(nvec, 256)), dim3(256), 0, s,
                       (const bf16_t*)pre, (bf16_t*)a, t, f);
  else
    hipLaunchKernelGGL(gelu_fwd_kernel, dim3(blocks_for(nvec, 256)), dim3(256), 0, s, act,
                       (const bf16_t*)pre, (bf16_t*)a, nvec);
  return hipGetLastError();
}

hipError_t launch_act_bwd(int act, const void* da, const void* pre, void* dpre, int64_t t,
                          int64_t f, hipStream_t s) {
  if (t == 0) return hipSuccess;
  if (f % 8 != 0) return hipErrorInvalidValue;
  const int64_t nvec = t * f / 8;
  ProfScope prof(PROF_ELEMENTWISE, (act == 2 ? 10.0 : 6.0) * (double)t * (double)f, s);
  if (act == 2)
    hipLaunchKernelGGL(swiglu_bwd_kernel, dim3(blocks_for(nvec, 256)), dim3(256), 0, s,
                       (const bf16_t*)da, (const bf16_t*)pre, (bf16_t*)dpre, t, f);
  else
    hipLaunchKernelGGL(gelu_bwd_kernel, dim3(blocks_for(nvec, 256)), dim3(256), 0, s, act,
                       (const bf16_t*)da, (const bf16_t*)pre, (bf16_t*)dpre, nvec);
  return hipGetLastError();
}

hipError_t launch_gelu_bwd_colsum(int act, const void* da, const void* pre, void* dpre, float* colsum,
                                  PartialSums& sums, int64_t t, int64_t f, hipStream_t s) {
  if (f % 8 != 0 || (act != 0 && act != 1)) return hipErrorInvalidValue;
  const int64_t P = colsum_partial_rows(t);
  float* partial = nullptr;
  hipError_t e = sums.take(P, f, {colsum}, s, &partial);
  if (e != hipSuccess) return e;
  ProfScope prof(PROF_ELEMENTWISE, 6.0 * (double)t * (double)f, s);
  hipLaunchKernelGGL(gelu_bwd_colsum_kernel, dim3(blocks_for(f, 512), (unsigned)P), dim3(256), 0, s, act,
                     (const bf16_t*)da, (const bf16_t*)pre, (bf16_t*)dpre, partial, t, f);
  return hipGetLastError();
}

// Row chunks of the column sums: what the second stage reads is chunks x n floats, so a chunk holds at least 16 rows
// (four a wavefront, all in flight); 512 chunks fill the chip.  2880 x 4096: second stage 7.2 us with 512 chunks,
// 3.9 us with 180, the first stage unchanged.
int64_t colsum_partial_rows(int64_t t) { return std::max<int64_t>(1, std::min<int64_t>(512, t / 16)); }

hipError_t launch_colsum(const void* x, int64_t ldx, float* out, PartialSums& sums, int64_t t, int64_t n, hipStream_t s) {
  if (n % 8 != 0 || ldx % 8 != 0) return hipErrorInvalidValue;
  const int64_t P = colsum_partial_rows(t);
  float* partial = nullptr;
  hipError_t e = sums.take(P, n, {out}, s, &partial);
  if (e != hipSuccess) return e;
  ProfScope prof(PROF_ELEMENTWISE, 2.0 * (double)t * (double)n, s);
  hipLaunchKernelGGL(colsum_partial_kernel, dim3(blocks_for(n, 512), (unsigned)P), dim3(256), 0, s,
                     (const bf16_t*)x, ldx, partial, t, n);
  return hipGetLastError();
}

hipError_t launch_scatter_rows(const void* src, void* dst, const int32_t* rows, int64_t n_rows,
                               int64_t d, int gather, hipStream_t s) {
  if (n_rows == 0) return hipSuccess;
  if (d % 8 != 0) return hipErrorInvalidValue;
  const int64_t n = n_rows * (d / 8);
  ProfScope prof(PROF_ELEMENTWISE, 4.0 * (double)n_rows * (double)d, s);
  hipLaunchKernelGGL(scatter_rows_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s,
                     (const bf16_t*)src, (bf16_t*)dst, rows, n_rows, d / 8, gather);
  return hipGetLastError();
}

hipError_t launch_pool_rows(const void* src, void* dst, const int32_t* first, const int32_t* count,
                            int64_t n_out, int64_t d, hipStream_t s) {
  if (n_out == 0) return hipSuccess;
  if (d % 8 != 0) return hipErrorInvalidValue;
  const int64_t n = n_out * (d / 8);
  ProfScope prof(PROF_ELEMENTWISE, 4.0 * (double)n_out * (double)d, s);
  hipLaunchKernelGGL(pool_rows_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, (const bf16_t*)src,
                     (bf16_t*)dst, first, count, n_out, d / 8);
  return hipGetLastError();
}

hipError_t launch_unpool_rows(const void* src, void* dst, const int32_t* window, const int32_t* count,
                              int64_t n_rows, int64_t d, hipStream_t s) {
  if (n_rows == 0) return hipSuccess;
  if (d % 8 != 0) return hipErrorInvalidValue;
  const int64_t n = n_rows * (d / 8);
  ProfScope prof(PROF_ELEMENTWISE, 4.0 * (double)n_rows * (double)d, s);
  hipLaunchKernelGGL(unpool_rows_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, (const bf16_t*)src,
                     (bf16_t*)dst, window, count, n_rows, d / 8);
  return hipGetLastError();
}

hipError_t launch_connector_grad(const void* dy, void* dproj, void* dx_seq, const int32_t* rows, const uint32_t* scattered, int64_t n_rows,
                                 int64_t n_seq, int64_t d, hipStream_t s) {
  if (n_seq == 0) return hipSuccess;
  if (d % 8 != 0) return hipErrorInvalidValue;
  const unsigned first = blocks_for(n_rows * (d / 8), 256), rest = blocks_for(n_seq * (d / 8), 256);
  ProfScope prof(PROF_ELEMENTWISE, 4.0 * (double)(n_rows + n_seq) * (double)d, s);
  hipLaunchKernelGGL(connector_grad_kernel, dim3(first + rest), dim3(256), 0, s, (const uint4*)dy, (uint4*)dproj, (uint4*)dx_seq, rows, scattered, n_rows,
                     n_seq, d / 8, (int)first);
  return hipGetLastError();
}

hipError_t launch_splitk_reduce(const float* partial, void* c, int splits, int64_t m, int64_t n, int out_fp32,
                                int accumulate, const void* bias, const void* residual, int64_t ldres, hipStream_t s) {
  if (m == 0 || n == 0) return hipSuccess;
  if (n % 8 != 0 || (residual && ldres % 8 != 0)) return hipErrorInvalidValue;
  const int64_t nvec = m * n / 8;
  ProfScope prof(PROF_ELEMENTWISE, (double)m * (double)n * (4.0 * splits + (out_fp32 ? (accumulate ? 8.0 : 4.0) : (residual ? 4.0 : 2.0))), s);
  const dim3 grid(blocks_for(nvec, 256)), block(256);
  if (out_fp32)
    hipLaunchKernelGGL(splitk_reduce_kernel<true>, grid, block, 0, s, (const float4*)partial, c, splits, nvec, n / 8, accumulate,
                       (const bf16_t*)bias, (const bf16_t*)nullptr, (int64_t)0);
  else
    hipLaunchKernelGGL(splitk_reduce_kernel<false>, grid, block, 0, s, (const float4*)partial, c, splits, nvec, n / 8, 0,
                       (const bf16_t*)bias, (const bf16_t*)residual, ldres);
  return hipGetLastError();
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  if (bytes % 16 != 0) return hipErrorInvalidValue;
  const int64_t nvec = (int64_t)(bytes / 16);
  ProfScope prof(PROF_ELEMENTWISE, 2.0 * (double)bytes, s);
  hipLaunchKernelGGL(copy_kernel, dim3(blocks_for(nvec, 256)), dim3(256), 0, s, (const uint4*)src,
                     (uint4*)dst, nvec);
  return hipGetLastError();
}

}  // namespace mllm
