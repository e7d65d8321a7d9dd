// Shared device-side helpers for the gfx950 kernels: bf16 conversion, MFMA fragment types,
// LDS transposing reads, wavefront reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mllm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef uint16_t bf16_t;  // raw storage type in global memory

#define MLLM_LDS __attribute__((address_space(3)))

// fp32 -> bf16, round to nearest even, through the hardware conversion (v_cvt_pk_bf16_f32).
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_t;
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  const bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
  return __builtin_bit_cast(uint32_t, b);
}
__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

union Frag8 {  // eight bf16 = one MFMA A/B operand of the k=16 (32x32) or k=32 (16x16) shapes
  bf16x8 v;
  uint4 u;
  uint32_t w[4];
  s16x4 h[2];
};

// LDS transposing read.  Within each group of 16 lanes, lane i returns
// tile[k0 + e][n0 + i] for e = 0..3 when the lane passes the address of
// tile[k0 + i/4][n0 + 4*(i%4)] (tile rows are `stride` elements apart).
__device__ __forceinline__ s16x4 lds_read_tr4(const bf16_t* tile, int stride, int k0, int n0,
                                              int lane16) {
  const bf16_t* p = tile + (k0 + (lane16 >> 2)) * stride + n0 + 4 * (lane16 & 3);
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLLM_LDS s16x4*)p);
}

// erf to 1.5e-7 absolute (Abramowitz and Stegun 7.1.26: 1 - (a1 t + ... + a5 t^5) exp(-x^2) with
// t = 1 / (1 + p |x|), odd in x), with the hardware reciprocal and exp2: a dozen instructions where
// the library routine takes several times as many, which made the GELU kernels ALU-bound.  The
// results are rounded to bf16 (2^-9 relative), far above this error.
__device__ __forceinline__ float fast_erf(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.f));
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * ax * ax);
  return copysignf(fmaf(-p * t, e, 1.f), x);
}
// GELU (act 0: exact erf form, 1: tanh form) and its derivative.
// tanh through the hardware exp2 and reciprocal: 1 - 2 / (1 + e^(2u)); exact at both ends (e = inf or 0).
__device__ __forceinline__ float fast_tanh(float u) {
  return fmaf(-2.f, __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(2.8853900817779268f * u)), 1.f);
}
__device__ __forceinline__ float gelu_f(int act, float z) {
  if (act == 1) {
    float u = 0.7978845608028654f * (z + 0.044715f * z * z * z);
    return 0.5f * z * (1.f + fast_tanh(u));
  }
  return 0.5f * z * (1.f + fast_erf(z * 0.7071067811865476f));
}
__device__ __forceinline__ float gelu_grad_f(int act, float z) {
  if (act == 1) {
    float u = 0.7978845608028654f * (z + 0.044715f * z * z * z);
    float t = fast_tanh(u);
    return 0.5f * (1.f + t) +
           0.5f * z * (1.f - t * t) * 0.7978845608028654f * (1.f + 3.f * 0.044715f * z * z);
  }
  return 0.5f * (1.f + fast_erf(z * 0.7071067811865476f)) +
         z * __builtin_amdgcn_exp2f(-0.7213475204444817f * z * z) * 0.3989422804014327f;
}

// Loads from memory straight into LDS, written as assembly so that the compiler does not know them for what they are.  Told (through the builtin), it makes LDS
// reads wait for every such load in flight into the same LDS variable, which turns a queue of several tiles on their way
// into one tile at a time; it cannot see that the loads go to a stage nobody reads.  The kernels wait for their loads by
// count and separate writers from readers with barriers, as they have to anyway.
// The 64 lanes' 16 (or 4) bytes land side by side from LDS address `lds_addr` (wavefront-uniform).
// The statements set M0 themselves; M0 is a reserved register that the compiler holds no value in and
// sets anew in front of each of its own uses, so overwriting it here disturbs nothing.
// `row_off` (wavefront-uniform) is added to the lanes' offsets, and the range check covers the sum.
typedef int i32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4_t raw_rsrc(const void* base, uint32_t bytes) {   // untyped buffer over [base, base + bytes)
  const uint64_t b = (uint64_t)base;
  i32x4_t r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(b >> 32) & 0xffffu));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}
__device__ __forceinline__ void load_to_lds_b128(i32x4_t rsrc, uint32_t lds_addr, uint32_t byte_off, uint32_t row_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_addr), "v"(byte_off), "s"(rsrc), "s"(row_off) : "memory");
}
__device__ __forceinline__ void load_to_lds_b32(i32x4_t rsrc, uint32_t lds_addr, uint32_t byte_off, uint32_t row_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
               :: "s"(lds_addr), "v"(byte_off), "s"(rsrc), "s"(row_off) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(MLLM_LDS const void* p) { return (uint32_t)(size_t)p; }
// At most N of the loads above still in flight (the compiler does not count them, so neither can its builtin).
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace mllm
