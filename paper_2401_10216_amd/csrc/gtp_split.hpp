// Split-operand contractions on the 16-bit matrix cores: in two fp16 parts
// (gtp_mfma.hip: v as h1 + h2, h1 = fp16(v), h2 = fp16(v - h1)), and in three
// bf16 parts (gtp_mixq.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gtp {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2v __attribute__((ext_vector_type(2)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma(u4 a, u4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f4 mfma32(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Two values as (h1, h1') and (h2, h2'), rounded to nearest even.
__device__ __forceinline__ void split2(float a, float b, uint32_t& p1, uint32_t& p2) {
  const h2v h = __builtin_convertvector(f2v{a, b}, h2v);
  p1 = __builtin_bit_cast(uint32_t, h);
  // a - float(h[0]), b - float(h[1]): exact, one instruction each
  float ra, rb;
  asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(ra) : "v"(p1), "v"(a));
  asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rb) : "v"(p1), "v"(b));
  p2 = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{ra, rb}, h2v));
}
// Four values as the operand quad (h1 x 4, h2 x 4).
__device__ __forceinline__ u4 split4(float a, float b, float c, float d) {
  u4 q;
  uint32_t p, r;
  split2(a, b, p, r);
  q[0] = p;
  q[2] = r;
  split2(c, d, p, r);
  q[1] = p;
  q[3] = r;
  return q;
}

__device__ __forceinline__ f4 mfma_bf(u4 a, u4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
}

// Two values in three bf16 parts each, rounded to nearest even: b1 = bf16(v),
// b2 = bf16(v - b1), b3 = v - b1 - b2.  Exact for every fp32 value from 2^-110
// up (|b2| <= 2^-8 |v|, |b3| <= 2^-16 |v|, and v's last bit is 2^-23 of its
// first), whatever the values beside it: bf16 has fp32's exponents.
__device__ __forceinline__ void split3(float a, float b, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
  p1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, b2v));
  float ra = a - __uint_as_float(p1 << 16), rb = b - __uint_as_float(p1 & 0xffff0000u);
  p2 = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{ra, rb}, b2v));
  ra -= __uint_as_float(p2 << 16);
  rb -= __uint_as_float(p2 & 0xffff0000u);
  p3 = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{ra, rb}, b2v));
}
// Eight values as three operands.
__device__ __forceinline__ void split3x8(const float (&v)[8], u4 (&o)[3]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t a, b, c;
    split3(v[2 * j], v[2 * j + 1], a, b, c);
    o[0][j] = a;
    o[1][j] = b;
    o[2][j] = c;
  }
}

// Sums and maxima over the four 16-lane rows (gfx950 permlane swaps).
template <typename Op>
__device__ __forceinline__ float rows_all(float v, Op op) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float add_rows(float v) {
  return rows_all(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float max_rows(float v) {
  return rows_all(v, [](float a, float b) { return fmaxf(a, b); });
}

}  // namespace
}  // namespace gtp
