// Rotary-embedding arithmetic shared by the kernels that rotate new tokens: fp64 rotation of a
// pair, rounded once to bf16, so that every kernel produces the same bits for the same input.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace efim {

__device__ __forceinline__ double bf16_bits_to_f64(uint32_t bits16) {
  return (double)__uint_as_float(bits16 << 16);
}

// fp64 -> bf16, round to nearest even, with a single rounding.  The conversion goes through
// fp32; the only case where the detour could round twice is an inexact fp32 result sitting
// exactly on a bf16 midpoint, which is nudged to the side the exact value lies on.
__device__ __forceinline__ uint32_t f64_to_bf16_bits(double x) {
  float f = (float)x;
  uint32_t u = __float_as_uint(f);
  if ((u & 0xFFFFu) == 0x8000u) {
    double back = (double)f;
    if (back != x) u = (fabs(x) > fabs(back)) ? u + 1u : u - 1u;
  }
  // round to nearest even on the upper 16 bits (NaN stays NaN: quiet bit is in the upper half)
  uint32_t lsb = (u >> 16) & 1u;
  if ((u & 0x7F800000u) != 0x7F800000u) u += 0x7FFFu + lsb;
  return u >> 16;
}

// (x1, x2) rotated by the angle whose cosine and sine are c and s, in fp64; products and sums are
// separate operations (no fused multiply-add).
__device__ __forceinline__ void rotate_pair_f64(uint32_t x1_bits, uint32_t x2_bits, double c, double s, double* y1,
                                                double* y2) {
#pragma clang fp contract(off)
  const double x1 = bf16_bits_to_f64(x1_bits), x2 = bf16_bits_to_f64(x2_bits);
  *y1 = x1 * c - x2 * s;
  *y2 = x2 * c + x1 * s;
}

// The same, rounded once to bf16 each.
__device__ __forceinline__ void rotate_pair_bf16(uint32_t x1_bits, uint32_t x2_bits, double c, double s,
                                                 uint32_t* y1_bits, uint32_t* y2_bits) {
  double y1, y2;
  rotate_pair_f64(x1_bits, x2_bits, c, s, &y1, &y2);
  *y1_bits = f64_to_bf16_bits(y1);
  *y2_bits = f64_to_bf16_bits(y2);
}

// Two fp32 values as bf16 words, nearest even: one instruction (it agrees with the integer rounding
// of f64_to_bf16_bits on every float that is no signalling NaN).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

// Lower halves of two fp32 values, each zero where the value is a midpoint of two bf16 numbers: there
// alone the way from fp64 through fp32 can round twice.
__device__ __forceinline__ uint32_t off_midpoint(float lo, float hi) {
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x05040100u) ^ 0x80008000u;
}

}  // namespace efim
