// 8-bit floating point (OCP FP8 E4M3: 1 sign, 4 exponent bits with bias 7, 3 mantissa bits, no
// infinities, largest finite value 448) as used for the 8-bit KV cache.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace efim {

// binary32 -> E4M3 code: round to nearest, ties to the even code; magnitudes of 448 and above
// saturate to +-448; NaN gives the NaN code.  Integer arithmetic on the bit pattern, so the
// result does not depend on any conversion instruction's mode bits.
__device__ __forceinline__ uint32_t f32_to_e4m3(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t sign = (u >> 24) & 0x80u;
  const uint32_t a = u & 0x7FFFFFFFu;
  if (a > 0x7F800000u) return 0x7Fu;                 // NaN
  if (a >= 0x43E00000u) return sign | 0x7Eu;         // |f| >= 448
  if (a >= 0x3C800000u) {                            // |f| >= 2^-6: normal E4M3 range
    // keep 3 mantissa bits: add half of the dropped part (less one when the kept part is even)
    const uint32_t r = (a + 0x7FFFFu + ((a >> 20) & 1u)) >> 20;  // (biased exponent << 3) | mantissa
    return sign | (r - ((127u - 7u) << 3));
  }
  // below the smallest normal the codes are the integers m = |f| * 2^9 (m == 8 is 2^-6 itself)
  return sign | (uint32_t)__builtin_rintf(__builtin_fabsf(f) * 512.f);
}

// The correctly rounded binary32 quotient of a bf16 value and a binary32 scale, from inv = 1 / (double)scale.
// The fp64 product is within 2^-52 of the quotient, which has at least 2^-49 to the next midpoint of two
// binary32 numbers: in whole units of the last places the difference of the value and midpoint x scale is an
// integer below 2^49 and not zero (a 25-bit odd midpoint times the scale has more than the 8 bits of the
// value).  Only quotients below 2^-126, whose midpoints are shorter, may differ, and all of those give code 0.
__device__ __forceinline__ float bf16_quotient(uint32_t f32_bits, double inv) {
  return (float)((double)__uint_as_float(f32_bits) * inv);
}

// E4M3 codes of two quotients in the lower (HIGH: upper) half of a word, NaN excepted: the conversion instruction
// agrees with f32_to_e4m3 on every float once the magnitude is clamped (beyond 448 it would depend
// on a mode bit).
template <bool HIGH>
__device__ __forceinline__ uint32_t e4m3_pair(float a, float b, uint32_t word) {
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(a, -448.f, 448.f),
                                                   __builtin_amdgcn_fmed3f(b, -448.f, 448.f), (int)word, HIGH);
}

// Code of a bf16 value (bit pattern) under a per-tensor scale: the quotient is the binary32
// division, correctly rounded; inv = 1 / (double)scale.
__device__ __forceinline__ uint32_t bf16_bits_to_e4m3(uint32_t bits16, double inv) {
  const float f = bf16_quotient(bits16 << 16, inv);
  return f != f ? 0x7Fu : e4m3_pair<false>(f, f, 0u) & 0xFFu;
}

}  // namespace efim
