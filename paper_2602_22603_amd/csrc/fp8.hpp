// fp8.hpp - the 8-bit E4M3 KV-cache code on gfx950: quantisation of a float
// and conversion of stored codes to bf16 for the matrix cores (the native
// conversion instructions).
// Internal to libsq.
//
// E4M3 (the OCP 8-bit format, gfx950's native FP8): sign, 4 exponent bits
// with bias 7, 3 mantissa bits; exponent field 0 holds the subnormals
// m * 2^-9; codes 0x7F / 0xFF are NaN; the largest finite magnitude is 448.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sq {

// The codes of y0 and y1 (bits 0-7 and 8-15): the nearest (ties to the even
// code), magnitudes >= 448 saturating to 448, the sign kept.  The conversion
// instruction rounds so but does not saturate, so the values are clamped in
// front of it.  Neither may be NaN.  With the code put together from the
// float's fields instead, appending 4096 tokens of 12 layers took 76 us; 60
// with the instruction.
__device__ inline uint32_t e4m3_encode2(float y0, float y1) {
  const float c0 = __builtin_amdgcn_fmed3f(y0, -448.f, 448.f);
  const float c1 = __builtin_amdgcn_fmed3f(y1, -448.f, 448.f);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c0, c1, 0, false) & 0xffffu;
}
__device__ inline uint32_t e4m3_encode(float y) { return e4m3_encode2(y, 0.f) & 0xffu; }

// Four codes (bytes of w, lowest first) as four bf16 values (two 32-bit
// words, lowest first).  Exact for every finite code.
__device__ inline uint2 e4m3x4_to_bf16(uint32_t w) {
  const auto lo = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
  const auto hi = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true);
  return make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
}

} // namespace sq
