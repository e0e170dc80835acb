// MXFP8 encoding shared by the quantizer and the GEMM epilogues (gfx950).
#pragma once
#include "common.h"

namespace moe {

typedef int i32x8 __attribute__((ext_vector_type(8)));

// floor(log2 amax) - 8 clamped to [-127, 127]; amax >= 0 finite.  A zero or
// subnormal amax (floor(log2) <= -127) clamps to -127.
__device__ __forceinline__ int mx_shared_exp(float amax) {
  const int ef = int((__float_as_uint(amax) >> 23) & 0xFFu);
  if (ef == 0) return -127;
  const int e = ef - 127 - 8;
  return e < -127 ? -127 : (e > 127 ? 127 : e);
}

// 2^-se for se in [-127, 119] (always a normal float).
__device__ __forceinline__ float mx_inv_scale(int se) { return __uint_as_float(uint32_t(127 - se) << 23); }

// E4M3 codes of four values with |v| < 512, packed low byte first: the nearest
// E4M3 value, ties to an even mantissa, magnitudes above 448 saturated to 448,
// the sign bit kept (also for zero).  gfx950's v_cvt_pk_fp8_f32 converts to OCP
// E4M3 rounding to nearest even; clamping to +-448 first gives the saturation.
// For every fp32 input with |v| < 512 this yields the codes of the definition
// (binade e = max(floor(log2 |v|), -6), spacing 2^(e-3), ties to even), which
// was checked over all 2^31 such bit patterns.
__device__ __forceinline__ uint32_t e4m3_pack4(float a, float b, float c, float d) {
  auto sat = [](float v) { return __builtin_amdgcn_fmed3f(v, -448.0f, 448.0f); };
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(sat(a), sat(b), 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(sat(c), sat(d), w, true);
  return uint32_t(w);
}

}  // namespace moe
