// Device helper of the kernels that place K/V rows in an fp8 cache: bf16 values to e4m3 codes.
#pragma once

#include <hip/hip_runtime.h>

namespace cronus {

typedef unsigned int codes8 __attribute__((ext_vector_type(2)));

// Eight codes e4m3_rne(clamp(x / scale, -448, 448)), those of one IEEE fp32 division each.  With
// r = RN(1 / scale), q = RN(x r) and d = RN(q scale - x), the quotient here is RN(q - d r) (the residual step
// of Markstein's method).  q can be 1.5 ulp from x / scale where his theorem asks for 1, so the quotient is not
// claimed to be correctly rounded; but q - d r is within 2^-22 ulp of x / scale, so it differs from the division only next to
// the midpoint of two fp32 numbers, and the code only if one of them is a boundary between two codes, B 2^n with
// 16 <= B < 32.  That asks for x = (B + 2^-20) 2^n scale (or B - 2^-20) but for a relative 2^-45, with scale =
// (k / 8 + j 2^-23) 2^m, 8 <= k < 16 and a small j: the bits of x below its 8-bit significand vanish
// only if B j = -k (or k), and 16 <= B > k has no such j.  Under- and overflow: for scales of
// 2^-64 .. 2^64 they concern quotients below 2^-11, whose code is a zero either way, and above
// 1024, where q is clamped first (the correction then only has to be positive or infinite).
// The residual's sign is such that -0 stays -0.  Other scales divide.  The kernel was bound by
// these instructions: 11 an element with the division, one conversion per code and a packing of bytes; 5.5 now.
struct Quantiser {
  float scale, r;
  bool exact;
};
__device__ __forceinline__ Quantiser make_quantiser(float scale) {
  return Quantiser{scale, 1.0f / scale, fabsf(scale) >= 0x1p-64f && fabsf(scale) <= 0x1p64f};
}
__device__ __forceinline__ codes8 quant_e4m3_x8(const float (&x)[8], const Quantiser& z) {
  float y[8];
  if (z.exact) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float q = __builtin_amdgcn_fmed3f(x[e] * z.r, -1024.0f, 1024.0f);
      y[e] = __builtin_fmaf(-__builtin_fmaf(q, z.scale, -x[e]), z.r, q);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = x[e] / z.scale;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] = fminf(fmaxf(y[e], -448.0f), 448.0f);
  codes8 c;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(y[4 * h], y[4 * h + 1], 0, false);
    c[h] = (unsigned int)__builtin_amdgcn_cvt_pk_fp8_f32(y[4 * h + 2], y[4 * h + 3], lo, true);
  }
  return c;
}

}  // namespace cronus
