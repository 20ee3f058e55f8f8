// The correctly rounded quotient x / s of a quantization block by the block's
// reciprocal.  Plain C++ (no HIP), so that it can be checked on any host.
#pragma once

#ifdef __HIP__
#define HYQ_HD __host__ __device__ inline
#else
#define HYQ_HD inline
#endif

namespace hyq {

// With r = fl32(1 / s): q = x * r, then one residual correction
// q + r * (x - q * s) with fused multiply-adds (the last step of Markstein's
// division, IBM Journal of Research and Development 34, 1990).  For bf16 x with |x| <= amax and s = fl32(amax / c),
// c one of 127, 7, 448, 6, 7.5, this is the correctly rounded float32
// quotient x / s, apart from the sign of a zero: tests/recip_check.cpp goes
// through every pair of mantissas and every exponent difference that can give
// a nonzero code (nothing else matters as long as no step under- or
// overflows, which recip_ok guarantees for those x; smaller x give a quotient
// below every rounding boundary either way).
HYQ_HD bool recip_ok(float s) { return s >= 0x1p-60f && s <= 0x1p125f; }
HYQ_HD float recip_quotient(float x, float s, float r) {
  const float q = x * r;
  return __builtin_fmaf(__builtin_fmaf(-q, s, x), r, q);
}

}  // namespace hyq
