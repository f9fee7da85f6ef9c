// The logarithm of the Gaussian draws: a fixed sequence of correctly rounded fp32 operations, usable
// (and tested) on the host as well.
#pragma once

#include <cmath>
#include <cstdint>

#ifdef __HIPCC__
#define TMZ_HD_INLINE __host__ __device__ __forceinline__
#else
#define TMZ_HD_INLINE inline
#endif

namespace tmz {

// The correctly rounded quotient n / d from an estimate r of 1 / d, for the operands the
// logarithm has: d = m + 1 in [1.7, 2.5], n = m - 1 zero or at least 2^-24 (m the mantissa in
// [sqrt(1/2), sqrt(2))), so nothing needs scaling and no special case occurs.  The estimate is
// refined once, the quotient corrected by its exact residual.
//   Over the 2^23 mantissas the result is the IEEE quotient for every estimate within 8 ulp,
// except at m = 1 - 2^-23: 1 / d lies 3e-8 of an ulp off the middle of two floats there and only
// the nearer one gives it.  (The radius of those draws is the same either way.)
TMZ_HD_INLINE float quotient_from_rcp(float n, float d, float r) {
  r = fmaf(fmaf(-d, r, 1.0f), r, r);
  const float q = n * r;
  return fmaf(fmaf(-d, q, n), r, q);
}

// Natural log for Box-Muller radii, u in (0, 1]: u = m 2^e with
// m in [sqrt(1/2), sqrt(2)); ln m = 2 atanh((m-1)/(m+1)) by its Taylor series
// through the 11th power; ln2 split in an exact high part and a low part.
template <typename Quotient>
TMZ_HD_INLINE float ln_unit_with(float u, Quotient quotient) {
  const uint32_t bits = __builtin_bit_cast(uint32_t, u);
  int ex = int(bits >> 23) - 127;
  const uint32_t mant = bits & 0x7FFFFFu;
  uint32_t mb = mant | 0x3F800000u;
  if (mant > 0x3504F3u) {
    mb -= 0x00800000u;
    ex += 1;
  }
  const float m = __builtin_bit_cast(float, mb);
  const float f = quotient(m - 1.0f, m + 1.0f);
  const float f2 = 2.0f * f;
  const float t = f * f;
  float p = fmaf(0x1.745d18p-4f, t, 0x1.c71c72p-4f);  // 1/11, 1/9
  p = fmaf(p, t, 0x1.24924ap-3f);                     // 1/7
  p = fmaf(p, t, 0x1.99999ap-3f);                     // 1/5
  p = fmaf(p, t, 0x1.555556p-2f);                     // 1/3
  const float lm = fmaf(f2 * t, p, f2);
  const float e = (float)ex;
  return fmaf(e, 0x1.62e000p-1f, fmaf(e, 0x1.0bfbe8p-15f, lm));
}

}  // namespace tmz
