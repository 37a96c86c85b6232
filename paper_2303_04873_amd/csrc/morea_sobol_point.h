// Barycentric coordinates of a Sobol point from its four words, with the bits
// of the definition: lambda_j = e_j / (e_0 + e_1 + e_2 + e_3), e_j = -ln r_j by
// the atanh series, r_j = v_j 2^-24, in FP32 with correctly rounded divisions.
// The divisions are one correction of a product with a reciprocal, which `rcp`
// need only give as one of the two FP32 neighbours of 1 / d -- but for the
// mantissa of all ones, where it has to be the nearest one (so it is on gfx950;
// all 2^23 words, and all mantissas for exponents -26 .. 8, were compared there
// with the divisions).  Plain code, so that it can be run on the host as well.
#pragma once
#include <stdint.h>

namespace morea {
namespace sobol {

// -ln(r) / 2 for r = v 2^-24, v odd and below 2^24: r = m 2^e, m in
// [sqrt(1/2), sqrt(2)], ln m = 2 atanh(s) with s = (m - 1) / (m + 1) and the
// series s (1 + s^2/3 + ... + s^10/11); every operation is that of -ln(r)
// with its result halved, so twice this is -ln(r) to the bit.
template <typename Rcp>
__device__ __forceinline__ float half_neg_log(uint32_t v, Rcp rcp) {
#pragma clang fp contract(off)
  const uint32_t u = __builtin_bit_cast(uint32_t, static_cast<float>(v));
  // -e 2^23: the exponent field of v, one higher from mantissa 0x3504f4
  // (the first above sqrt(2)), from that of 2^24
  const uint32_t x = ((152u << 23) - 1u - 0x4afb0cu - u) & 0xff800000u;
  const float m = __builtin_bit_cast(float, u + x - (24u << 23));
  const float n = m - 1.0f, d = m + 1.0f;
  const float r = rcp(d);
  const float q = n * r;
  const float s = __builtin_fmaf(__builtin_fmaf(-d, q, n), r, q);
  const float s2 = s * s;
  float c = __builtin_fmaf(s2, 0x1.745d18p-4f, 0x1.c71c72p-4f);
  c = __builtin_fmaf(s2, c, 0x1.24924ap-3f);
  c = __builtin_fmaf(s2, c, 0x1.99999ap-3f);
  c = __builtin_fmaf(s2, c, 0x1.555556p-2f);
  c = __builtin_fmaf(s2, c, 1.0f);
  const float p = s * c;
  return __builtin_fmaf(static_cast<float>(static_cast<int>(x)), 0x1.62e430p-25f, -p);
}

// lambda_1..3 of a point from its four words: h_j / (h_0 + h_1 + h_2 + h_3)
// with h_j = -ln r_j / 2.  The sum lies in [2^-23, 2^6]: its refined
// reciprocal is the correctly rounded one, and with it one correction of h r
// rounds the quotient correctly (Markstein's theorem).
template <typename Rcp>
__device__ __forceinline__ void lambdas(const uint32_t v[4], float l[3], Rcp rcp) {
#pragma clang fp contract(off)
  float h[4];
#pragma unroll
  for (int j = 0; j < 4; j++) h[j] = half_neg_log(v[j], rcp);
  const float sum = ((h[0] + h[1]) + h[2]) + h[3];
  float r = rcp(sum);
  r = __builtin_fmaf(__builtin_fmaf(-sum, r, 1.0f), r, r);
#pragma unroll
  for (int j = 0; j < 3; j++) {
    const float q = h[j + 1] * r;
    l[j] = __builtin_fmaf(__builtin_fmaf(-sum, q, h[j + 1]), r, q);
  }
}

}  // namespace sobol
}  // namespace morea
