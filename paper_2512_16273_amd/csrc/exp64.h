// exp(x) in fp64 for the inverse-CDF passes, where x = s - s_max <= 0 (small positive arguments work
// too).  Range reduction x = n*ln2 + r with |r| <= ln2/2, a degree-13 Taylor polynomial for exp(r)
// (truncation error below 2^-57) and a scaling by 2^n; the result is within about one ulp of the
// correctly rounded value.  Arguments below about -709 (including -inf and NaN) give exactly 0:
// results that would be subnormal are flushed.  Branch-free, and written with the operations that
// run at full rate on gfx950: rounding to an integer and the scaling are done with a "magic number"
// addition and an exponent-field construction instead of rint / convert / ldexp, which issue at a
// quarter of the rate there.
//
// pow_exp is the same function for the long sums, through a table that a workgroup builds in LDS.
#pragma once
#include <stdint.h>
#include <string.h>

#if defined(__HIPCC__)
#define TSLT_HD __host__ __device__ __forceinline__
#else
#define TSLT_HD inline
#endif

namespace tslt {

TSLT_HD double exp64(double x) {
  x = x > -800.0 ? x : -800.0;                                   // also maps -inf (and NaN) to -800
  // n = round(x / ln2): adding 1.5 * 2^52 leaves n in the low mantissa bits of t
  const double kMagic = 6755399441055744.0;
  const double t = __builtin_fma(x, 1.44269504088896338700e+00, kMagic);
  const double n = t - kMagic;
  uint64_t tb;
  memcpy(&tb, &t, 8);
  int32_t ni = int32_t(uint32_t(tb));                             // n as an integer (|n| < 2^31)
  double r = __builtin_fma(n, -6.93147180369123816490e-01, x);   // high part of ln2 (low 32 bits zero)
  r = __builtin_fma(n, -1.90821492927058770002e-10, r);          // low part of ln2
  double p = 1.6059043836821613e-10;                              // 1/13!
  p = __builtin_fma(p, r, 2.08767569878681e-09);                  // 1/12!
  p = __builtin_fma(p, r, 2.505210838544172e-08);                 // 1/11!
  p = __builtin_fma(p, r, 2.755731922398589e-07);                 // 1/10!
  p = __builtin_fma(p, r, 2.7557319223985893e-06);                // 1/9!
  p = __builtin_fma(p, r, 2.48015873015873e-05);                  // 1/8!
  p = __builtin_fma(p, r, 1.984126984126984e-04);                 // 1/7!
  p = __builtin_fma(p, r, 1.388888888888889e-03);                 // 1/6!
  p = __builtin_fma(p, r, 8.333333333333333e-03);                 // 1/5!
  p = __builtin_fma(p, r, 4.1666666666666664e-02);                // 1/4!
  p = __builtin_fma(p, r, 1.6666666666666666e-01);                // 1/3!
  p = __builtin_fma(p, r, 0.5);
  p = __builtin_fma(p, r, 1.0);
  p = __builtin_fma(p, r, 1.0);
  // 2^n built in the exponent field; n <= -1023 gives the bit pattern of 0.0
  ni = ni > -1023 ? ni : -1023;
  const uint64_t sb = uint64_t(uint32_t(ni + 1023)) << 52;
  double scale;
  memcpy(&scale, &sb, 8);
  return p * scale;
}

// exp(x) and exp(-x), |x| <= 700: the same series, its even and odd parts apart, so that the second value costs eight operations
// (a table of both signs takes little more than half the time).  Every rounding but the last is of a quantity below 0.07, or of r.
TSLT_HD void exp64_pair(double x, double& plus, double& minus) {
  const double kMagic = 6755399441055744.0;
  const double t = __builtin_fma(x, 1.44269504088896338700e+00, kMagic);
  const double n = t - kMagic;
  uint64_t tb;
  memcpy(&tb, &t, 8);
  const int32_t ni = int32_t(uint32_t(tb));
  double r = __builtin_fma(n, -6.93147180369123816490e-01, x);
  r = __builtin_fma(n, -1.90821492927058770002e-10, r);
  const double r2 = r * r;
  double odd = 1.6059043836821613e-10;                            // 1/13!
  odd = __builtin_fma(odd, r2, 2.505210838544172e-08);
  odd = __builtin_fma(odd, r2, 2.7557319223985893e-06);
  odd = __builtin_fma(odd, r2, 1.984126984126984e-04);
  odd = __builtin_fma(odd, r2, 8.333333333333333e-03);
  odd = __builtin_fma(odd, r2, 1.6666666666666666e-01);
  odd = odd * r2;                                                 // sinh(r) / r - 1
  double even = 2.08767569878681e-09;                             // 1/12!
  even = __builtin_fma(even, r2, 2.755731922398589e-07);
  even = __builtin_fma(even, r2, 2.48015873015873e-05);
  even = __builtin_fma(even, r2, 1.388888888888889e-03);
  even = __builtin_fma(even, r2, 4.1666666666666664e-02);
  even = __builtin_fma(even, r2, 0.5);
  even = even * r2;
  const uint64_t up = uint64_t(uint32_t(1023 + ni)) << 52, down = uint64_t(uint32_t(1023 - ni)) << 52;
  double scale_up, scale_down;
  memcpy(&scale_up, &up, 8);
  memcpy(&scale_down, &down, 8);
  const double p = 1.0 + r, m = 1.0 - r;                          // and what their rounding leaves
  const double dp = r - (p - 1.0), dm = (1.0 - m) - r;
  plus = (p + (dp + __builtin_fma(r, odd, even))) * scale_up;
  minus = (m + (dm + __builtin_fma(-r, odd, even))) * scale_down;
}

// exp(x) for a finite x with |x| <= 700 (in the kernels an fp32 value) through a table of 2^(i/2048):
// x = n * ln2/2048 + r, |r| <= ln2/4096, exp(x) = 2^(n div 2048) * table[n mod 2048] * (1 + r + r^2/2 + r^3/6) (the
// series is cut below 2^-54).  Half the fp64 operations of exp64, for one 8-byte read from LDS; within about 1.3
// ulp (exp64: 0.9).  An entry is 2^(i/2048) with i << 9 taken off its high word, so that adding n << 9 there scales by
// 2^(n div 2048) without n's low bits having to be masked out.
constexpr int kPowEntries = 2048;
TSLT_HD uint64_t pow_entry(int i) {
  // 2^(i/2048) = 2^m * exp(r), m = 0 or 1, r = (i - 2048 m) * ln2/2048 as a sum rh + rl (rh exact) with |r| <= ln2/2;
  // exp(r) = 1 + rh + c, where rounding in c counts for little and the last addition is the only one at full size
  const int m = i > kPowEntries / 2 ? 1 : 0;
  const double k = double(i - m * kPowEntries);
  const double rh = k * (6.93147180369123816490e-01 / kPowEntries);
  const double rl = k * (1.90821492927058770002e-10 / kPowEntries);
  double p = 1.1470745597729725e-11;                              // 1/14!
  p = __builtin_fma(p, rh, 1.6059043836821613e-10);
  p = __builtin_fma(p, rh, 2.08767569878681e-09);
  p = __builtin_fma(p, rh, 2.505210838544172e-08);
  p = __builtin_fma(p, rh, 2.755731922398589e-07);
  p = __builtin_fma(p, rh, 2.7557319223985893e-06);
  p = __builtin_fma(p, rh, 2.48015873015873e-05);
  p = __builtin_fma(p, rh, 1.984126984126984e-04);
  p = __builtin_fma(p, rh, 1.388888888888889e-03);
  p = __builtin_fma(p, rh, 8.333333333333333e-03);
  p = __builtin_fma(p, rh, 4.1666666666666664e-02);
  p = __builtin_fma(p, rh, 1.6666666666666666e-01);
  p = __builtin_fma(p, rh, 0.5);
  const double c0 = rh * rh * p;                                  // exp(rh) - 1 - rh
  const double c = c0 + rl * (1.0 + (rh + c0));
  const double big = 1.0 + rh;
  const double v = big + ((rh - (big - 1.0)) + c);
  uint64_t b;
  memcpy(&b, &v, 8);
  return b + (uint64_t(uint32_t(m << 20) - (uint32_t(i) << 9)) << 32);
}
TSLT_HD double pow_exp(float s, const uint64_t* table) {
  const double x = double(s);
  const double kMagic = 6755399441055744.0;
  const double t = __builtin_fma(x, 1.44269504088896338700e+00 * kPowEntries, kMagic);
  const double n = t - kMagic;
  uint64_t tb;
  memcpy(&tb, &t, 8);
  const uint32_t ni = uint32_t(tb);
  double r = __builtin_fma(n, -6.93147180369123816490e-01 / kPowEntries, x);
  r = __builtin_fma(n, -1.90821492927058770002e-10 / kPowEntries, r);
  double q = __builtin_fma(r, 1.6666666666666666e-01, 0.5);
  q = __builtin_fma(q, r, 1.0);
  q = q * r;
  const uint64_t e = table[ni & (kPowEntries - 1)];
#if defined(__HIP_DEVICE_COMPILE__)
  const double v = __hiloint2double(int(uint32_t(e >> 32) + (ni << 9)), int(uint32_t(e)));
#else
  const uint64_t b = (uint64_t(uint32_t(e >> 32) + (ni << 9)) << 32) | uint32_t(e);
  double v;
  memcpy(&v, &b, 8);
#endif
  return __builtin_fma(v, q, v);
}

}  // namespace tslt
