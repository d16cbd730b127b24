// gamma_c = floor(beta_c / delta_s + rho) of a softmax step by a short chain of operations; soft_gamma for a wave
// with one class per lane.
//
// The inner loop fixes the order of roundings from x^T z to gamma: the margins' maximum, exp, the pairwise
// normaliser, a division -- ~90 dependent fp64 instructions, 700 cycles of a lone wave.  With p0, the softmax
// before the offset, at hand the same number is
//   p_c = p0_c e_c / sum_k p0_k e_k,   e_c = exp(delta_c),   delta = what the margins moved by,
// which needs no maximum; the sum over classes is two fp64 4x4x4 matrix instructions (28 cycles each instead of
// four exchanges of 24), the reciprocal the hardware's with one correction, and the rest one multiply-add:
//   t = -k2 p0_c e_c / sum + C',   C' = kSoftDraw - rho + k2 p0_c,   k2 = (alpha / B) / delta_s
// whose high word is a constant minus gamma (plus: with the signs turned) and whose low word is the fraction.
// It differs from the fixed order by less than k2 2^-40 (|delta| <= 64, |phi| <= 1024, sum > 1/16; the fixed
// order's own roundings of the exponent, |phi| 2^-52, are most of that), i.e. 2^-19 for k2 < 2^21.  A step with a fraction within
// 2^-16 of an integer, or outside those bounds, is done in the fixed order: one gamma of 32768.
#pragma once

#include "halp_device.hpp"

namespace halp {

constexpr double kSoftMagic = 0x1.8p20;  // a double's last place is 2^-32 here, its high word counts whole numbers
constexpr int kSoftMagicHi = 0x41380000;
constexpr uint32_t kSoftNear = 1u << 16;  // 2^-16
constexpr double kSoftMaxK2 = 0x1p21;

// class of a lane: its four copies are lanes apart by 4
__device__ __forceinline__ int soft_class(int lane) { return (lane & 3) + 4 * (lane >> 4); }
__device__ __forceinline__ bool soft_first_copy(int lane) { return (lane & 12) == 0; }

// e^x to 2^-47, |x| <= 64
__device__ __forceinline__ double exp_short(double x) {
  const double k = __builtin_rint(x * 0x1.71547652b82fep+0);
  double r = __fma_rn(-k, 0x1.62e42fefa39efp-1, x);
  r = __fma_rn(-k, 0x1.abc9e3b39803fp-56, r);
  const double r2 = r * r, r4 = r2 * r2;
  const double a0 = __fma_rn(0x1.5555555555555p-3, r, 0x1.0000000000000p-1);
  const double a1 = __fma_rn(0x1.1111111111111p-7, r, 0x1.5555555555555p-5);
  const double a2 = __fma_rn(0x1.a01a01a01a01ap-13, r, 0x1.6c16c16c16c17p-10);
  const double a3 = __fma_rn(0x1.71de3a556c734p-19, r, 0x1.a01a01a01a01ap-16);
  const double a4 = __fma_rn(0x1.ae64567f544e4p-26, r, 0x1.27e4fb7789f5cp-22);
  const double b0 = __fma_rn(a1, r2, a0), b1 = __fma_rn(a3, r2, a2);
  const double q = __fma_rn(__fma_rn(a4, r4, b1), r4, b0);
  const double s = ldexp(1.0, (int)k);
  return __fma_rn(__fma_rn(r2, q, r), s, s);
}

// What a step needs of its class besides delta, made while the step before runs.
struct SoftDraw {
  double p0, kp, c;  // p0, k2 p0, C'
  bool wide;         // |phi| too large for the bound above
};
template <bool NEGATIVE>
__device__ __forceinline__ SoftDraw soft_draw(bool live, double p0, float phi, uint32_t rho, double k2) {
  SoftDraw v;
  v.p0 = live ? p0 : 0.0;
  v.kp = k2 * v.p0;
  const double r = (double)rho * 0x1p-32, near = kSoftNear * 0x1p-32;
  v.c = NEGATIVE ? (kSoftMagic + 1.0 + near) - r + v.kp : (kSoftMagic + near) + r - v.kp;
  v.wide = live && !(__builtin_fabs((double)phi) <= 1024.0);
  return v;
}

// true, and *hi = kSoftMagicHi -+ gamma before the clamp, unless the step has to be done in the fixed order
template <bool NEGATIVE>
__device__ __forceinline__ bool soft_gamma(const SoftDraw& v, bool live, double delta, int* hi) {
  const double e = exp_short(delta);
  const double kg = NEGATIVE ? -v.kp * e : v.kp * e;
  double s = __builtin_amdgcn_mfma_f64_4x4x4f64(v.p0 * e, 1.0, 0.0, 0, 0, 0);
  s = __builtin_amdgcn_mfma_f64_4x4x4f64(s, 1.0, 0.0, 0, 0, 0);
  double y = __builtin_amdgcn_rcp(s);
  y = __fma_rn(__fma_rn(-s, y, 1.0), y, y);
  const uint64_t bits = __builtin_bit_cast(uint64_t, __fma_rn(kg, y, v.c));
  *hi = (int)(bits >> 32);
  const bool bad = v.wide || !(__builtin_fabs(delta) <= 64.0) || !(s > 0x1p-4) || (live && (uint32_t)bits <= 2 * kSoftNear);
  return __ballot(bad) == 0;
}

// whether the bounds above hold for a chain's scales
__device__ __forceinline__ bool soft_covers(double dscale, double aB, double inv_s) {
  auto normal = [](double x) { return x > 1e-200 && x < 1e200; };
  return normal(dscale) && normal(aB) && normal(inv_s) && aB * inv_s < kSoftMaxK2;
}

}  // namespace halp
