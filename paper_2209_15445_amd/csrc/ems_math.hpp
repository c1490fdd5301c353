// ems_math.hpp -- double-precision logarithm, exponential, and sine and cosine
// of a turn, for the arguments of the transport.
//
// The step's FP64 work is bound by the instructions a diverged wave issues,
// and the general library functions were a fifth of them: log takes 98 vector
// instructions, exp 42, sincos 158 (double-double arithmetic, tests for
// special values, a reduction for huge angles).  The functions here take 36,
// 25 and 41.  They are for finite positive normal arguments (log), arguments
// whose exponential is in range or near it (exp) and fractions of a turn in
// [0, 1] (sincos), which is all the step code asks of them.  Largest errors
// on the device against long double (test_gpu_device_math.py prints them; 2 to
// 4 million arguments each): log 0.55 units in the last place (the library's
// 0.65), exp 0.73 (0.88), sine and cosine of a turn 1.4e-16 absolute (the
// library's, of the rounded angle, 7.0e-16).
//
// Coefficients: minimax polynomials from the Remez exchange algorithm in
// 60-digit arithmetic; the constants are rounded to double afterwards.
#pragma once
// (EMS_HD: see ems_core.hpp, which includes this file)
#include <stdint.h>
#include <string.h>

namespace ems {

EMS_HD uint64_t bits_of(double v) {
  uint64_t b;
  memcpy(&b, &v, 8);
  return b;
}
EMS_HD double double_of(uint64_t b) {
  double v;
  memcpy(&v, &b, 8);
  return v;
}
// an approximate reciprocal (24 bits or better) of a number in [1, 3]
EMS_HD double rcp_estimate(double d) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcp(d);
#else
  return (double)(1.0f / (float)d);
#endif
}

// ln x = k ln 2 + 2 atanh(s), x = 2^k m with m in [sqrt(1/2), sqrt(2)),
// s = (m - 1) / (m + 1).  s is kept to twice the precision (s + ds), and the
// leading terms k ln 2 (exact: 42 bits) and 2 s are added without error, so
// the result rounds almost correctly.
EMS_HD double pos_log(double x) {
  constexpr double kLn2Hi = 0x1.62e42fefa3800p-1, kLn2Lo = 0x1.ef35793c76730p-45;
  const uint64_t ix = bits_of(x);
  const int32_t t = (int32_t)(uint32_t)(ix >> 32) - 0x3fe6a09e;
  const int32_t k = t >> 20;
  const double m = double_of(ix - ((uint64_t)(uint32_t)(t & (int32_t)0xfff00000) << 32));
  const double f = m - 1.0, d = m + 1.0, dl = m - (d - 1.0);
  double y = rcp_estimate(d);
  y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
  y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
  const double s = f * y;
  const double ds = __builtin_fma(-s, dl, __builtin_fma(-s, d, f)) * y;
  const double z = s * s;
  double p = 0x1.2f097e703f9f9p-3;
  p = __builtin_fma(p, z, 0x1.39a15752c4a19p-3);
  p = __builtin_fma(p, z, 0x1.74664290191ddp-3);
  p = __builtin_fma(p, z, 0x1.c71c51f88c0c5p-3);
  p = __builtin_fma(p, z, 0x1.24924942048f4p-2);
  p = __builtin_fma(p, z, 0x1.999999997fc70p-2);
  p = __builtin_fma(p, z, 0x1.5555555555593p-1);
  const double kd = (double)k, hi = kd * kLn2Hi, s2 = s + s;
  const double w = hi + s2, e = (hi - w) + s2;
  const double lo = __builtin_fma(kd, kLn2Lo, __builtin_fma(ds, 2.0, e));
  return w + __builtin_fma(s * z, p, lo);
}

// e^x = 2^k e^r, |r| <= ln 2 / 2
EMS_HD double ranged_exp(double x) {
  constexpr double kLog2e = 0x1.71547652b82fep+0;
  constexpr double kLn2Hi = 0x1.62e42fefa3800p-1, kLn2Lo = 0x1.ef35793c76730p-45;
  const double k = __builtin_rint(x * kLog2e);
  const double rh = __builtin_fma(-k, kLn2Hi, x), rt = -k * kLn2Lo;
  const double r = rh + rt, rl = (rh - r) + rt;
  const double q = r * r;
  // (e^r - 1 - r) / r^2, even and odd coefficients apart (half the chain)
  double a = 0x1.28b043fd19902p-22, b = 0x1.af85aa0749158p-26;
  a = __builtin_fma(a, q, 0x1.a019969947856p-16);
  b = __builtin_fma(b, q, 0x1.71dddfb9955b3p-19);
  a = __builtin_fma(a, q, 0x1.6c16c185a549bp-10);
  b = __builtin_fma(b, q, 0x1.a01a01bae89d2p-13);
  a = __builtin_fma(a, q, 0x1.5555555550039p-5);
  b = __builtin_fma(b, q, 0x1.111111110d62dp-7);
  a = __builtin_fma(a, q, 0x1.000000000000bp-1);
  b = __builtin_fma(b, q, 0x1.5555555555561p-3);
  // 1 + r and what its rounding lost
  const double h = 1.0 + r, hl = (1.0 - h) + r;
  const double p = __builtin_fma(__builtin_fma(b, r, a), q, rl);
  return __builtin_ldexp(h + (hl + p), (int)k);
}

// sine and cosine of 2 pi u, u in [0, 1]: the nearest quarter turn is taken
// off exactly, the rest (at most an eighth of a turn) by polynomials
EMS_HD void sincos_turn(double u, double* sn, double* cs) {
  const double q = __builtin_rint(4.0 * u);
  const double th = __builtin_fma(-0.25, q, u) * 0x1.921fb54442d18p+2;
  const double z = th * th;
  double a = 0x1.5d92451995283p-33, b = -0x1.8fadd03e3cbe6p-37;
  a = __builtin_fma(a, z, -0x1.ae5e63c6f5ddcp-26);
  b = __builtin_fma(b, z, 0x1.1ee9ea6c54044p-29);
  a = __builtin_fma(a, z, 0x1.71de3574b0bddp-19);
  b = __builtin_fma(b, z, -0x1.27e4f807d564ap-22);
  a = __builtin_fma(a, z, -0x1.a01a019c0e3eep-13);
  b = __builtin_fma(b, z, 0x1.a01a019caef23p-16);
  a = __builtin_fma(a, z, 0x1.111111110f861p-7);
  b = __builtin_fma(b, z, -0x1.6c16c16c15162p-10);
  a = __builtin_fma(a, z, -0x1.5555555555549p-3);
  b = __builtin_fma(b, z, 0x1.555555555554cp-5);
  const double s = __builtin_fma(th * z, a, th);
  // 1 - z/2 and what its rounding lost
  const double h = __builtin_fma(z, -0.5, 1.0), hl = __builtin_fma(z, -0.5, 1.0 - h);
  const double c = h + __builtin_fma(z * z, b, hl);
  const int n = (int)q;
  const double x = (n & 1) ? c : s, y = (n & 1) ? s : c;
  *sn = (n & 2) ? -x : x;
  *cs = ((n + 1) & 2) ? -y : y;
}

// square root, and quotients of numbers whose magnitudes are far from the ends
// of the range (2^+-400, in single precision 2^+-50): the compiler's own
// sequences without the scaling that the ends need (22 and 11 instructions,
// here 13 and 8; a further quotient by the same divisor 3 to 5), so the
// results are the correctly rounded ones.  The root's are from 2^-968 up, and
// zero's and infinity's; below, where its last residual is rounded, it is
// within a unit in the last place down to the smallest normal number and keeps
// 40 bits below that.
#if defined(__HIP_DEVICE_COMPILE__)
EMS_HD double plain_sqrt(double v) {
  const double y = __builtin_amdgcn_rsq(v);
  double g = v * y, h = 0.5 * y;
  const double e = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, e, g);
  h = __builtin_fma(h, e, h);
  g = __builtin_fma(__builtin_fma(-g, g, v), h, g);
  g = __builtin_fma(__builtin_fma(-g, g, v), h, g);
  return __builtin_amdgcn_class(v, 0x260) ? v : g;  // (zeros and infinity)
}
template <class R>
struct Recip;
template <>
struct Recip<double> {
  double d, y;
  EMS_HD explicit Recip(double v) : d(v), y(__builtin_amdgcn_rcp(v)) {
    y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
    y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
  }
  EMS_HD double of(double a) const {
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-d, q, a), y, q);
  }
};
template <>
struct Recip<float> {
  float d, y;
  EMS_HD explicit Recip(float v) : d(v), y(__builtin_amdgcn_rcpf(v)) {
    y = __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
  }
  EMS_HD float of(float a) const {
    float q = a * y;
    q = __builtin_fmaf(__builtin_fmaf(-d, q, a), y, q);
    return __builtin_fmaf(__builtin_fmaf(-d, q, a), y, q);
  }
};
#else
template <class R>
struct Recip {
  R d;
  EMS_HD explicit Recip(R v) : d(v) {}
  EMS_HD R of(R a) const { return a / d; }
};
#endif
template <class R>
EMS_HD R quot(R a, R b) {
  return Recip<R>(b).of(a);
}

}  // namespace ems
