// Sine and cosine of a phase of any size.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

namespace pt {

constexpr double kHalfPi = 1.57079632679489661923;        // pi/2, leading double
constexpr double kHalfPiLo = 6.123233995736766036e-17;    // and the next one

// The remainder of a large |x| (2^45 and more) by the nearest multiple of pi/2, and
// that multiple mod 4: Payne and Hanek's reduction in integers.  x = m 2^e, so
// x / (2 pi) mod 1 is m times the bits of 1/(2 pi) from the e-th on; 192 of them
// leave 139 bits of the fraction, and no double lies nearer than 2^-64 to a
// multiple of a quarter turn.  NaN for infinities and NaN.
__host__ __device__ inline double far_remainder(double x, int &k) {
  // 64 zeros, then 1/(2 pi)
  static constexpr uint64_t kInv2Pi[20] = {
      0, 0x28BE60DB9391054Aull, 0x7F09D5F47D4D3770ull, 0x36D8A5664F10E410ull,
      0x7F9458EAF7AEF158ull, 0x6DC91B8E909374B8ull, 0x01924BBA82746487ull, 0x3F877AC72C4A69CFull,
      0xBA208D7D4BAED121ull, 0x3A671C09AD17DF90ull, 0x4E64758E60D4CE7Dull, 0x272117E2EF7E4A0Eull,
      0xC7FE25FFF7816603ull, 0xFBCBC462D6829B47ull, 0xDB4D9FB3C9F2C26Dull, 0xD3D18FD9A797FA8Bull,
      0x5D49EEB1FAF97C5Eull, 0xCF41CE7DE294A4BAull, 0x9AFED7EC47E35742ull, 0x1580CC11BF1EDAEAull};
  using u128 = unsigned __int128;
  uint64_t b;
  memcpy(&b, &x, 8);
  const uint64_t m = (b & 0xFFFFFFFFFFFFFull) | 0x10000000000000ull;
  const int at = (int)(b >> 52 & 0x7FF) - 1075 + 64;   // first bit: 57 .. 1036
  const uint64_t *t = kInv2Pi + (at >> 6);
  const int sh = at & 63;
  const uint64_t a2 = t[0] << sh | t[1] >> 1 >> (63 - sh);
  const uint64_t a1 = t[1] << sh | t[2] >> 1 >> (63 - sh);
  const uint64_t a0 = t[2] << sh | t[3] >> 1 >> (63 - sh);
  const u128 lo = (u128)m * a1 + (uint64_t)((u128)m * a0 >> 64);
  const uint64_t f0 = (uint64_t)lo, f1 = m * a2 + (uint64_t)(lo >> 64);   // the fraction of a turn
  const uint64_t n = (f1 + (1ull << 61)) >> 62;   // nearest quarter, 0 .. 3 (4: a whole turn, wrapped)
  const int64_t d = (int64_t)(f1 - (n << 62));
  const double turn = 6.283185307179586476925286766559;
  const double r = ((double)d * 0x1p-64 + (double)f0 * 0x1p-128) * turn + (x - x);
  const bool minus = b >> 63;
  k = (int)(minus ? 0 - n : n) & 3;
  return minus ? -r : r;
}

constexpr double kFarPhase = 0x1p45;

// sin and cos of x: x less the nearest multiple n of pi/2 by two fused steps (the
// first is exact and the two doubles of pi/2 leave n 2^-109), then the Taylor series
// to r^15 and r^16 on |r| <= pi/4, whose next terms are below half a unit in the
// last place.  FAR takes |x| >= kFarPhase by far_remainder; without it |x| has to be
// below (the branch takes 30 registers, which the TOA pass does not have: 246 us
// a launch with it at 45 pulsars, 17 harmonics with DM and 256 chains, 198 without).  The library's
// sincos had most of the instructions and registers of its CW terms.
template <bool FAR>
__host__ __device__ inline void sincos_phase(double x, double &sn, double &cs) {
  const double n = rint(x * 0.63661977236758134308);
  double r = fma(-n, kHalfPi, x);
  r = fma(-n, kHalfPiLo, r);
  int k = (int)fma(-4.0, floor(0.25 * n), n);
  if (FAR && __builtin_expect(!(fabs(x) < kFarPhase), 0)) r = far_remainder(x, k);
  const double z = r * r;
  double ps = -1.0 / 1307674368000.0, pc = 1.0 / 20922789888000.0;
  ps = fma(ps, z, 1.0 / 6227020800.0);
  ps = fma(ps, z, -1.0 / 39916800.0);
  ps = fma(ps, z, 1.0 / 362880.0);
  ps = fma(ps, z, -1.0 / 5040.0);
  ps = fma(ps, z, 1.0 / 120.0);
  ps = fma(ps, z, -1.0 / 6.0);
  pc = fma(pc, z, -1.0 / 87178291200.0);
  pc = fma(pc, z, 1.0 / 479001600.0);
  pc = fma(pc, z, -1.0 / 3628800.0);
  pc = fma(pc, z, 1.0 / 40320.0);
  pc = fma(pc, z, -1.0 / 720.0);
  pc = fma(pc, z, 1.0 / 24.0);
  pc = fma(pc, z, -0.5);
  const double s = fma(r * z, ps, r), c = fma(pc, z, 1.0);
  const double a = (k & 1) ? c : s, b = (k & 1) ? s : c;
  sn = (k & 2) ? -a : a;
  cs = (k == 1 || k == 2) ? -b : b;
}

}  // namespace pt
