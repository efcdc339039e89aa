// FP64 elementary functions for arguments whose range the caller knows: no
// scaling of denormals, no infinities, NaN only through.  The library's
// versions spend a third to a half of their instructions on those.
//
//   m64_rcp      1/x: the hardware reciprocal and two Newton steps
//   m64_root     sqrt(x) and 1/sqrt(x): the hardware reciprocal square root,
//                one coupled (Goldschmidt) step, and a correction by the
//                exact remainder x - g^2
//   m64_log      log(x) from a 33-entry table: x = m 2^e, c = 1/(1 + k/32)
//                rounded to FP32 with 1 + k/32 nearest to m, so that
//                log x = e ln 2 - log c + log1p(m c - 1), |m c - 1| <= 1/64; the
//                large parts are multiples of 2^-34 and add exactly
//   m64_sincos   sine and cosine of 2 pi (k + 1/2) 2^-32 from a 65-entry
//                table of the angles j/64 and the addition theorem, the
//                remainder (at most 2 pi/128) by its Taylor series
#pragma once

#include "common.h"

namespace vgx {

__device__ __forceinline__ double m64_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  return fma(y, fma(-x, y, 1.0), y);
}

struct Root64 { double g, y; };  // sqrt(x); 1/sqrt(x) to about 2^-46

__device__ __forceinline__ Root64 m64_root(double x) {
  const double y0 = __builtin_amdgcn_rsq(x);
  double g = x * y0, h = 0.5 * y0;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, x), h, g);
  return {g, 2.0 * h};
}

// 1/sqrt(x) to the last bits
__device__ __forceinline__ double m64_rsqrt(double x) {
  const Root64 k = m64_root(x);
  return fma(k.y, fma(-k.g, k.y, 1.0), k.y);
}

// The tables, in LDS.
struct M64Tables {
  struct Log { float c, lo; double hi; } log[33];  // c, and -log c = hi + lo
  double2 sc[65];                                  // sine and cosine of 2 pi j/64, FP64 ...
  float2 sc_lo[65];                                // ... and what is left of them
};

// sin(2 pi j/64), j = 0 .. 16, rounded to FP64, and the rest (computed with
// 60 decimal digits).
struct M64Sine { double hi; float lo; };
__device__ const M64Sine kM64Sine[17] = {
    {0.0, 0.0f}, {0x1.917a6bc29b42cp-4, -0x1.e2718e0000000p-60f}, {0x1.8f8b83c69a60bp-3, -0x1.26d19c0000000p-57f},
    {0x1.294062ed59f06p-2, -0x1.5d28da0000000p-56f}, {0x1.87de2a6aea963p-2, -0x1.72cede0000000p-57f},
    {0x1.e2b5d3806f63bp-2, 0x1.e0d8920000000p-58f}, {0x1.1c73b39ae68c8p-1, 0x1.b25dd20000000p-55f},
    {0x1.44cf325091dd6p-1, 0x1.8076a20000000p-57f}, {0x1.6a09e667f3bcdp-1, -0x1.bdd3420000000p-55f},
    {0x1.8bc806b151741p-1, -0x1.2c5e120000000p-55f}, {0x1.a9b66290ea1a3p-1, 0x1.9f630e0000000p-60f},
    {0x1.c38b2f180bdb1p-1, -0x1.6e0b180000000p-56f}, {0x1.d906bcf328d46p-1, 0x1.457e620000000p-56f},
    {0x1.e9f4156c62ddap-1, 0x1.760b1e0000000p-55f}, {0x1.f6297cff75cb0p-1, 0x1.5621720000000p-56f},
    {0x1.fd88da3d12526p-1, -0x1.87df640000000p-55f}, {1.0, 0.0f}};

// ln 2 = kLn2Hi + kLn2Lo: the multiple of 2^-34 nearest to it, and the rest
// rounded to FP32 (the table's last entry has the same two parts, so that
// x just below 1 = 2^-1 (2 - ...) cancels exactly)
constexpr double kLn2Hi = 11908177887.0 * 0x1p-34;
constexpr float kLn2Lo = 0x1.1cf79ap-36f;

// Fills the tables (every thread of the workgroup; the caller synchronises).
__device__ inline void m64_tables(M64Tables& t) {
  for (int k = threadIdx.x; k < 33; k += blockDim.x) {
    const float c = 1.0f / (1.0f + (float)k / 32.0f);
    const double l = -log((double)c);
    const double hi = k == 32 ? kLn2Hi : rint(l * 0x1p34) * 0x1p-34;
    t.log[k] = {c, k == 32 ? kLn2Lo : (float)(l - hi), hi};
  }
  for (int k = threadIdx.x; k < 65; k += blockDim.x) {
    auto sine = [](int j, double& hi, float& lo) {  // the quarter wave, mirrored
      const int r = j & 31;
      const M64Sine v = kM64Sine[r <= 16 ? r : 32 - r];
      hi = j & 32 ? -v.hi : v.hi;
      lo = j & 32 ? -v.lo : v.lo;
    };
    sine(k, t.sc[k].x, t.sc_lo[k].x);
    sine(k + 16, t.sc[k].y, t.sc_lo[k].y);
  }
}

__device__ __forceinline__ double m64_log(const M64Tables& t, double x) {
  const int hi = __double2hiint(x);
  const M64Tables::Log l = t.log[((hi & 0xFFFFF) + 0x4000) >> 15];
  const double m = __hiloint2double((hi & 0xFFFFF) | 0x3FF00000, __double2loint(x));
  const double e = (double)((hi >> 20) - 1023);
  const double r = fma(m, (double)l.c, -1.0);
  double p = fma(r, 1.0 / 9, -1.0 / 8);
  p = fma(r, p, 1.0 / 7);
  p = fma(r, p, -1.0 / 6);
  p = fma(r, p, 1.0 / 5);
  p = fma(r, p, -1.0 / 4);
  p = fma(r, p, 1.0 / 3);
  p = fma(r, p, -1.0 / 2);
  p = fma(r * r, p, fma(e, (double)kLn2Lo, (double)l.lo));
  return fma(e, kLn2Hi, l.hi) + (r + p);
}

__device__ __forceinline__ void m64_sincos(const M64Tables& t, uint32_t k, double& sn, double& cs) {
  const uint32_t j = (k >> 26) + ((k >> 25) & 1);  // nearest of 64 steps
  const double2 a = t.sc[j];
  const float2 b = t.sc_lo[j];
  // (k + 1/2 - j 2^26) 2^-32 turns, exact
  const double d = ((double)(int32_t)(k - (j << 26)) + 0.5) * (6.283185307179586477 * 0x1p-32);
  const double d2 = d * d;
  double s = fma(d2, -1.0 / 5040, 1.0 / 120);
  s = fma(d2, s, -1.0 / 6);
  s = fma(d * d2, s, d);              // sin d
  double c = fma(d2, 1.0 / 40320, -1.0 / 720);
  c = fma(d2, c, 1.0 / 24);
  c = fma(d2, c, -0.5) * d2;          // cos d - 1
  sn = a.x + fma(a.x, c, fma(a.y, s, (double)b.x));
  cs = a.y + fma(a.y, c, fma(-a.x, s, (double)b.y));
}

}  // namespace vgx
