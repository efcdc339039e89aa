// Device integrands of libvgx.  Each integrand is a small struct with
//   static constexpr int lds_doubles(...)  -- extra LDS it stages (in doubles)
//   __device__ void stage(double* lds)      -- cooperative LDS staging
//   __device__ double eval(const double (&x)[D]) const
// Parameters live in a fixed-size by-value kernel argument.
#pragma once

#include "common.h"

namespace vgx {

constexpr int MAX_PARAMS = 2 * VGX_MAX_DIM + 4;

struct IntegrandParams {
  double p[MAX_PARAMS];
};

// Integrands without LDS staging share this no-op.
struct NoStage {
  static constexpr bool kStage = false;
  __device__ __forceinline__ void stage(float*) {}
};

// exp(-e) for e >= 0 and not NaN: n = round(-e log2 e), r = -e - n ln 2 (ln 2
// in two parts), a polynomial of degree 11 on |r| <= ln 2 / 2 (the interpolant
// of (exp r - 1 - r)/r^2 in ten Chebyshev nodes, computed with 60 digits:
// relative error 1.6e-17), scaled by 2^n, which underflows as it should
// (e > 1000 gives the zero of e = 1000).  The library's exp tests for
// overflow, underflow and NaN: 6 instructions more.
__device__ __forceinline__ double exp_neg(double e) {
  e = fmin(e, 1000.0);
  const double n = rint(e * -0x1.71547652b82fep+0);
  const double r = fma(n, -0x1.cf79abc9e3b3ap-40, fma(n, -0x1.62e42fefa0000p-1, -e));
  double p = fma(r, 0x1.af38a9b0ec855p-26, 0x1.289185613a3d6p-22);
  p = fma(r, p, 0x1.71de0dae63bb3p-19);
  p = fma(r, p, 0x1.a019b90d2ae7ap-16);
  p = fma(r, p, 0x1.a01a01a7c41d5p-13);
  p = fma(r, p, 0x1.6c16c1788bd90p-10);
  p = fma(r, p, 0x1.11111111109b3p-7);
  p = fma(r, p, 0x1.5555555553d63p-5);
  p = fma(r, p, 0x1.5555555555556p-3);
  p = fma(r, p, 0x1.0000000000001p-1);
  p = fma(r, p, 1.0);
  p = fma(r, p, 1.0);
  return __builtin_amdgcn_ldexp(p, (int)n);
}

// prod_j N(x_j; c_j, s_j), each factor normalised on R.  One exp of the
// summed exponent; the normalisation prod 1/(s_j sqrt(2 pi)) is folded on
// the host into p[2D] so that the device does only the data-dependent part.
template <int D, typename R>
struct Gauss : NoStage {
  using Real = R;
  IntegrandParams prm;  // [c_0..c_{D-1}, 1/(s_j sqrt 2) .., norm]
  __device__ __forceinline__ R exponent(const double (&x)[D]) const {
    R e = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      // z = (x - c) k as x k - c k (one FMA; c k is loop-invariant)
      const R k = (R)prm.p[D + j];
      const R z = fma((R)x[j], k, -((R)prm.p[j] * k));
      e = fma(z, z, e);
    }
    return e;
  }
  __device__ __forceinline__ double eval(const double (&x)[D]) const {
    return (double)((R)prm.p[2 * D] * exp(-exponent(x)));
  }
  // At a point the grid map made: a NaN exponent comes from the parameters
  // alone, and then the norm is NaN too (set on the host).
  __device__ __forceinline__ double eval_inside(const double (&x)[D]) const {
    if constexpr (sizeof(R) == 8) return prm.p[2 * D] * exp_neg(exponent(x));
    else return eval(x);
  }
};

// Genz oscillatory: cos(2 pi w_1 + sum_j c_j x_j).  p = [2 pi w_1, c_0 ..].
template <int D, typename R>
struct GenzOsc : NoStage {
  using Real = R;
  IntegrandParams prm;
  __device__ __forceinline__ double eval(const double (&x)[D]) const {
    R a = (R)prm.p[0];
#pragma unroll
    for (int j = 0; j < D; ++j) a = fma((R)prm.p[1 + j], (R)x[j], a);
    return (double)cos(a);
  }
};

// Genz product peak: prod_j (c_j^-2 + (x_j - w_j)^2)^-1.
// p = [w_0..w_{D-1}, c_0^-2 .. c_{D-1}^-2].
template <int D, typename R>
struct GenzPeak : NoStage {
  using Real = R;
  IntegrandParams prm;
  __device__ __forceinline__ double eval(const double (&x)[D]) const {
    R den = 1;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const R z = (R)x[j] - (R)prm.p[j];
      den *= fma(z, z, (R)prm.p[D + j]);
    }
    return (double)((R)1 / den);
  }
};

}  // namespace vgx
