// euler.hpp -- device-side pieces of the hyperbolic step: the maximum wave
// speed bound and the pieces of the limiter line search (Sec. 3.1, 3.3).
#pragma once

#include <hip/hip_runtime.h>

namespace ns {

// FP64 reciprocal and square root from the hardware seeds (v_rcp_f64,
// v_rsq_f64) refined by Newton / Goldschmidt iterations: 5 and 10
// instructions instead of the 10-16 of the IEEE-exact sequences, which the
// VALU-bound graph-viscosity sweep spends most of its division and square
// root time in.  For positive normal arguments (the only ones they get:
// densities, pressures, |c_ij|, sums of positive terms) the results agree
// with the correctly rounded ones to within an ulp (on 2^20 samples over
// 2^-20 .. 2^20 both were exact).  fast_sqrt(0) is 0: the seed is taken at
// max(x, 2^-1000), so x * seed stays 0 and every later step keeps it there
// (|c_ii| = 0 on interior rows is an argument it does get).
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

__device__ __forceinline__ double fast_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(fmax(x, 0x1p-1000));  // ~ x^(-1/2)
  double g = x * y, h = 0.5 * y;             // ~ x^(1/2), x^(-1/2)/2
  double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  return fma(fma(-g, g, x), h, g);           // one residual correction
}

// Exponent (gamma-1)/(2 gamma) of the two-rarefaction pressure and its
// inverse; for gamma = 7/5 the inverse is the integer 7.
struct Gas {
  double gamma;
  double gm1;      // gamma - 1
  double ex;       // (gamma - 1) / (2 gamma)
  double inv_ex;   // 2 gamma / (gamma - 1)
  double cg;       // (gamma + 1) / (2 gamma)
  double lgm1;     // log(gamma - 1)
  int seven;       // 1 when gamma == 7/5
};

// SEV: 1 when gamma == 7/5 is fixed at compile time (integer powers and the
// polynomial entropy test), 0 for a general gamma (pow).  The kernels are
// instantiated for both and the host picks by Gas::seven, so the gamma = 7/5
// kernels carry no pow code at all.
template <int SEV>
__device__ __forceinline__ double pow_inv_ex(const Gas &g, double x) {
  if constexpr (SEV) {
    const double x2 = x * x;
    const double x4 = x2 * x2;
    return x4 * x2 * x;
  }
  return pow(x, g.inv_ex);
}

// Guaranteed upper bound on the largest wave speed of the 1D Riemann problem
// with left state (uL, pL, aL) and right state (uR, pR, aR) along the unit
// direction n (u = v.n).  bL = aL pL^(-ex), bR likewise (precomputed per
// node).  Two-rarefaction bound on the star pressure, valid for
// 1 < gamma <= 5/3, inserted in the extreme shock/rarefaction speeds.
template <int SEV>
__device__ __forceinline__ double lambda_max(const Gas &g, double uL, double pL,
                                             double aL, double bL, double uR,
                                             double pR, double aR, double bR) {
#pragma clang fp contract(off)  // the same bits in every kernel
  const double num = fma(-0.5 * g.gm1, uR - uL, aL + aR);
  double ptr = 0.0;
  if (num > 0.0) ptr = pow_inv_ex<SEV>(g, num * fast_rcp(bL + bR));
  const double sL = fast_sqrt(fma(g.cg, fmax(fma(ptr, fast_rcp(pL), -1.0), 0.0), 1.0));
  const double sR = fast_sqrt(fma(g.cg, fmax(fma(ptr, fast_rcp(pR), -1.0), 0.0), 1.0));
  const double l1 = fma(-aL, sL, uL), l3 = fma(aR, sR, uR);
  return fmax(fmax(-l1, 0.0), fmax(l3, 0.0));
}

// ---------------------------------------------------------------------------
// FP32 evaluation of the same bound for gamma = 7/5 (mixed-precision mode
// with FP32 arithmetic).  Approximate reciprocal and square root (1 ulp) are
// enough: the caller inflates the result by 2^-16 relative
// (kLambdaInflate) and uses it only where the rounding error is provably
// below that, i.e. where
//   (a) neither extreme speed u_L - a_L S_L, u_R + a_R S_R cancels by more
//       than a factor 3: max(|u| + a S) over both sides <= 3 lambda, and
//   (b) where a side is in the shock branch (S > 1), the star-pressure
//       numerator a_L + a_R - (gamma-1)/2 (u_R - u_L) cancels by at most a
//       factor 2 against a_L + a_R + (gamma-1)/2 (|u_L| + |u_R|) (its
//       relative error is amplified 7-fold by the power).
// With u = 2^-24 (the inputs rounded to FP32, the normal velocities formed
// in FP32): the numerator carries <= 8u relative, the quotient by b_L + b_R
// <= 12u, the 7th power <= 88u, p*/p <= 91u, each S <= 49u (dS/S <=
// d(p*/p)/2 since 1 - (gamma+1)/(2 gamma) > 0), each a S <= 51u, so each
// extreme speed is off by <= 52u (|u| + a S) <= 156u lambda, and with |c_ij|
// (3u) the product lambda |c_ij| by <= 160u < 2^-16 = 256u.  Elsewhere *ok
// is false and the caller evaluates lambda_max in FP64.
constexpr double kLambdaInflate = 1.0 + 1.0 / 65536.0;

__device__ __forceinline__ float lambda_max_f32(const Gas &g, float uL, float pL, float aL,
                                               float bL, float uR, float pR, float aR,
                                               float bR, bool *ok) {
  const float gm1 = (float)g.gm1, cg = (float)g.cg;
  const float num = aL + aR - 0.5f * gm1 * (uR - uL);
  float ptr = 0.0f;
  if (num > 0.0f) {
    const float x = num * __builtin_amdgcn_rcpf(bL + bR);
    const float x2 = x * x;
    const float x4 = x2 * x2;
    ptr = x4 * x2 * x;  // x^(2 gamma/(gamma-1)) = x^7
  }
  const float rL = ptr * __builtin_amdgcn_rcpf(pL), rR = ptr * __builtin_amdgcn_rcpf(pR);
  const float SL = __builtin_amdgcn_sqrtf(1.0f + cg * fmaxf(rL - 1.0f, 0.0f));
  const float SR = __builtin_amdgcn_sqrtf(1.0f + cg * fmaxf(rR - 1.0f, 0.0f));
  const float eL = aL * SL, eR = aR * SR;
  const float lam = fmaxf(fmaxf(eL - uL, 0.0f), fmaxf(uR + eR, 0.0f));
  const float M = fmaxf(fabsf(uL) + eL, fabsf(uR) + eR);
  const bool shock = rL > 0.999f || rR > 0.999f;
  *ok = M <= 3.0f * lam &&
        (!shock || aL + aR + 0.5f * gm1 * (fabsf(uL) + fabsf(uR)) <= 2.0f * num);
  return lam;
}

// x^(7/5) for x > 0: x z with z = x^(2/5) from two Newton steps for z^5 = x^2
// on an FP32 start (relative error e -> 2 e^2: 1e-6, 2e-12, rounding), x
// scaled by a power of 2^5 into the FP32 range first.  The last step's
// residual is formed with the rounding errors of its products and its
// correction enters the final product, so the result is within 0.54 ulp, as
// close as pow.  0 and infinity as pow.  A quarter
// of pow's instructions.
__device__ __forceinline__ double pow_seven_fifths(double x) {
#pragma clang fp contract(off)  // the same bits in every kernel
  const int k = (__builtin_amdgcn_frexp_exp(x) * 205) >> 10;  // about e / 5
  const double y = ldexp(x, -5 * k), y2 = y * y;
  double z = (double)__builtin_amdgcn_exp2f(0.4f * __builtin_amdgcn_logf((float)y));
  {
    const double z2 = z * z, z4 = z2 * z2;
    z = fma(fma(-z4, z, y2), 0.2 * fast_rcp(z4), z);
  }
  const double z2 = z * z, z4 = z2 * z2;
  const double z4e = fma(z2, z2, -z4) + 2.0 * z2 * fma(z, z, -z2);
  const double rest = fma(-z4, z, y2) + (fma(y, y, -y2) - z4e * z);
  const double r = ldexp(fma(y, z, y * (rest * (0.2 * fast_rcp(z4)))), 7 * k);
  return x == 0.0 || x == INFINITY ? x : r;
}

// psi(l) = eps(u + l P) - phi_min rho(u + l P)^gamma and its derivative.
// power(rho, l) is rho^gamma.
template <int DIM, class Power>
__device__ __forceinline__ double psi_with(const Gas &g, const double *u,
                                           const double *P, double l,
                                           double phi_min, double *dpsi,
                                           const Power &power) {
#pragma clang fp contract(off)  // the same bits in every kernel
  const double r = fma(l, P[0], u[0]);
  double m2 = 0.0, mp = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    const double mk = fma(l, P[1 + k], u[1 + k]);
    m2 = fma(mk, mk, m2);
    mp = fma(mk, P[1 + k], mp);
  }
  const double E = fma(l, P[DIM + 1], u[DIM + 1]);
  const double ir = 1.0 / r;
  const double eps = fma(-0.5 * m2, ir, E);
  const double rg = power(r, l);
  if (dpsi) {
    // d eps/dl = P_E - (m.P_m)/rho + |m|^2 P_rho / (2 rho^2)
    const double deps = fma(0.5 * m2 * ir * ir, P[0], fma(-mp, ir, P[DIM + 1]));
    *dpsi = fma(-phi_min * g.gamma * rg * ir, P[0], deps);
  }
  return fma(-phi_min, rg, eps);
}
template <int DIM, int SEV>
__device__ __forceinline__ double psi_eval(const Gas &g, const double *u,
                                           const double *P, double l,
                                           double phi_min, double *dpsi) {
  return psi_with<DIM>(g, u, P, l, phi_min, dpsi, [&](double r, double) {
    return SEV ? pow_seven_fifths(r) : pow(r, g.gamma);
  });
}

// Is u + l P inside the entropy bound Phi >= phi_min?  For gamma = 7/5 the
// test eps >= phi_min rho^(7/5) is taken division- and pow-free as
// (rho eps)^5 >= phi_min^5 rho^12 with rho eps = rho E - |m|^2/2 (both sides
// are non-negative exactly when eps >= 0); pmin5 = phi_min^5.  A general gamma
// asks log q = log phi_min + (gamma + 1) log rho - log(rho eps) <= 0 in FP32
// first, whose error is below 1e-6 of its terms' sizes, and pow only where that
// leaves it open.
template <int DIM, int SEV>
__device__ __forceinline__ bool entropy_ok(const Gas &g, const double *u,
                                           const double *P, double l,
                                           double phi_min, double pmin5) {
  // no fused multiply-adds of the compiler's choosing: a pair's two rows
  // evaluate the same test in different kernels and must agree bit for bit
#pragma clang fp contract(off)
  const double r = u[0] + l * P[0];
  double m2 = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    const double mk = u[1 + k] + l * P[1 + k];
    m2 += mk * mk;
  }
  const double E = u[DIM + 1] + l * P[DIM + 1];
  if constexpr (SEV) {
    const double A = r * E - 0.5 * m2;
    if (!(A > 0.0)) return false;
    const double A2 = A * A;
    const double r2 = r * r, r4 = r2 * r2, r8 = r4 * r4;
    return A2 * A2 * A >= pmin5 * (r8 * r4);
  }
  else {
    const float g1 = (float)(g.gamma + 1.0), lp = __builtin_amdgcn_logf((float)phi_min);
    const float lr = g1 * __builtin_amdgcn_logf((float)r);
    const float la = __builtin_amdgcn_logf((float)(r * E - 0.5 * m2));
    const float lq = lp + lr - la, size = fabsf(lp) + fabsf(lr) + fabsf(la) + g1 + 2.0f;
    // (false also for infinities and NaN: arguments beyond FP32, bounds <= 0)
    if (fabsf(lq) > 1e-6f * size && size < 1e4f) return lq < 0.0f;
    return E - 0.5 * m2 / r - phi_min * pow(r, g.gamma) >= 0.0;
  }
}

// Root of psi in (a, b) with psi(a) >= 0 > psi(b).  psi is concave in l, so
// from the feasible end a the chord's root stays feasible and from the
// infeasible end b the tangent's root stays infeasible: both ends move towards
// the root at once.  Every candidate is checked by evaluating psi, so the
// returned end is feasible even under round-off.  Stops when the bracket is
// below 1e-14 (l is dimensionless, in [0,1]).
template <int DIM, int SEV>
__device__ __forceinline__ double entropy_root(const Gas &g, const double *u,
                                            const double *P, double b,
                                            double phi_min) {
#pragma clang fp contract(off)  // the same bits in every kernel
  double a = 0.0;
  double fa = psi_eval<DIM, SEV>(g, u, P, 0.0, phi_min, nullptr);
  double dfb;
  double fb = psi_eval<DIM, SEV>(g, u, P, b, phi_min, &dfb);
  if (fa < 0.0) return 0.0;
  if (fb >= 0.0) return b;
  for (int it = 0; it < 24 && b - a > 1e-14; ++it) {
    const double w0 = b - a;
    const double xs = a - fa * (b - a) / (fb - fa);
    if (xs > a && xs < b) {
      const double f = psi_eval<DIM, SEV>(g, u, P, xs, phi_min, nullptr);
      if (f >= 0.0) { a = xs; fa = f; }
      else { b = xs; fb = f; dfb = 0.0; }
    }
    if (dfb < 0.0) {
      const double xn = b - fb / dfb;
      if (xn > a && xn < b) {
        double d;
        const double f = psi_eval<DIM, SEV>(g, u, P, xn, phi_min, &d);
        if (f < 0.0) { b = xn; fb = f; dfb = d; }
        else { a = xn; fa = f; }
      }
    }
    if (b - a > 0.5 * w0) {
      const double xm = 0.5 * (a + b);
      double d;
      const double f = psi_eval<DIM, SEV>(g, u, P, xm, phi_min, &d);
      if (f >= 0.0) { a = xm; fa = f; }
      else { b = xm; fb = f; dfb = d; }
    }
    if (dfb == 0.0 && b - a > 1e-14) psi_eval<DIM, SEV>(g, u, P, b, phi_min, &dfb);
  }
  return a;
}

// Root of the entropy bound for gamma = 7/5 (the last Newton step, of at most
// 1e-9, is taken in full precision) on the polynomial form of the test: with rho(l) = rho + l P_rho and A(l) = rho(l) E(l) -
// |m(l)|^2/2 = a0 + a1 l + a2 l^2 (rho(l) eps(l)) the bound holds where
// q = phi_min^5 rho^12 / A^5 <= 1.  Newton on log q, whose slope changes
// little over (0, b) (on A^5 - phi_min^5 rho^12, twelfth powers, one lane in
// a hundred took over 30 steps; here 4, and the slowest lane decides), kept
// inside the bracket [lo, hi] (q(lo) <= 1 < q(hi)) by bisection.  No division
// by state values, no pow: some 40 instructions a step.
template <int DIM>
__device__ __forceinline__ double entropy_root_seven(const double *u,
                                                    const double *P, double b,
                                                    double pmin5) {
#pragma clang fp contract(off)  // the same bits in every kernel
  const double r0 = u[0], pr = P[0];
  double m0p = 0.0, pm2 = 0.0, m02 = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    m0p = fma(u[1 + k], P[1 + k], m0p);
    pm2 = fma(P[1 + k], P[1 + k], pm2);
    m02 = fma(u[1 + k], u[1 + k], m02);
  }
  const double E0 = u[DIM + 1], pE = P[DIM + 1];
  const double a0 = fma(r0, E0, -0.5 * m02);
  const double a1 = fma(r0, pE, fma(pr, E0, -m0p));
  const double a2 = fma(pr, pE, -0.5 * pm2);
  double lo = 0.0, hi = b, x = 0.0;
  for (int it = 0; it < 40; ++it) {
    const double r = fma(x, pr, r0);
    const double A = fma(x, fma(x, a2, a1), a0);
    const double A2 = A * A;
    const double r2 = r * r, r4 = r2 * r2, r8 = r4 * r4;
    const double t = fma(pmin5 * r8 * r4, fast_rcp(A2 * A2 * A), -1.0);  // q - 1
    if (A > 0.0 && t <= 0.0) lo = x;
    else hi = x;
    const double lq = fabs(t) < 0.01
                          ? t * fma(-t, fma(-t, fma(-t, 0.25, 1.0 / 3.0), 0.5), 1.0)
                          : 0.6931471805599453 * (double)__builtin_amdgcn_logf((float)(1.0 + t));
    // d(log q)/dl = 12 rho'/rho - 5 A'/A
    const double dq = fma(12.0 * pr, A, -5.0 * r * fma(2.0 * x, a2, a1));
    const double d = -lq * (A * r) * fast_rcp(dq);
    if (fabs(d) <= 1e-9) return fmin(fmax(x + d, lo), hi);
    x += d;
    if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);
  }
  return x;
}

// The same for a general gamma, as a start for Newton steps on psi: log q =
// log phi_min + (gamma + 1) log rho - log A in FP32 (to some 1e-6, in units of
// the state's change along P), so no pow.  Returns the last iterate.
template <int DIM>
__device__ __forceinline__ double entropy_root_start(const Gas &g, const double *u,
                                                     const double *P, double b, double pmin) {
#pragma clang fp contract(off)  // the same bits in every kernel
  double m0p = 0.0, pm2 = 0.0, m02 = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    m0p = fma(u[1 + k], P[1 + k], m0p);
    pm2 = fma(P[1 + k], P[1 + k], pm2);
    m02 = fma(u[1 + k], u[1 + k], m02);
  }
  const double r0 = u[0], pr = P[0], E0 = u[DIM + 1], pE = P[DIM + 1];
  const double a0 = fma(r0, E0, -0.5 * m02);
  const double a1 = fma(r0, pE, fma(pr, E0, -m0p));
  const double a2 = fma(pr, pE, -0.5 * pm2);
  const float g1 = (float)(g.gamma + 1.0), lp = __builtin_amdgcn_logf((float)pmin);
  double lo = 0.0, hi = b, x = 0.0;
  for (int it = 0; it < 20; ++it) {
    const double r = fma(x, pr, r0);
    const double A = fma(x, fma(x, a2, a1), a0);
    const float lq = lp + g1 * __builtin_amdgcn_logf((float)r) - __builtin_amdgcn_logf((float)A);
    if (A > 0.0 && lq <= 0.0f) lo = x;
    else hi = x;
    // d(log q)/dl = (gamma + 1) rho'/rho - A'/A
    const double dq = fma((double)g1 * pr, A, -r * fma(2.0 * x, a2, a1));
    const double d = -0.6931471805599453 * (double)lq * (A * r) * fast_rcp(dq);
    if (fabs(d) <= 1e-4) return fmin(fmax(x + d, lo), hi);
    x += d;
    if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);
  }
  return x;
}

// Root of the entropy bound to the accuracy of psi itself: one Newton step on
// psi from the root of log q (gamma = 7/5), two from the rougher start of a
// general gamma.  psi is concave, so a tangent's root x lies at or beyond the
// root (within round-off of it from such a close start), and a point a below
// x with psi(a) >= 0 is within x - a of the root.  The rounding of psi
// blurs its sign change over a band of some 2^-52 E / |psi'|: the step back
// starts at a quarter of that, 2e-15 at least, and doubles until psi confirms a
// feasible point.  If none is confirmed (x was not close), the bracketing search
// on psi runs.  Against 128-bit roots, in units of that band or 1e-14, the larger:
// rms 0.2 - 0.6, at most 4 (steps of 2e-15 times powers of 8, gamma = 7/5: 0.3 -
// 0.9, at most 17; the bracketing search alone: 0.2 - 0.6, at most 40).
// A general gamma takes pow once, at the start x0: rho differs by less than
// 3e-5 afterwards, where three terms of (1 + d)^gamma are exact to rounding.
// The bracketing search takes 15, and its slowest lane holds up its wave: gamma =
// 5/3, 1% noise on the Mach-3 tube state at 2048^2 (every row limited),
// k_lim_rows 10.4 -> 2.7 ms per stage, the step 35.9 -> 12.3 ms.
template <int DIM, int SEV>
__device__ __forceinline__ double entropy_root_fast(const Gas &g, const double *u,
                                                   const double *P, double lr,
                                                   double pmin, double pmin5) {
#pragma clang fp contract(off)  // the same bits in every kernel
  double x0, x, d, w0 = 0.0, dr = 0.0;
  if constexpr (SEV) {
    x0 = entropy_root_seven<DIM>(u, P, lr, pmin5);
  } else {
    x0 = entropy_root_start<DIM>(g, u, P, lr, pmin);
    const double r0 = fma(x0, P[0], u[0]);
    w0 = pow(r0, g.gamma);
    dr = P[0] / r0;
  }
  auto power = [&](double r, double l) {
    if constexpr (SEV) {
      return pow_seven_fifths(r);
    } else {
      const double t = (l - x0) * dr, c = g.gamma;
      const double p = fma(t, fma(t, (c - 2.0) * (1.0 / 3.0), 1.0) * (0.5 * (c - 1.0)), 1.0);
      return fma(w0, c * t * p, w0);
    }
  };
  x = x0;
  bool ok = true;
#pragma unroll
  for (int t = SEV; t < 2; ++t) {
    const double f = psi_with<DIM>(g, u, P, x, pmin, &d, power);
    x -= f / d;
    if (t == 0) x = fmin(x, lr);
    ok = ok && d < 0.0 && x > 0.0;
    if (!SEV) ok = ok && fabs((x - x0) * dr) <= 3e-5;
  }
  if (ok && x <= lr) {
    double h = fmax(2e-15, 0x1p-54 * fabs(fma(x, P[DIM + 1], u[DIM + 1]) / d));
    for (int k = 0; k < 5; ++k, h *= 2.0) {
      const double a = fmax(x - h, 0.0);
      if (psi_with<DIM>(g, u, P, a, pmin, nullptr, power) >= 0.0) return a;
    }
  }
  return entropy_root<DIM, SEV>(g, u, P, lr, pmin);
}

}  // namespace ns
