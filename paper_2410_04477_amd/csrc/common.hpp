// Shared device-side definitions of the block Vecchia HIP library (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vecchia.h"

namespace bv {

constexpr int kMaxThetaPerLaunch = 24;   // theta values passed by value in kernel arguments
constexpr double kLog2Pi = 1.83787706640934548356065947281123527;
constexpr double kLn2 = 0.693147180559945309417232121458176568;
constexpr double kLog2E = 1.44269504088896340735992468100189214;

// Order-only constants of the Bessel form (host-computed per theta): the
// order nu = n + mu with |mu| <= 1/2; Gamma(1 + mu), Gamma(1 - mu); Temme's
// Gamma1(mu) = (1/Gamma(1 - mu) - 1/Gamma(1 + mu)) / (2 mu) and Gamma2(mu) =
// (1/Gamma(1 - mu) + 1/Gamma(1 + mu)) / 2; mu pi / sin(mu pi);
// log(2^(1 - nu) / Gamma(nu)) and its derivative in nu, -log 2 - psi(nu).
struct BesselOrder {
  double mu, gplus, gminus, gam1, gam2, mu_pi_csc, lognorm, dlognorm;
  int n;
};

// One parameter vector as the kernels need it.  inv_scale[k] = 1 / (range * aniso[k]),
// so the Matern argument is x = || (s_i - s_j) * inv_scale ||.
struct ThetaDev {
  double sigma2;
  double nugget;
  double inv_scale[3];
  double inv_range;   // 1 / range (gradient w.r.t. range)
  int nu_code;        // 0: nu = 1/2, 1: nu = 3/2, 2: nu = 5/2, 3: any other nu (Bessel form)
  BesselOrder bes;    // nu_code 3: order-only constants of the Bessel form
};

struct ThetaPack {
  ThetaDev t[kMaxThetaPerLaunch];
};

// K_mu(x) and K_(mu+1)(x), |mu| <= 1/2, 0 < x <= 2: Temme's series (N. M.
// Temme, J. Comput. Phys. 19 (1975) 324-337).  With c_k = (x^2/4)^k / k!,
//   K_mu = sum_k c_k f_k,   K_(mu+1) = (2/x) sum_k c_k (p_k - k f_k),
// where p_k, q_k are p_0 = Gamma(1 + mu) (x/2)^-mu / 2 and q_0 = Gamma(1 - mu)
// (x/2)^mu / 2 divided by (1 - mu)..(k - mu) and (1 + mu)..(k + mu), and
// f_k = (k f_(k-1) + p_(k-1) + q_(k-1)) / (k^2 - mu^2) starts from
// f_0 = mu pi / sin(mu pi) [Gamma1 cosh(s) + Gamma2 ln(2/x) sinh(s) / s],
// s = mu ln(2/x).  About 15 terms reach FP64 rounding on this range.
__device__ inline void bessel_k_pair_series(double x, const BesselOrder& o, double& k_mu, double& k_mu1) {
  const double log2x = log(2.0 / x);
  const double s = o.mu * log2x;
  const double sinhc = fabs(s) < 1e-14 ? 1.0 : sinh(s) / s;
  const double es = exp(s);   // (2/x)^mu
  double f = o.mu_pi_csc * (o.gam1 * cosh(s) + o.gam2 * log2x * sinhc);
  double pk = 0.5 * o.gplus * es;
  double qk = 0.5 * o.gminus / es;
  const double quarter_x2 = 0.25 * x * x;
  double ck = 1.0;
  double sum_mu = f, sum_mu1 = pk;
  for (int k = 1; k < 60; ++k) {
    const double dk = (double)k;
    const double dm = dk - o.mu, dp = dk + o.mu;
    f = (dk * f + pk + qk) / (dm * dp);
    pk /= dm;
    qk /= dp;
    ck *= quarter_x2 / dk;
    const double t_mu = ck * f, t_mu1 = ck * (pk - dk * f);
    sum_mu += t_mu;
    sum_mu1 += t_mu1;
    if (fabs(t_mu) <= 1e-17 * fabs(sum_mu) && fabs(t_mu1) <= 1e-17 * fabs(sum_mu1)) break;
  }
  k_mu = sum_mu;
  k_mu1 = sum_mu1 * (2.0 / x);
}

// K_mu(x) and K_(mu+1)(x), |mu| <= 1/2, x > 2: the trapezoidal rule on the
// integral representation K_v(x) = int_0^inf exp(-x cosh t) cosh(v t) dt,
// whose integrand is analytic and decays doubly exponentially, so the rule
// converges geometrically in 1/h (L. N. Trefethen and J. A. C. Weideman,
// SIAM Review 56 (2014) 385-458).  Step h = min(1/8, 0.7/sqrt(x)) keeps the
// discretisation error below FP64 rounding for |v| <= 3/2 (the integrand's
// width shrinks like 1/sqrt(x)); nodes are added until the integrand falls
// below 1e-18 of the sum, at most 64 (13 to 31 on this range).  e^(+-v t) and
// e^(+-t) advance by multiplication, so each node costs one exponential.
__device__ inline void bessel_k_pair_quad(double x, double mu, double& k_mu, double& k_mu1) {
  const double h = fmin(0.125, 0.7 * rsqrt(x));
  const double a = exp(mu * h), ai = 1.0 / a, b = exp(h), bi = 1.0 / b;
  double emu = 1.0, emui = 1.0, et = 1.0, eti = 1.0;   // e^(mu t), e^(-mu t), e^t, e^-t
  double w = exp(-x);
  double s_mu = 0.5 * w, s_mu1 = 0.5 * w;              // the t = 0 node carries weight 1/2
  for (int k = 1; k < 64; ++k) {
    emu *= a;
    emui *= ai;
    et *= b;
    eti *= bi;
    w = exp(-0.5 * x * (et + eti));
    const double c1 = 0.5 * (emu * et + emui * eti);   // cosh((mu + 1) t)
    s_mu += w * 0.5 * (emu + emui);
    s_mu1 += w * c1;
    if (w * c1 < 1e-18 * s_mu1) break;
  }
  k_mu = h * s_mu;
  k_mu1 = h * s_mu1;
}

// Matern correlation for any nu > 0, eq. (maternkernel) with the modified
// Bessel function of the second kind: rho(x) = 2^(1-nu)/Gamma(nu) x^nu K_nu(x),
// in FP64.  K at the reduced order mu, then raised to nu = n + mu by the
// three-term recurrence K_(v+1) = K_(v-1) + (2 v / x) K_v, which is stable
// upwards for K.  Also returns g = 2^(1-nu)/Gamma(nu) x^(nu+1) K_(nu-1)(x),
// from d/dx [x^nu K_nu(x)] = -x^nu K_(nu-1)(x): d rho(h/range) / d range =
// g / range.  Not inlined: its loops would otherwise be copied into every
// generation site.  The FP64 kernels call it only for distances outside the range of
// bessel4 below, the FP32 kernels for all.
__device__ __noinline__ inline void matern_general(double x, const BesselOrder& o, double* rho, double* g) {
  if (x <= 1e-140) {   // a coincident pair (distance<double> gives 1e-150); a NaN goes on to NaN
    *rho = 1.0;
    *g = 0.0;
    return;
  }
  double k_lo, k_hi;   // K_(v-1), K_v as v climbs from mu
  {
    double k_mu, k_mu1;
    if (x <= 2.0)
      bessel_k_pair_series(x, o, k_mu, k_mu1);
    else
      bessel_k_pair_quad(x, o.mu, k_mu, k_mu1);
    // K_(mu-1) = K_(mu+1) - (2 mu / x) K_mu
    k_lo = o.n == 0 ? k_mu1 - (2.0 * o.mu / x) * k_mu : k_mu;
    k_hi = o.n == 0 ? k_mu : k_mu1;
    for (int v = 1; v < o.n; ++v) {
      const double next = k_lo + (2.0 * (o.mu + v) / x) * k_hi;
      k_lo = k_hi;
      k_hi = next;
    }
  }
  const double nu = o.mu + o.n, logx = log(x);
  *rho = exp(o.lognorm + nu * logx) * k_hi;
  *g = exp(o.lognorm + (nu + 1.0) * logx) * k_lo;
}

// rho and g as matern_general, and d rho / d nu.  K_mu, K_(mu+1) and their
// derivatives in the order come from the trapezoidal rule on
//   K_v(x) = int_0^inf exp(-x cosh t) cosh(v t) dt,
//   d K_v / d v = int_0^inf t exp(-x cosh t) sinh(v t) dt
// for every x > 0 (the same nodes serve all four; the step as in
// bessel_k_pair_quad, nodes until the integrands fall below 1e-18 of the sums
// and t > 1, at most 320: about 110 at x = 1e-4, fewer as x grows).  The
// order is raised by the recurrence K_(v+1) = K_(v-1) + (2 v / x) K_v and its
// derivative D_(v+1) = D_(v-1) + (2 v / x) D_v + (2 / x) K_v (mu moves with
// nu).  Then d rho / d nu = 2^(1-nu)/Gamma(nu) x^nu [K_nu (log x - log 2 -
// psi(nu)) + D_nu].
__device__ __noinline__ inline void matern_general_dnu(double x, const BesselOrder& o, double* rho, double* g,
                                                       double* drho_dnu) {
  if (x <= 1e-140) {   // a coincident pair (distance<double> gives 1e-150); a NaN goes on to NaN
    *rho = 1.0;
    *g = 0.0;
    *drho_dnu = 0.0;
    return;
  }
  const double h = fmin(0.125, 0.7 * rsqrt(x));
  const double a = exp(o.mu * h), ai = 1.0 / a, b = exp(h), bi = 1.0 / b;
  double emu = 1.0, emui = 1.0, et = 1.0, eti = 1.0;
  const double w0 = exp(-x);
  double k0 = 0.5 * w0, k1 = 0.5 * w0, d0 = 0.0, d1 = 0.0;   // t = 0: weight 1/2, sinh(0) = 0
  for (int k = 1; k < 320; ++k) {
    emu *= a;
    emui *= ai;
    et *= b;
    eti *= bi;
    const double t = k * h;
    const double w = exp(-0.5 * x * (et + eti));
    const double c1 = 0.5 * (emu * et + emui * eti), s1 = 0.5 * (emu * et - emui * eti);
    k0 += w * 0.5 * (emu + emui);
    k1 += w * c1;
    d0 += w * t * 0.5 * (emu - emui);
    d1 += w * t * s1;
    if (t > 1.0 && w * t * c1 < 1e-18 * k1) break;
  }
  k0 *= h;
  k1 *= h;
  d0 *= h;
  d1 *= h;
  double klo, khi, dhi;   // K_(nu-1), K_nu, d K_nu / d nu
  if (o.n == 0) {
    klo = k1 - (2.0 * o.mu / x) * k0;
    khi = k0;
    dhi = d0;
  } else {
    klo = k0;
    khi = k1;
    double dlo = d0;
    dhi = d1;
    for (int v = 1; v < o.n; ++v) {
      const double vv = o.mu + v;
      const double kn = klo + (2.0 * vv / x) * khi;
      const double dn = dlo + (2.0 * vv / x) * dhi + (2.0 / x) * khi;
      klo = khi;
      khi = kn;
      dlo = dhi;
      dhi = dn;
    }
  }
  const double nu = o.mu + o.n, logx = log(x);
  const double c = exp(o.lognorm + nu * logx);
  *rho = c * khi;
  *g = c * x * klo;
  *drho_dnu = c * (khi * (logx + o.dlognorm) + dhi);
}

template <typename T> __device__ __forceinline__ T expneg(T x);
template <> __device__ __forceinline__ double expneg<double>(double x) { return exp(-x); }
template <> __device__ __forceinline__ float expneg<float>(float x) { return __expf(-x); }

// 2^-x.  FP32: one v_exp_f32.  FP64, x >= 0: 2^-x = 2^m 2^f with m = -x rounded
// to an integer (by adding 3 2^51: the sum's low word is m, with no conversion, which
// would be undefined beyond 32 bits; hence the bound, past which 2^-x is zero)
// and f = -x - m exact, |f| <= 1/2, and 2^f = 1 + f q(f), q the
// degree-10 interpolant of (2^f - 1) / f at the Chebyshev nodes (8.4e-18
// relative; with rounding 1.35e-16 at most and 3.8e-17 in the mean over
// x in [1e-10, 1e3], as the library's exp2): 16 instructions.  A NaN x gives zero: the
// callers multiply by a polynomial in x.
constexpr double kExpBound = 2200.0, kExpShift = 0x1.8p52;
__device__ __forceinline__ int low_word(double t) { return (int)__builtin_bit_cast(unsigned long long, t); }
// 2^-x as 2^m (1 + w): the products with it round once (scaled)
struct Exp2Parts {
  double w;
  int m;
};
__device__ __forceinline__ double scaled(const Exp2Parts& e, double p) {
  return __builtin_amdgcn_ldexp(__builtin_fma(e.w, p, p), e.m);
}
// 2^f - 1, |f| <= 1/2
__device__ __forceinline__ double exp2m1(double f) {
  double q = 0x1.e9d3fe3952179p-32;
  q = __builtin_fma(q, f, 0x1.e6063f7217bc6p-28);
  q = __builtin_fma(q, f, 0x1.b524fae627834p-24);
  q = __builtin_fma(q, f, 0x1.62bfd47773353p-20);
  q = __builtin_fma(q, f, 0x1.ffcbfc670dcd4p-17);
  q = __builtin_fma(q, f, 0x1.430913096fd9fp-13);
  q = __builtin_fma(q, f, 0x1.5d87fe78a5276p-10);
  q = __builtin_fma(q, f, 0x1.3b2ab6fba1ddap-7);
  q = __builtin_fma(q, f, 0x1.c6b08d704a0c2p-5);
  q = __builtin_fma(q, f, 0x1.ebfbdff82c598p-3);
  q = __builtin_fma(q, f, 0x1.62e42fefa39efp-1);
  return q * f;
}
__device__ __forceinline__ Exp2Parts exp2neg_parts(double x) {
  x = __builtin_fmin(x, kExpBound);
  const double t = kExpShift - x;
  return {exp2m1(-x - (t - kExpShift)), low_word(t)};
}
// 2^-(x y), the product unrounded; past the bound (where 2^-(x y) is zero) x y < 2^40
__device__ __forceinline__ double exp2neg_product(double x, double y) {
  const double t = kExpShift - __builtin_fmin(x * y, kExpBound);
  return scaled({exp2m1(__builtin_fma(-x, y, kExpShift - t)), low_word(t)}, 1.0);
}
template <typename T> __device__ __forceinline__ T exp2neg(T x);
template <> __device__ __forceinline__ double exp2neg<double>(double x) { return scaled(exp2neg_parts(x), 1.0); }
template <> __device__ __forceinline__ float exp2neg<float>(float x) { return __builtin_amdgcn_exp2f(-x); }

template <typename T> __device__ __forceinline__ T sqrt_(T x);
template <> __device__ __forceinline__ double sqrt_<double>(double x) { return sqrt(x); }
template <> __device__ __forceinline__ float sqrt_<float>(float x) { return sqrtf(x); }

// Matern correlation rho_nu(x) for half-integer nu, eq. (maternkernel) in closed form.
template <typename T>
__device__ __forceinline__ T matern_rho(T x, int nu_code) {
  const T e = expneg<T>(x);
  if (nu_code == 0) return e;
  if (nu_code == 1) return (T(1) + x) * e;
  return (T(1) + x + x * x * T(1.0 / 3.0)) * e;
}

// Branch-free closed forms: rho = e^-x (1 + c1 x + c2 x^2) with (c1, c2) =
// (0, 0), (1, 0), (1, 1/3) for nu = 1/2, 3/2, 5/2, and
// d rho / d range = (x / range) e^-x (g0 + g1 x + g2 x^2) with (g0, g1, g2) =
// (1, 0, 0), (0, 1, 0), (0, 1/3, 1/3).
template <typename T>
struct MaternCoef {
  T c1, c2, g0, g1, g2;
  __device__ __forceinline__ explicit MaternCoef(int nu_code)
      : c1(nu_code == 0 ? T(0) : T(1)),
        c2(nu_code == 2 ? T(1.0 / 3.0) : T(0)),
        g0(nu_code == 0 ? T(1) : T(0)),
        g1(nu_code == 0 ? T(0) : (nu_code == 1 ? T(1) : T(1.0 / 3.0))),
        g2(nu_code == 2 ? T(1.0 / 3.0) : T(0)) {}
  __device__ __forceinline__ T rho(T x) const { return expneg<T>(x) * (T(1) + x * (c1 + c2 * x)); }
  __device__ __forceinline__ void rho_drange(T x, T inv_range, T& r, T& dr) const {
    const T e = expneg<T>(x);
    r = e * (T(1) + x * (c1 + c2 * x));
    dr = x * inv_range * e * (g0 + x * (g1 + g2 * x));
  }
  __device__ __forceinline__ T drange(T x, T inv_range) const {
    return x * inv_range * expneg<T>(x) * (g0 + x * (g1 + g2 * x));
  }
  // -(sigma2 rho) and d rho / d range for a distance u = x log2(e) and e = 2^-u = e^-x
  // (FP64: its parts) with the scales and sign in the coefficients: (s0, s1, s2) =
  // -sigma2 (1, c1 ln 2, c2 ln(2)^2), (h0, h1, h2) = (g0 ln 2, g1 ln(2)^2,
  // g2 ln(2)^3) / range
  static __device__ __forceinline__ float neg_cov_log2(float u, float e, float s0, float s1, float s2) {
    return e * (s0 + u * (s1 + s2 * u));
  }
  static __device__ __forceinline__ float drange_log2(float u, float e, float h0, float h1, float h2) {
    return u * e * (h0 + u * (h1 + h2 * u));
  }
  static __device__ __forceinline__ double neg_cov_log2(double u, const Exp2Parts& e, double s0, double s1, double s2) {
    return scaled(e, s0 + u * (s1 + s2 * u));
  }
  static __device__ __forceinline__ double drange_log2(double u, const Exp2Parts& e, double h0, double h1, double h2) {
    return scaled(e, u * (h0 + u * (h1 + h2 * u)));
  }
};

// 1 / sqrt(x) in FP64, 0 < x < inf normal: the hardware estimate y (2^-24) and one
// third-order step, y + y e (1/2 + 3/8 e) with e = 1 - x y^2: 1.4e-16 relative
// at most (1 / sqrt(x) through the library: 1.7e-16), 5 dependent operations
// instead of about 20.
__device__ __forceinline__ double rsqrt_fast(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-(x * y), y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

// Distance sqrt(dx^2 + dy^2 + dz^2).  FP64: from the estimate y of 1 / sqrt, g = x y
// with one second-order step (2^-47) and one with the exact residual x - g^2, which
// leaves the rounding of the last operation (1.1e-16, as the library's square
// root; a third-order step instead of the two is one operation less and 1.4e-16).
// The sum starts from 1e-300, so coincident points
// come out at 1e-150 instead of 0 * inf.  A sum of squares that overflows, and any
// coordinate that is not finite, gives NaN, and so does the covariance.
template <typename T> __device__ __forceinline__ T distance(T dx, T dy, T dz);
template <> __device__ __forceinline__ double distance<double>(double dx, double dy, double dz) {
  const double x = __builtin_fma(dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, 1e-300)));
  const double y = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * y;
  double g = x * y;
  g = __builtin_fma(g, __builtin_fma(-h, g, 0.5), g);
  return __builtin_fma(__builtin_fma(-g, g, x), h, g);
}
template <> __device__ __forceinline__ float distance<float>(float dx, float dy, float dz) {
  return __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz);
}

// 2^-u as the kernels keep it until it multiplies a polynomial
template <typename T> struct ExpOf { typedef T type; };
template <> struct ExpOf<double> { typedef Exp2Parts type; };

// distance() and exp2neg() of four pairs.  STAGED (FP64): step by step across the
// four.  A dependent FP64 operation waits about 8 cycles and issues in 4, and the
// scheduler left to itself runs the pairs one after the other, so the kernels
// that hold one wave per SIMD would wait half of the time.
template <bool STAGED>
__device__ __forceinline__ void distance_exp2neg4(const double (&dx)[4], const double (&dy)[4], const double (&dz)[4],
                                                  double (&u)[4], Exp2Parts (&p)[4]) {
  if constexpr (!STAGED) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      u[r] = distance<double>(dx[r], dy[r], dz[r]);
      p[r] = exp2neg_parts(u[r]);
    }
    return;
  }
#define BV_STEP(...)                             \
  do {                                           \
    _Pragma("unroll") for (int r = 0; r < 4; ++r) { __VA_ARGS__; } \
    __builtin_amdgcn_sched_barrier(0);           \
  } while (0)
  double y[4], e[4], t[4];
  BV_STEP(u[r] = __builtin_fma(dz[r], dz[r], 1e-300));
  BV_STEP(u[r] = __builtin_fma(dy[r], dy[r], u[r]));
  BV_STEP(u[r] = __builtin_fma(dx[r], dx[r], u[r]));
  BV_STEP(y[r] = __builtin_amdgcn_rsq(u[r]));
  BV_STEP(t[r] = u[r] * y[r]);
  BV_STEP(y[r] = 0.5 * y[r]);
  BV_STEP(e[r] = __builtin_fma(-y[r], t[r], 0.5));
  BV_STEP(t[r] = __builtin_fma(t[r], e[r], t[r]));
  BV_STEP(e[r] = __builtin_fma(-t[r], t[r], u[r]));
  BV_STEP(u[r] = __builtin_fma(e[r], y[r], t[r]));
  BV_STEP(e[r] = __builtin_fmin(u[r], kExpBound));
  BV_STEP(t[r] = kExpShift - e[r]);
  BV_STEP(y[r] = t[r] - kExpShift; p[r].m = low_word(t[r]));
  BV_STEP(y[r] = -e[r] - y[r]);
  BV_STEP(p[r].w = __builtin_fma(0x1.e9d3fe3952179p-32, y[r], 0x1.e6063f7217bc6p-28));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.b524fae627834p-24));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.62bfd47773353p-20));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.ffcbfc670dcd4p-17));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.430913096fd9fp-13));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.5d87fe78a5276p-10));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.3b2ab6fba1ddap-7));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.c6b08d704a0c2p-5));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.ebfbdff82c598p-3));
  BV_STEP(p[r].w = __builtin_fma(p[r].w, y[r], 0x1.62e42fefa39efp-1));
  BV_STEP(p[r].w = p[r].w * y[r]);
#undef BV_STEP
}
template <bool STAGED>
__device__ __forceinline__ void distance_exp2neg4(const float (&dx)[4], const float (&dy)[4], const float (&dz)[4],
                                                  float (&u)[4], float (&w)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    u[r] = distance<float>(dx[r], dy[r], dz[r]);
    w[r] = exp2neg<float>(u[r]);
  }
}

// ---- Bessel form of four pairs at once ---------------------------------------
// K_v(x) = int_0^inf exp(-x cosh t) cosh(v t) dt by the trapezoidal rule with the
// fixed step h = 43/256 for kBesselLo <= x <= kBesselMid, and h / 2 up to kBesselHi:
// the discretisation error, about exp(x - pi^2 / h), is below 3e-19 there.  With a
// fixed step cosh t and the weights depend on the node alone: a workgroup forms
// them once, and a node costs one exponential and two products (four with
// d / d nu).  12 to 50 nodes for the distances of neighbouring points, 108 at
// x = 1e-6.  Rows kBesselNodes on are the nodes halfway, as far as x > kBesselMid needs
// them (exp(-x (cosh t - 1)) < 1e-20 past the last).
// Rounding: the nodes are exact numbers, cosh(t) log2(e) is a rounded constant, and
// the product with x enters the exponential unrounded; the sums run over even and
// odd nodes apart.  Against 113-bit arithmetic rho is then off by 1.4e-16 to
// 3e-16 in the mean (root of squares, nu up to 2) and 1e-15 at most for x in
// [1e-3, 16], 1.2e-15 and 3e-15 up to 72; the functions above 1.6e-16 to 5e-16 and
// 4e-15, 1.8e-15 and 1.1e-14.
constexpr int kBesselNodes = 128, kBesselHalf = 14;
constexpr int kBesselCols = 6;   // log2(e) cosh t, the weights of K_mu and of the second order, of their derivatives, a constant
constexpr double kBesselStep = 43.0 / 256.0, kBesselLo = 6e-8, kBesselMid = 16.0, kBesselHi = 72.0;
constexpr double kBesselNear = 1.0 / 256.0;
constexpr int kBesselBytes = (kBesselNodes + kBesselHalf) * kBesselCols * (int)sizeof(double);
typedef const __attribute__((address_space(3))) double LdsDouble;

// log2(e) cosh(k h), k = 0 .. 127, then log2(e) cosh((k + 1/2) h), k = 0 .. 13
static __device__ const double kBesselCosh[kBesselNodes + kBesselHalf] = {
    0x1.71547652b82fep+0, 0x1.768d5f615ce91p+0, 0x1.865de951e93f9p+0, 0x1.a1389229253b4p+0, 0x1.c7dfc40e6493dp+0,
    0x1.fb6b54ca32a2dp+0, 0x1.1ea837d787692p+1, 0x1.47b6119b8d70dp+1, 0x1.7a086f5ebf3dfp+1, 0x1.b70ba0ffa22f3p+1,
    0x1.003cae05e42fap+2, 0x1.2c329cc9106d5p+2, 0x1.60a5df5c4dcf9p+2, 0x1.9f122e75c64f0p+2, 0x1.e93b75fc3bda8p+2,
    0x1.209d4e64294aep+3, 0x1.54c659d00f70dp+3, 0x1.92927cacafc9ap+3, 0x1.dbc11b4852385p+3, 0x1.193202e56fa43p+4,
    0x1.4c7739efd9b70p+4, 0x1.892360c5f6903p+4, 0x1.d0edb6cda6269p+4, 0x1.12eefc6827557p+5, 0x1.452d89d97941ap+5,
    0x1.809e442777926p+5, 0x1.c6ef7f289c582p+5, 0x1.0d0f26c499a07p+6, 0x1.3e4273272de26p+6, 0x1.7875d654eda5bp+6,
    0x1.bd4eaab53199bp+6, 0x1.075faef89714cp+7, 0x1.378ac4b368776p+7, 0x1.70854f53807f0p+7, 0x1.b3ebd05ad5c00p+7,
    0x1.01d31e359bc68p+8, 0x1.30fae3f3b97e5p+8, 0x1.68c29cdb255ffp+8, 0x1.aabe1d2a058cep+8, 0x1.f8cb157e6a682p+8,
    0x1.2a8f4a92c49c1p+9, 0x1.612a82790133dp+9, 0x1.a1c28724b8c98p+9, 0x1.ee2afba12c4d5p+9, 0x1.2446856cc1530p+10,
    0x1.59bb862b63d0bp+10, 0x1.98f782bab49a0p+10, 0x1.e3c44684f9bcap+10, 0x1.1e1fabfb5ee17p+11, 0x1.5274a479878bcp+11,
    0x1.905bea2a42138p+11, 0x1.d995a5d0782dep+11, 0x1.1819fc0497bd6p+12, 0x1.4b54fb9dec5e8p+12, 0x1.87eeb5bfe4d1dp+12,
    0x1.cf9de46d140f4p+12, 0x1.1234bfecbe06ap+13, 0x1.445bb5c9b8aa5p+13, 0x1.7faee96db21d3p+13, 0x1.c5dbd8ed0846bp+13,
    0x1.0c6f48185df9ep+14, 0x1.3d880385918f3p+14, 0x1.779b90026c290p+14, 0x1.bc4e6176188a6p+14, 0x1.06c8e92ca2f63p+15,
    0x1.36d91a305f479p+15, 0x1.6fb3b9dbc0d1fp+15, 0x1.b2f4629dda3c8p+15, 0x1.0140fb8e6103ap+16, 0x1.304e338b96230p+16,
    0x1.67f67c7c8c505p+16, 0x1.a9ccc706f350bp+16, 0x1.f7adb66599cc9p+16, 0x1.29e68d8cb0ed7p+17, 0x1.6062f25dc525dp+17,
    0x1.a0d67f3022eb7p+17, 0x1.ed13cf0abb0edp+17, 0x1.23a16a40b2585p+18, 0x1.58f83acecf3d3p+18, 0x1.9810815080e6ap+18,
    0x1.e2b306a6c0fe8p+18, 0x1.1d7e0fb49a77cp+19, 0x1.51b579da27ec0p+19, 0x1.8f79c9379a7ffp+19, 0x1.d88a29729aa9dp+19,
    0x1.177bc7df77b7ep+20, 0x1.4a99d82b95d2cp+20, 0x1.8711582f0642ep+20, 0x1.ce980a21a6b15p+20, 0x1.1199e08d36b06p+21,
    0x1.43a482f72144fp+21, 0x1.7ed634dccfd01p+21, 0x1.c4db81bebc4b0p+21, 0x1.0bd7ab49f6b2dp+22, 0x1.3cd4abe0a33f6p+22,
    0x1.76c76b269049ap+22, 0x1.bb536f89fbe19p+22, 0x1.06347d4dd2754p+23, 0x1.362988e3dc12ap+23, 0x1.6ee40c1525e0bp+23,
    0x1.b1feb8d75ac2cp+23, 0x1.00afaf6916e0cp+24, 0x1.2fa2543d0bea1p+24, 0x1.672b2db904a4ep+24, 0x1.a8dc48ede3cafp+24,
    0x1.f6913be1c9957p+24, 0x1.293e4c5209b11p+25, 0x1.5f9beb0f1cb80p+25, 0x1.9feb10e7a8b35p+25, 0x1.ebfd5158763d5p+25,
    0x1.22fcb39bd57b2p+26, 0x1.583563e652953p+26, 0x1.972a079260277p+26, 0x1.e1a26582ce6cdp+26, 0x1.1cdcd090a3c92p+27,
    0x1.50f6bcc5864fbp+27, 0x1.8e982950acf5bp+27, 0x1.d77f4547b26c9p+27, 0x1.16dded8e5f1d7p+28, 0x1.49df1ed226c28p+28,
    0x1.863477fc0ac98p+28, 0x1.cd92c404b4a2fp+28, 0x1.10ff58c59d5fep+29, 0x1.42edb7b74dbf1p+29, 0x1.7dfdfac75cf31p+29,
    0x1.c3dbbb6b45cdap+29, 0x1.0b40642506a19p+30, 0x1.3c21b98d62585p+30, 0x1.72a219e3904f6p+0, 0x1.7d1d5b6f0007cp+0,
    0x1.925fc05dfcb0bp+0, 0x1.b30331bd22b98p+0, 0x1.dff3fa0f80787p+0, 0x1.0d3bb9fc782d6p+1, 0x1.321a9ed8bd513p+1,
    0x1.5fa199ef32304p+1, 0x1.971a4545eb1fep+1, 0x1.da1638ca18024p+1, 0x1.153d32dae553bp+2, 0x1.454666b033747p+2,
    0x1.7e827b6168551p+2, 0x1.c28fccebdee2ep+2};

// The table of one order by the 64 lanes of a wave; the caller orders the LDS accesses.
// The second order is mu + 1, or 1 - mu for nu < 1/2 (K_(nu-1) = K_(1-nu), which
// the recurrence downwards would get by a cancellation).
__device__ inline void bessel_table(double* tab, const BesselOrder& o, int ln) {
  for (int k = ln; k < kBesselNodes + kBesselHalf; k += 64) {
    const double t = (k < kBesselNodes ? k : k - kBesselNodes + 0.5) * kBesselStep;   // exact
    const double w = k == 0 ? 0.5 * kBesselStep : kBesselStep;
    const double a = o.mu * t, e = exp(t);
    double em = exp(a);
    em = __builtin_fma(em, __builtin_fma(o.mu, t, -a), em);   // e^(mu t) for the exact product
    const double p = o.n == 0 ? e / em : em * e, emi = 1.0 / em, pi = 1.0 / p;
    double* row = tab + k * kBesselCols;
    row[0] = kBesselCosh[k];
    row[1] = w * 0.5 * (em + emi);
    row[2] = w * 0.5 * (p + pi);
    row[3] = w * t * 0.5 * (em - emi);
    row[4] = w * t * 0.5 * (p - pi);
    row[5] = k == 0 ? o.mu : k == 1 ? (double)o.n : k == 2 ? o.lognorm : k == 3 ? o.dlognorm
           : k == 4 ? o.gplus : k == 5 ? o.gminus : k == 6 ? o.gam1 : k == 7 ? o.gam2 : o.mu_pi_csc;
  }
}

// The functions of four distances: WHAT 0 rho, 1 g (as matern_general), 2 g and
// d rho / d nu.  One copy for all tiles of a kernel (a copy per tile made the
// kernels 90 to 460 KB); the results come back in registers.  Bound by the FP64
// operations of the exponentials: 2,000 blocks, m = 30, d l / d range and d l / d nu
// 1,112 us one distance at a time with its own step (about 110 nodes at
// x = 1e-4, all weights recomputed, arrays in scratch), 514 us with a rounded
// exponent (rho off by up to 1e-14), 530 us now.  Outside
// [kBesselLo, kBesselHi] the functions above are called, lane by lane.
typedef double BesselOut __attribute__((ext_vector_type(8)));
typedef double Bessel4 __attribute__((ext_vector_type(4)));
template <int WHAT>
__device__ __noinline__ inline BesselOut bessel4(Bessel4 x, LdsDouble* tab) {
  constexpr bool DNU = WHAT == 2;
  const int order = (int)tab[kBesselCols + 5];
  const double mu = tab[5], lognorm = tab[2 * kBesselCols + 5], dlognorm = tab[3 * kBesselCols + 5];
  // The smallest distance of the wave sets the number of nodes, 6 log(80 / x), where
  // Temme's series takes 15 terms for any x <= 2: below kBesselNear (58 nodes, where
  // both cost the same), if no distance of the wave exceeds 2, the series serves them
  // all (g of nu < 1/2 excepted, which it has by a cancellation).  20,000 points
  // of which every second lies within 1e-7 of another, range 0.1, m = 30, value / value
  // and gradient: 389 / 1,103 us with nodes throughout, 311 / 846 us so.  (With the line
  // at 1/32 for g points without such neighbours take 642 instead of 614 us.)
  // sums over the even ([0]) and the odd nodes apart; with the derivatives in the order
  // over all (the gradient kernel of G = 3 would lose its second wave)
  constexpr int ODD = DNU ? 0 : 1;
  double z[4], k0[2][4], k1[2][4], d0[4], d1[4], last[4];
  bool rare = false, half = false, near = false, far = false;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const bool in = x[r] >= kBesselLo && x[r] <= kBesselHi;
    rare |= !in & (x[r] > 1e-140);
    half |= in & (x[r] > kBesselMid);
    near |= in & (x[r] < kBesselNear);
    far |= x[r] > 2.0;
    z[r] = in ? x[r] : 1.0;
    k0[0][r] = k1[0][r] = k0[1][r] = k1[1][r] = d0[r] = d1[r] = 0.0;
  }
  auto node = [&](LdsDouble* row, int s) __attribute__((always_inline)) {
    const double ch = row[0], c0 = row[1], c1 = row[2], s0 = row[3], s1 = row[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double e = exp2neg_product(z[r], ch);
      k0[s][r] = __builtin_fma(e, c0, k0[s][r]);
      k1[s][r] = __builtin_fma(e, c1, k1[s][r]);
      if (DNU) {
        d0[r] = __builtin_fma(e, s0, d0[r]);
        d1[r] = __builtin_fma(e, s1, d1[r]);
      }
      last[r] = e * s1;
    }
  };
  const bool series = __any(near) && !__any(far) && (WHAT == 0 || (WHAT == 1 && order > 0));   // the same in every lane
  if (__any(half)) {
    // the nodes halfway first: their sums count for x > kBesselMid only, and both
    // sets then weigh one half
#pragma nounroll
    for (int k = kBesselNodes; k < kBesselNodes + kBesselHalf; ++k) node(tab + k * kBesselCols, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool take = z[r] > kBesselMid;
      k0[0][r] = take ? k0[0][r] : 0.0;
      k1[0][r] = take ? k1[0][r] : 0.0;
      d0[r] = take ? d0[r] : 0.0;
      d1[r] = take ? d1[r] : 0.0;
    }
  }
#pragma nounroll
  for (int k = 0; k < kBesselNodes && !series; k += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) node(tab + (k + q) * kBesselCols, q & ODD);
    // past t = 1 t sinh of the second order exceeds a third of every other weight of a node
    bool more = k < 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) more |= last[r] > 1e-19 * k1[ODD][r];
    if (!__any(more)) break;
  }
  const double nu = mu + order;
  BesselOut out = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double w = z[r] > kBesselMid ? 0.5 : 1.0, zi = 1.0 / z[r];
    const double a0 = k0[0][r] + k0[1][r], a1 = k1[0][r] + k1[1][r];
    double klo = order == 0 ? a1 : a0, khi = order == 0 ? a0 : a1;   // K_(nu-1), K_nu
    double dlo = d0[r], dhi = order == 0 ? d0[r] : d1[r];   // their derivatives in nu
    for (int v = 1; v < order; ++v) {
      const double f = 2.0 * (mu + v) * zi;
      const double kn = klo + f * khi;
      if (DNU) {
        const double dnx = dlo + f * dhi + (2.0 * zi) * khi;
        dlo = dhi;
        dhi = dnx;
      }
      klo = khi;
      khi = kn;
    }
    const double logx = log(z[r]);
    const double c = w * exp(lognorm + nu * logx);
    const bool at0 = x[r] <= 1e-140;   // a coincident pair (distance<double> gives 1e-150)
    const double nan = x[r] - x[r];    // 0, or NaN for a NaN distance
    if (WHAT == 0) out[r] = at0 ? 1.0 : c * khi + nan;
    if (WHAT >= 1) out[r] = at0 ? 0.0 : c * z[r] * klo + nan;
    if (DNU) out[r + 4] = at0 ? 0.0 : c * (khi * (logx + dlognorm) + dhi) + nan;
  }
  if (series || __any(rare)) {
    BesselOrder o;
    o.mu = mu;
    o.n = order;
    o.lognorm = lognorm;
    o.dlognorm = dlognorm;
    o.gplus = tab[4 * kBesselCols + 5];
    o.gminus = tab[5 * kBesselCols + 5];
    o.gam1 = tab[6 * kBesselCols + 5];
    o.gam2 = tab[7 * kBesselCols + 5];
    o.mu_pi_csc = tab[8 * kBesselCols + 5];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (x[r] > 1e-140 && (series || !(x[r] >= kBesselLo && x[r] <= kBesselHi))) {
        double rho, g, dn = 0.0;
        if (DNU) matern_general_dnu(x[r], o, &rho, &g, &dn);
        else matern_general(x[r], o, &rho, &g);
        out[r] = WHAT == 0 ? rho : g;
        if (DNU) out[r + 4] = dn;
      }
  }
  return out;
}

// rho and x * d rho / d x * (-1) / range, i.e. d rho(h/range) / d range.
template <typename T>
__device__ __forceinline__ void matern_rho_drange(T x, int nu_code, T inv_range, T& rho, T& drho) {
  const T e = expneg<T>(x);
  T g;
  if (nu_code == 0) {
    rho = e;
    g = e;
  } else if (nu_code == 1) {
    rho = (T(1) + x) * e;
    g = x * e;
  } else {
    rho = (T(1) + x + x * x * T(1.0 / 3.0)) * e;
    g = x * T(1.0 / 3.0) * (T(1) + x) * e;
  }
  drho = x * inv_range * g;
}

__host__ __device__ constexpr int threads_for_grid(int G) {
  return ((G * (G + 1) / 2 + 63) / 64) * 64;
}

// Register-tile configurations: tile size R, tile grid G (G x G lower triangle of
// tiles, one tile per thread), joint capacity P = R * G.
struct TileCfg {
  int R, G;
};
constexpr TileCfg kCfgs[] = {
    {1, 10}, {2, 10}, {3, 10}, {4, 10}, {3, 15}, {4, 15}, {4, 18},
    {4, 22}, {5, 22}, {6, 22}, {8, 18}, {7, 22}, {8, 22},
};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);

__host__ __device__ inline int cfg_for_joint(int p) {
  for (int c = 0; c < kNumCfgs; ++c)
    if (kCfgs[c].R * kCfgs[c].G >= p) return c;
  return -1;
}

// Matrix-core engine: 16 x 16 tiles, G tile rows for the bordered (p + 1)-row
// matrix, G = 1..kMfmaMaxG; configuration id = G - 1.
constexpr int kMfmaMaxG = 11;
__host__ __device__ inline int cfg_mfma_for_joint(int p) {
  const int g = (p + 1 + 15) / 16;
  return (g >= 1 && g <= kMfmaMaxG) ? g - 1 : -1;
}

enum { kEngineMfma = 0, kEngineTiles = 1, kEngineMfmaWg = 2 };

}  // namespace bv
