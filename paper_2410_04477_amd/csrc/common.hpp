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
__device__ __forceinline__ Exp2Parts exp2neg_parts(double x) {
  x = __builtin_fmin(x, kExpBound);
  const double t = kExpShift - x;
  const double f = -x - (t - kExpShift);
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
  return {q * f, low_word(t)};
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
// fixed step h = 1/6 for kBesselLo <= x <= kBesselMid, and h = 1/12 up to kBesselHi:
// the discretisation error, about exp(x - pi^2 / h), is below 1e-16 there, the
// rounding error of the sums at most 1.2e-15.  With a fixed step cosh t,
// cosh(mu t), cosh((mu + 1) t) and t times their sinh depend on the node alone:
// a workgroup forms them once, and a node costs one exponential and two products
// (four with d / d nu).  12 to 50 nodes for the distances of neighbouring points,
// 111 at x = 1e-6.  Rows kBesselNodes on are the nodes halfway, as far as
// x > kBesselMid needs them (exp(-x (cosh t - 1)) < 1e-20 past the last).
constexpr int kBesselNodes = 128, kBesselHalf = 14;
constexpr int kBesselCols = 6;   // cosh t, h cosh(mu t), h cosh((mu + 1) t), h t sinh(mu t), h t sinh((mu + 1) t), a constant
constexpr double kBesselStep = 1.0 / 6.0, kBesselLo = 6e-8, kBesselMid = 16.0, kBesselHi = 72.0;
constexpr int kBesselBytes = (kBesselNodes + kBesselHalf) * kBesselCols * (int)sizeof(double);
typedef const __attribute__((address_space(3))) double LdsDouble;

// The table of one order by the 64 lanes of a wave; the caller orders the LDS accesses.
__device__ inline void bessel_table(double* tab, const BesselOrder& o, int ln) {
  for (int k = ln; k < kBesselNodes + kBesselHalf; k += 64) {
    const double t = (k < kBesselNodes ? k : k - kBesselNodes + 0.5) * kBesselStep;
    const double w = k == 0 ? 0.5 * kBesselStep : kBesselStep;
    const double e = exp(t), em = exp(o.mu * t);
    const double p = em * e, ei = 1.0 / e, emi = 1.0 / em, pi = 1.0 / p;
    double* row = tab + k * kBesselCols;
    row[0] = 0.5 * (e + ei);
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
// 520 us, one distance at a time with its own step (about 110 nodes at
// x = 1e-4, all weights recomputed, arrays in scratch) 1,112 us.  Outside
// [kBesselLo, kBesselHi] the functions above are called, lane by lane.
typedef double BesselOut __attribute__((ext_vector_type(8)));
typedef double Bessel4 __attribute__((ext_vector_type(4)));
template <int WHAT>
__device__ __noinline__ inline BesselOut bessel4(Bessel4 x, LdsDouble* tab) {
  constexpr bool DNU = WHAT == 2;
  const int order = (int)tab[kBesselCols + 5];
  const double mu = tab[5], lognorm = tab[2 * kBesselCols + 5], dlognorm = tab[3 * kBesselCols + 5];
  double u[4], k0[4], k1[4], d0[4], d1[4];
  bool rare = false, half = false;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const bool in = x[r] >= kBesselLo && x[r] <= kBesselHi;
    rare |= !in & (x[r] > 1e-140);
    half |= in & (x[r] > kBesselMid);
    u[r] = (in ? x[r] : 1.0) * kLog2E;
    k0[r] = k1[r] = d0[r] = d1[r] = 0.0;
  }
  auto node = [&](LdsDouble* row) __attribute__((always_inline)) {
    const double ch = row[0], c0 = row[1], c1 = row[2], s0 = row[3], s1 = row[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double e = exp2neg<double>(u[r] * ch);
      k0[r] = __builtin_fma(e, c0, k0[r]);
      k1[r] = __builtin_fma(e, c1, k1[r]);
      if (DNU) {
        d0[r] = __builtin_fma(e, s0, d0[r]);
        d1[r] = __builtin_fma(e, s1, d1[r]);
      }
    }
  };
  if (__any(half)) {
    // the nodes halfway first: their sums count for x > kBesselMid only, and both
    // sets then weigh one half
#pragma nounroll
    for (int k = kBesselNodes; k < kBesselNodes + kBesselHalf; ++k) node(tab + k * kBesselCols);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool take = u[r] > kBesselMid * kLog2E;
      k0[r] = take ? k0[r] : 0.0;
      k1[r] = take ? k1[r] : 0.0;
      d0[r] = take ? d0[r] : 0.0;
      d1[r] = take ? d1[r] : 0.0;
    }
  }
#pragma nounroll
  for (int k = 0; k < kBesselNodes; k += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) node(tab + (k + q) * kBesselCols);
    // past t = 1 t sinh((mu + 1) t) exceeds a third of every other weight of a node
    const double ch = tab[(k + 3) * kBesselCols], s1 = tab[(k + 3) * kBesselCols + 4];
    bool more = k < 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) more |= exp2neg<double>(u[r] * ch) * s1 > 1e-19 * k1[r];
    if (!__any(more)) break;
  }
  const double nu = mu + order;
  BesselOut out = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double w = u[r] > kBesselMid * kLog2E ? 0.5 : 1.0;
    const double z = u[r] * kLn2, zi = 1.0 / z;
    double klo = k0[r], khi = k1[r], dlo = d0[r], dhi = d1[r];   // K_(nu-1), K_nu, their derivatives in nu
    if (order == 0) {
      klo = k1[r] - (2.0 * mu * zi) * k0[r];
      khi = k0[r];
      dhi = d0[r];
    }
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
    const double logx = log(z);
    const double c = w * exp(lognorm + nu * logx);
    const bool at0 = x[r] <= 1e-140;   // a coincident pair (distance<double> gives 1e-150)
    const double nan = x[r] - x[r];    // 0, or NaN for the distance of a point that is not finite
    if (WHAT == 0) out[r] = at0 ? 1.0 : c * khi + nan;
    if (WHAT >= 1) out[r] = at0 ? 0.0 : c * z * klo + nan;
    if (DNU) out[r + 4] = at0 ? 0.0 : c * (khi * (logx + dlognorm) + dhi) + nan;
  }
  if (__any(rare)) {
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
      if (x[r] > 1e-140 && !(x[r] >= kBesselLo && x[r] <= kBesselHi)) {
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
