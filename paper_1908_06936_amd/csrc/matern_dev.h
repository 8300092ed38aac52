// Matern covariance (paper eq. 3) and its theta-derivatives on the device.
//
//   Sigma(r) = sigma2 c(nu) x^nu K_nu(x),   x = r / beta,   c(nu) = 2^(1-nu) / Gamma(nu)
//
// K_nu comes from its integral form  K_nu(x) = int_0^inf exp(-x cosh t) cosh(nu t) dt
// (DLMF 10.32.9), evaluated as  e^-x * T(x)  with the trapezoidal rule
//   T(x) = h [ f(0)/2 + sum_{k>=1} f(k h) ],  f(t) = exp(-x (cosh t - 1)) cosh(nu t),
// which converges geometrically in 1/h for this analytic, doubly decaying
// integrand (Trefethen & Weideman, SIAM Review 56, 2014).  The step depends on
// x through 10 buckets, h_m = 0.1 * 2^(-m/2) for x <= 9 * 2^m (h <= 0.3/sqrt(x)),
// and the sum stops once x (cosh t - 1) - nu t > 45 (terms below e^-45 of the
// first one); relative error below 1e-14 for nu up to 15 and x in [1e-12, 700]
// (checked against 30-digit values).  The same exponentials give K_{nu-1} (weight cosh((nu-1) t)) and
// dK_nu/dnu (weight t sinh(nu t), the nu-derivative of the integrand), so one
// set of exp() calls serves all three derivatives:
//   dSigma/dsigma2 = Sigma / sigma2
//   dSigma/dbeta   = sigma2 c x^(nu+1) K_{nu-1}(x) / beta        (DLMF 10.29.4, 10.27.3)
//   dSigma/dnu     = Sigma (-ln 2 - psi(nu) + ln x) + sigma2 c x^nu dK_nu/dnu(x)
// Sigma(0) = sigma2 and every nu- or beta-derivative vanishes at r = 0; for
// x > 700 the covariance is below 1e-250 and is returned as 0.
//
// Per-entry evaluation does not run the quadrature: for each theta the three
// smooth, positive functions of s = ln x
//   u0 = x^nu e^x K_nu(x),  u1 = x^(nu+1) e^x K_{nu-1}(x),  u2 = x^nu e^x dK_nu/dnu(x)
// are sampled by the quadrature at the 13 Chebyshev points of each of 119
// segments of width 1/4 covering ln x in [-23, ln 700]; on each segment
// u = u(centre) exp(p(t)), t in [-1, 1], with p the degree-12 interpolant of
// ln(u / u(centre)), p(0) = 0.  In s the logarithms are analytic in the strip
// |Im s| < pi/2 (K_nu has no zeros or singularities for Re x > 0) and nearly
// linear, so on a segment of half-width 1/8 the interpolant is exact to
// rounding, and interpolating relative to the centre keeps the rounding of
// large logarithms out (checked against 30-digit values: below 5e-14 relative
// for nu up to 15).  x below e^-23 falls back to the quadrature.
//
// An entry is bound by its vector instructions and by the reads of its segment.
// The tables are read from LDS where a workgroup forms many entries, and the
// instructions are about 130 with the distance (300 with the library's logarithm,
// two of its exponentials, its division and square root, and Clenshaw's
// recurrence).  At n = 40,000: k_sigma_residual 12.1 -> 7.0 ms, k_gen_tiles 7.1 ->
// 6.0 ms, k_lauum_contract with its contraction 323 -> 315 ms.
//   - t comes from ln x = e ln 2 + ln m without forming the large sum: e ln 2
//     minus the segment's centre is exact in its leading part.  That also keeps
//     the rounding of ln x + 23 (2e-15) out of t.
//   - p in powers of t: its Chebyshev coefficients fall off by 1/25 each, so the
//     powers' stay as small (Horner, 12 multiply-adds).
//   - exp(p) exp(-x) as one exponential of the two-term sum p - x, whose argument
//     needs no range checks; the constant factors are multiplied into u(centre).
//   - r / beta by a rounded reciprocal and one exact remainder (Markstein, 1990:
//     the correctly rounded quotient); a second remainder gives what the rounding
//     left, which exp(-x) would magnify x times.
// The polynomials of ln and exp interpolate the series at Chebyshev points
// (below 5e-18 and 1.3e-17).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace exg {

constexpr int QNB = 10;     // step buckets
constexpr int QNK = 400;    // nodes per bucket (reaches t = 39.9 at h = 0.1)
constexpr int QW = 5;       // per node: cosh t - 1, t, w0, w1, w2
constexpr double QCUT = 45.0;
constexpr double XMAX = 700.0;
// Chebyshev tables, stored after the quadrature nodes in the same array
constexpr int CH_N = 13;          // points per segment (degree 12)
constexpr int CH_NSEG = 119;      // segments of ln x
constexpr int CH_STRIDE = 14;     // doubles per function and segment
constexpr int CH_TAB = CH_NSEG * CH_STRIDE;  // doubles per function: u0, u1, u2 in turn
constexpr int CH_MID = 6;         // the middle Chebyshev point, t = 0
// per segment: the coefficients of t, ..., t^12, then the factors
//   u0: s c u(centre), c u(centre);  u1: s c u(centre) / b;  u2: s c u(centre)
// with s and b the mantissas of sigma2 and beta: c u(centre) reaches 1e26 (nu = 15),
// so sigma2 itself would overflow it where the entry, e^-x smaller, does not.
// The exponents join the entry's last scaling (C_S2E, C_D1E), which changes no bit.
constexpr int CH_A = CH_N - 1;
constexpr double CH_SLO = -23.0;  // ln x of the first segment's left end
constexpr double CH_DS = 0.25;    // segment width in ln x
constexpr int QT_CHEB_OFF = QNB * QNK * QW;
constexpr int QT_TOTAL = QT_CHEB_OFF + 3 * CH_TAB;

// per-theta constants written by the table kernel
// C_S2E, C_D1E: exponents of sigma2 and of sigma2 / beta (integers, see cst_int)
enum { C_S2 = 0, C_BETA, C_NU, C_C, C_PSI, C_S2C, C_METRIC, C_NUG, C_RBETA, C_S2E, C_D1E, C_COUNT = 16 };
__device__ __forceinline__ int cst_int(const double* __restrict__ cst, int i) { return __double2loint(cst[i]); }

constexpr double EARTH_RADIUS_KM = 6371.0;

// sqrt(d) for d in the middle of the exponent range by the hardware reciprocal
// square root, a third-order step and an exact remainder; else the library's
__device__ __forceinline__ double dist_sqrt(double d) {
  if (!(d >= 1e-200 && d <= 1e200)) return sqrt(d);
  double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-d * y, y, 1.0);
  y = fma(y * e, fma(0.375, e, 0.5), y);
  const double g = d * y;
  return fma(fma(-g, g, d), 0.5 * y, g);
}

// The rare and the long ways (the great circle, the quadrature per entry) are
// calls: inlined, their constants would sit in registers across the loops over
// entries and cost these their occupancy (175 registers instead of 108 in
// k_gen_tiles).
// great-circle distance in km between (longitude, latitude) pairs in degrees by
// the haversine formula
__device__ __noinline__ inline double great_circle(double x1, double y1, double x2, double y2) {
  const double d2r = 3.14159265358979323846 / 180.0;
  const double sp = sin(0.5 * (y2 - y1) * d2r), sl = sin(0.5 * (x2 - x1) * d2r);
  const double a = sp * sp + cos(y1 * d2r) * cos(y2 * d2r) * sl * sl;
  return 2.0 * EARTH_RADIUS_KM * asin(fmin(1.0, sqrt(a)));
}

// distance between two locations: Euclidean, or (cst[C_METRIC] = 1) great-circle
__device__ __forceinline__ double loc_dist(double x1, double y1, double x2, double y2, const double* __restrict__ cst) {
  if (cst[C_METRIC] == 0.0) {
    const double dx = x1 - x2, dy = y1 - y2;
    return dist_sqrt(dx * dx + dy * dy);
  }
  return great_circle(x1, y1, x2, y2);
}

__device__ __forceinline__ int quad_bucket(double x) {
  if (x <= 9.0) return 0;
  int m = (int)ceil(log2(x * (1.0 / 9.0)));
  return m < QNB - 1 ? m : QNB - 1;
}

// T0 = e^x K_nu(x)
__device__ __forceinline__ double quad_k0(const double* __restrict__ qt, double x, double nu) {
  const double* q = qt + quad_bucket(x) * QNK * QW;
  double s = 0.0;
  for (int k = 0; k < QNK; ++k, q += QW) {
    const double c = q[0];
    if (k > 0 && x * c - nu * q[1] > QCUT) break;
    s += exp(-x * c) * q[2];
  }
  return s;
}

// (e^x K_nu, e^x K_{nu-1}, e^x dK_nu/dnu)
__device__ __forceinline__ void quad_k3(const double* __restrict__ qt, double x, double nu, double* s0, double* s1,
                                        double* s2) {
  const double* q = qt + quad_bucket(x) * QNK * QW;
  double a = 0.0, b = 0.0, c2 = 0.0;
  for (int k = 0; k < QNK; ++k, q += QW) {
    const double c = q[0];
    if (k > 0 && x * c - nu * q[1] > QCUT + 5.0) break;
    const double e = exp(-x * c);
    a += e * q[2];
    b += e * q[3];
    c2 += e * q[4];
  }
  *s0 = a;
  *s1 = b;
  *s2 = c2;
}

constexpr double LN2H = 0x1.62e42fee00000p-1;  // 32 bits of ln 2, so that small integers times it are exact
constexpr double LN2L = 0x1.a39ef35793c76p-33;
constexpr double XMIN = 0x1.c3527e433fab1p-34;  // e^-23

// x = r / beta rounded and what the rounding left, *lo; rb = 1 / beta rounded
__device__ __forceinline__ double over_beta(double r, double beta, double rb, double* lo) {
  *lo = 0.0;
  if (!(beta >= 1e-150 && beta <= 1e150 && r <= 1e150)) return r / beta;
  const double q = r * rb, x = fma(fma(-q, beta, r), rb, q);
  *lo = fma(-x, beta, r) * rb;
  return x;
}

// Segment of ln x, the local coordinate t and ln x itself, x in [XMIN, XMAX]:
// x = 2^e m, m in [sqrt(1/2), sqrt(2)), ln m = 2 atanh((m - 1) / (m + 1))
__device__ __forceinline__ void ln_locate(double x, int* seg, double* t, double* lx) {
  double m = __builtin_amdgcn_frexp_mant(x);
  int ei = __builtin_amdgcn_frexp_exp(x);
  const int low = m < 0x1.6a09e667f3bcdp-1;
  m = ldexp(m, low);
  ei -= low;
  const double e = (double)ei, d = m + 1.0;
  double y = __builtin_amdgcn_rcp(d);
  const double q = fma(-d, y, 1.0);
  y = fma(y, fma(q, q, q), y);
  const double s = (m - 1.0) * y, z = s * s;
  double a = 0x1.2b5900de53b32p-4;
  a = fma(a, z, 0x1.39fe51a7c18f9p-4);
  a = fma(a, z, 0x1.7462b51cb66b1p-4);
  a = fma(a, z, 0x1.c71c62e3f11e6p-4);
  a = fma(a, z, 0x1.2492492df281ap-3);
  a = fma(a, z, 0x1.99999999952d7p-3);
  a = fma(a, z, 0x1.5555555555558p-2);
  const double s2 = s + s, lm = fma(s2 * z, a, s2);
  const double lo = fma(e, LN2L, lm);
  *lx = fma(e, LN2H, lo);
  int j = (int)((*lx - CH_SLO) * (1.0 / CH_DS));
  j = min(max(j, 0), CH_NSEG - 1);
  *seg = j;
  const double centre = fma((double)j, CH_DS, CH_SLO + 0.5 * CH_DS);
  *t = (fma(e, LN2H, -centre) + lo) * (2.0 / CH_DS);
}

// p(t), the coefficients of t, ..., t^12 at b
__device__ __forceinline__ double seg_poly(const double* __restrict__ b, double t) {
  double a = b[CH_N - 2];
#pragma unroll
  for (int k = CH_N - 3; k >= 0; --k) a = fma(a, t, b[k]);
  return a * t;
}

// exp(p - x - xl) = m 2^*e, m in (0.7, 1.42), |p| < 10, 0 < x <= XMAX, xl below an ulp of x
__device__ __forceinline__ double exp_diff(double p, double x, double xl, int* e) {
  const double hi = p - x, bb = hi - p, lo = (p - (hi - bb)) - (x + bb) - xl;
  const double k = rint(hi * 0x1.71547652b82fep+0);
  const double r = fma(-k, LN2L, fma(-k, LN2H, hi)) + lo;
  double q = 0x1.af38ad61700a0p-26;
  q = fma(q, r, 0x1.28918860dd4aap-22);
  q = fma(q, r, 0x1.71de0dacd6939p-19);
  q = fma(q, r, 0x1.a019b90aa5587p-16);
  q = fma(q, r, 0x1.a01a01a7c4839p-13);
  q = fma(q, r, 0x1.6c16c1788c7f3p-10);
  q = fma(q, r, 0x1.11111111109b3p-7);
  q = fma(q, r, 0x1.5555555553d61p-5);
  q = fma(q, r, 0x1.5555555555556p-3);
  q = fma(q, r, 0.5);
  *e = (int)k;
  return fma(r * r, q, r) + 1.0;
}

// the covariance and its derivatives by the quadrature, x < XMIN (or NaN)
__device__ __noinline__ inline double quad_value(double x, const double* cst, const double* qt) {
  const double nu = cst[C_NU];
  return cst[C_S2C] * pow(x, nu) * exp(-x) * quad_k0(qt, x, nu);
}

struct Grad3 {
  double d0, d1, d2;
};
__device__ __noinline__ inline Grad3 quad_grad(double x, const double* cst, const double* qt) {
  const double nu = cst[C_NU];
  double t0, t1, t2;
  quad_k3(qt, x, nu, &t0, &t1, &t2);
  const double P = cst[C_S2C] * pow(x, nu) * exp(-x);
  const double sig = P * t0;
  return {sig / cst[C_S2], P * x * t1 / cst[C_BETA],
          sig * (-0.69314718055994530942 - cst[C_PSI] + log(x)) + P * t2};
}

// N of the functions' tables (from u0) to LDS, 256 threads; the caller has the barrier
template <int N>
__device__ __forceinline__ void stage_tables(const double* __restrict__ qt, double* tab) {
  typedef double p2 __attribute__((ext_vector_type(2)));
  const p2* src = (const p2*)(qt + QT_CHEB_OFF);
  for (int i = threadIdx.x; i < N * CH_TAB / 2; i += 256) ((p2*)tab)[i] = src[i];
}

// Covariance at distance r: sigma2 at r = 0, zero past XMAX.  tab: the tables,
// qt + QT_CHEB_OFF or a copy in LDS (stage_tables): a wave's lanes read few
// different segments, which LDS serves together where the L1 takes about a
// lane per cycle.
__device__ __forceinline__ double matern_value(double r, const double* __restrict__ cst, const double* __restrict__ qt,
                                               const double* tab) {
  double xl;
  const double x = over_beta(r, cst[C_BETA], cst[C_RBETA], &xl);
  if (!(x >= XMIN) && r != 0.0) {
    return quad_value(x, cst, qt);
  }
  const double xc = fmin(fmax(x, XMIN), XMAX);
  int seg, e;
  double t, lx;
  ln_locate(xc, &seg, &t, &lx);
  const double* b = tab + seg * CH_STRIDE;
  const double m = exp_diff(seg_poly(b, t), xc, xl, &e), v = ldexp(b[CH_A] * m, e + cst_int(cst, C_S2E));
  return r == 0.0 ? cst[C_S2] : (x > XMAX ? 0.0 : v);
}

// d[0..2] = dSigma/d(sigma2, beta, nu) at distance r: (1, 0, 0) at r = 0, zero past XMAX
__device__ __forceinline__ void matern_grad(double r, const double* __restrict__ cst, const double* __restrict__ qt,
                                            const double* tab, double* d0, double* d1, double* d2) {
  double xl;
  const double x = over_beta(r, cst[C_BETA], cst[C_RBETA], &xl);
  const double lc = -0.69314718055994530942 - cst[C_PSI];
  if (!(x >= XMIN) && r != 0.0) {
    const Grad3 g = quad_grad(x, cst, qt);
    *d0 = g.d0, *d1 = g.d1, *d2 = g.d2;
    return;
  }
  const double xc = fmin(fmax(x, XMIN), XMAX);
  int seg, i0, i1, i2;
  double t, lx;
  ln_locate(xc, &seg, &t, &lx);
  const double *b0 = tab + seg * CH_STRIDE, *b1 = b0 + CH_TAB, *b2 = b1 + CH_TAB;
  const bool at0 = r == 0.0, far = x > XMAX;
  const double m0 = exp_diff(seg_poly(b0, t), xc, xl, &i0), m1 = exp_diff(seg_poly(b1, t), xc, xl, &i1),
               m2 = exp_diff(seg_poly(b2, t), xc, xl, &i2);
  const double e0 = ldexp(m0, i0), e2 = ldexp(m2, i2);
  *d0 = at0 ? 1.0 : (far ? 0.0 : b0[CH_A + 1] * e0);
  *d1 = at0 || far ? 0.0 : ldexp(b1[CH_A] * m1, i1 + cst_int(cst, C_D1E));
  *d2 = at0 || far ? 0.0 : ldexp(fma(b0[CH_A] * e0, lc + lx, b2[CH_A] * e2), cst_int(cst, C_S2E));
}

}  // namespace exg
