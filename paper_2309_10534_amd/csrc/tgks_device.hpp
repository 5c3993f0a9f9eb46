// tgks_device.hpp -- device math of the TENO-D gas-kinetic scheme (gfx950, FP64).
//
// Mu et al., "High-order gas-kinetic scheme with TENO class reconstruction for
// the Euler and Navier-Stokes equations", arXiv:2309.10534.
//
//   * TENO-D selection and candidate values (Sec. 4.2, Eqs. 4.5-4.14; the
//     candidate polynomials of Sec. 3.1-3.2, slopes Eqs. 3.22-3.24).
//   * Tangential Gauss-point reconstruction (Sec. 3.2 Steps 1-3).
//   * Gas-kinetic flux at one Gauss point (Sec. 2.1, Eqs. 2.2-2.9 with the
//     kinetic weighting of Eqs. 3.25-3.26), in closed form: moments of the
//     normal velocity by the half-space erfc/exp recursion, micro slopes from
//     primitive derivatives in the frame of the tangential velocity.
//
// The selection arithmetic (smoothness indicators, gamma_k, cut-offs) and the
// candidate values follow one fixed evaluation order (constant divisors as
// multiplications by their correctly rounded reciprocals) with floating-point
// contraction disabled, so that the stencil flags are a deterministic
// function of the input bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

// Every function is a template on the scalar type R: double in the kernels,
// an operation-counting type on the host (algorithmic flop counts).
#define TGKS_HD __host__ __device__ __forceinline__

namespace tgks {

// bits of TenoCfg::fast
constexpr int TENO_RATIO_OK = 1;   // the fixed ratios of teno_flag hold (teno_cfg)
constexpr int TENO_FILTER_OK = 2;  // the multiplied-out comparisons of teno_select are valid

struct TenoCfg {
  double ct1, ct2, eps;
  int q;
  int fast;  // TENO_RATIO_OK | TENO_FILTER_OK where they hold (teno_cfg)
  // for the certain decisions: 4 eps, and the cut-offs times 1 +- 2^-30
  double eps4, ct1_up, ct1_dn, ct2_up, ct2_dn;
};

// The selection parameters, with the fast bits set where teno_flag's
// shortcuts are exact.
//
// TENO_RATIO_OK, fixed ratios of the certain decisions.  With b_k = beta_k
// + eps, gamma_k = b_k^-7 (q = 7) and m = min(b_0, b_1, b_2), whose gamma
// is the largest of the small stencils':
//   b_3 <= 4 m: gamma_3 / sum_{k<=3} gamma >= 1 / (3 4^7 + 1) (the three
//       small gammas at most gamma_max each): the large stencil is kept
//       (Eq. 4.7) if C_T1 <= 1 / (3 4^7 + 1) = 2.03e-5;
//   b_3 > 16 m: gamma_3 / sum < 1 / (16^7 + 1) (the sum holds gamma_max):
//       rejected if C_T1 >= 1 / (16^7 + 1) = 3.7e-9;
//   then b_k <= 4 m: gamma_k / sum_{k<3} gamma >= 1 / (2 4^7 + 1): kept
//       (Eq. 4.12) if C_T2 <= 3.05e-5; b_k > 8 m: gamma_k / sum <
//       1 / (8^7 + 1): dropped if C_T2 >= 4.8e-7.
// Each bound is reached in the limit (equal small indicators for the keeps,
// the other small stencils infinitely rough for the rejections).  The
// ratios are powers of two (exact products), and the cut-offs must clear
// each bound by a relative 1e-9, far above the rounding of the weights'
// evaluation (a few ulps of b^7, its reciprocal and the sums).  Also
// q = 7 and eps >= 1e-40 (b^7 and 1 / b^7 stay finite and normal).  The
// paper's C_T1 = 1e-7, C_T2 = 1e-5 are inside.
//
// TENO_FILTER_OK, the weights' comparisons multiplied out, with a margin
// (teno_select): q = 7, 1e-40 <= eps < 1e40 and 1e-20 <= C_T1, C_T2 <= 1/2
// (the smallest indicator is scaled into [1, 2) and all are cut at 2048, so one
// is cut from 1024 times the smallest on, at a weight below 1024^-7 = 8.5e-22 of
// the largest: a twelfth of the smallest cut-off allowed).
inline TenoCfg teno_cfg(double ct1, double ct2, double eps, int q) {
  const double d = 1e-9;
  const bool ok = q == 7 && eps >= 1e-40 && ct1 * (1.0 + d) <= 1.0 / (3.0 * 16384.0 + 1.0) &&
                  ct1 * (1.0 - d) >= 1.0 / (268435456.0 + 1.0) && ct2 * (1.0 + d) <= 1.0 / (2.0 * 16384.0 + 1.0) &&
                  ct2 * (1.0 - d) >= 1.0 / (2097152.0 + 1.0);
  const bool filt = q == 7 && eps >= 1e-40 && eps < 1e40 && ct1 >= 1e-20 && ct1 <= 0.5 && ct2 >= 1e-20 &&
                    ct2 <= 0.5;
  const double up = 1.0 + 0x1p-30, dn = 1.0 - 0x1p-30;
  return TenoCfg{ct1, ct2, eps, q, (ok ? TENO_RATIO_OK : 0) | (filt ? TENO_FILTER_OK : 0),
                 4.0 * eps, ct1 * up, ct1 * dn, ct2 * up, ct2 * dn};
}

// An approximate reciprocal: the device's one-instruction estimate.  On the
// host, 1 / x with the low 29 bits of the significand cleared (relative error
// up to 2^-23), so that host checks exercise the same refinement.
TGKS_HD double rcp_approx(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcp(x);
#else
  double r = 1.0 / x;
  uint64_t u;
  __builtin_memcpy(&u, &r, sizeof u);
  u &= ~((uint64_t(1) << 29) - 1);
  __builtin_memcpy(&r, &u, sizeof r);
  return r;
#endif
}

// 1/x to about one ulp (not always correctly rounded): the estimate and two
// Newton steps, each of which squares its relative error; for quantities
// that feed only the flux.  0 and infinities give NaN (the states they come
// from are rejected as non-physical).  The operation-counting type counts
// one division.
template <class R>
TGKS_HD R recip(R x) {
  return R(1.0) / x;
}
TGKS_HD double recip(double x) {
  double r = rcp_approx(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// a b + c, rounded once in double
template <class R>
TGKS_HD R fma_(R a, R b, R c) {
  return a * b + c;
}
TGKS_HD double fma_(double a, double b, double c) { return fma(a, b, c); }

// ---------------------------------------------------------------------------
// Differences of five values Q_{-2..2} = a..e that the selection and the
// Gauss-point values share: x = d - b; second differences t[k] of the three
// small stencils; one-sided slopes l0 = a - 4 b + 3 c, l2 = 3 c - 4 d + e;
// y = e - a; third and fourth differences y3, y4.  Each is evaluated in the
// oracle's order (a product by 2 or 4 is exact, so the fma rounds as the
// separate operations do): where the data are constant up to rounding, the
// selection is decided by their rounding residues.
// ---------------------------------------------------------------------------
template <class R>
struct TenoParts {
  R b, c, d, x, t[3], l0, l2, y, y3, y4;
};

template <class R>
TGKS_HD void teno_parts(const R* Q, TenoParts<R>& p) {
#pragma clang fp contract(off)
  const R a = Q[0], b = Q[1], c = Q[2], d = Q[3], e = Q[4];
  const R c3 = 3.0 * c, f = fma_(R(-4.0), b, a);
  p.b = b;
  p.c = c;
  p.d = d;
  p.x = d - b;
  p.t[0] = fma_(R(-2.0), b, a) + c;
  p.t[1] = fma_(R(-2.0), c, b) + d;
  p.t[2] = fma_(R(-2.0), d, c) + e;
  p.l0 = f + c3;
  p.l2 = fma_(R(-4.0), d, c3) + e;
  p.y = e - a;
  p.y3 = fma_(R(-2.0), p.x, p.y);
  p.y4 = fma_(R(-4.0), d, f + 6.0 * c) + e;
}

// Whether the large stencil is kept for certain (true only where it is), from
// the shared second differences alone; needs the fixed ratios of teno_cfg
// (TENO_RATIO_OK).  EQ: also true for five equal values, where every
// candidate polynomial is the constant and the selection does not matter.
//
// With e_a = t1 - t0, e_b = t2 - t1 the third differences and N^2 = x^2 +
// 13/3 t1^2 = 4 beta_1, the other indicators are 4 beta_0 = (x - e_a)^2 +
// 13/3 (t1 - e_a)^2, 4 beta_2 = (x - e_b)^2 + 13/3 (t1 + e_b)^2 and 4 beta_3 =
// (x - y3/6)^2 + 13/3 (t1 - 0.0846 y4)^2 + 781/720 y3^2 + 4.339 y4^2, y3 =
// e_a + e_b, y4 = e_b - e_a.  If |e_a|, |e_b| <= r N then sqrt(4 beta_0),
// sqrt(4 beta_2) >= (1 - 2.31 r) N and sqrt(4 beta_3) <= (1 + 4.52 r) N, so at
// r = 1/10 beta_3 <= 3.57 min(beta_0, beta_1, beta_2): the large stencil is
// kept (ratio 4 of teno_cfg).  N >= 2^-29 |c| keeps the rounding of every
// indicator (20 ulps of the values, here and in the oracle's order) below
// 2^-18 N, far inside the margin; data with less variation than that is left
// to the general evaluation, and so is data whose indicators leave the range
// of teno_cfg (N^2 < 1e39: all four are then below 1e39; beyond 1e154 the
// squares here would be infinite and any data pass for smooth).
template <bool EQ>
TGKS_HD bool teno_smooth(const TenoParts<double>& p) {
#pragma clang fp contract(off)
  const double ea = p.t[1] - p.t[0], eb = p.t[2] - p.t[1];
  const double n = fma(13.0 / 3.0, p.t[1] * p.t[1], p.x * p.x), cs = p.c * 0x1p-29;
  // both within r N: by the sum of their squares, which a NaN in either fails
  const bool small = (fma(eb, eb, ea * ea) <= 0.01 * n) & (n < 1e39);
  const bool seen = cs * cs <= n;
  return EQ ? small & (seen | (n == 0.0)) : small & seen;
}

// A selection: the large stencil, or the surviving small ones.
struct TenoSel {
  bool lg, k0, k1, k2;
  // bit0 = delta_{3,1}; if it is 0, bits 1..3 = delta_{0,2}, delta_{1,2}, delta_{2,2}
  TGKS_HD unsigned flag() const { return lg ? 1u : (k0 ? 2u : 0u) | (k1 ? 4u : 0u) | (k2 ? 8u : 0u); }
};

TGKS_HD TenoSel teno_sel(unsigned flag) {
  return TenoSel{(flag & 1u) != 0, (flag & 2u) != 0, (flag & 4u) != 0, (flag & 8u) != 0};
}

// ---------------------------------------------------------------------------
// TENO-D selection (Sec. 4.2), a function of the input bits.
//
// teno_exact: the weights gamma_k = (beta_k + eps)^-q by correctly rounded
// divisions, summed and compared in one fixed order.  teno_select reaches
// the same selection, bit for bit, with less work where the decision is
// certain, and calls teno_exact where it is not:
//
// SEL_FILTER (the 1-D and 2-D kernels): the comparisons multiplied out, no
// division.  b_k = 4 (beta_k + eps) as sums of squares of the shared
// differences (fused multiply-adds; every term is positive, and s1, s2 lose
// at most what y3, y4 hold beside them, so each b_k is within 100 rounding
// errors of the oracle's); scaled by a power of two so that the smallest of
// b_0..b_2 is in [1, 2) and cut at 2048 (t_k); p_k = t_k^7.  With
// P = p_0 p_1 p_2 and S = p_0 p_1 + p_1 p_2 + p_0 p_2 the weights are
// p_j p_k / P and 1 / p_3, so
//   gamma_3 >= C_T1 sum       <=>  P >= C_T1 (S p_3 + P),
//   gamma_i >= C_T2 sum_{k<3} <=>  p_j p_k >= C_T2 S.
// Both sides are within 2^-41 of the oracle's, and a comparison is certain
// when it holds with the cut-off times 1 +- 2^-30 on either side; an
// undecided input (within 1e-9 of a cut-off, a NaN, indicators >= 1e40)
// takes teno_exact.  All comparisons are evaluated (bitwise operators, no
// short-circuit branches), so that one rarely taken branch remains.
// 105 vector instructions where four reciprocal estimates with their
// measured residuals took 129, of which the estimates issue over four
// cycles each.  With the branch-free Gauss-point values (teno_poly) and the
// exact weights called instead of inlined, 20 steps of the 2-D four-quadrant
// problem at 1024^2 take 18.2 ms (21.9 before), 2 steps of the 3-D
// Taylor-Green vortex at 128^3 24.4 ms (25.1).
//
// SEL_RATIO (3-D normal reconstruction and first sweep): the fixed ratios of
// teno_cfg first (when TENO_RATIO_OK; no powers at all), taken where they
// decide for every lane of the wavefront: smooth data keeps the large
// stencil; constant data (the quadratics' indicators vanish exactly, the
// quartic's keeps a rounding residue) rejects it with the quadratics kept.
// Then as SEL_FILTER.
//
// The operation-counting type always evaluates the exact weights.
// ---------------------------------------------------------------------------
constexpr int SEL_EXACT = 0, SEL_FILTER = 1, SEL_RATIO = 2;

template <class R>
TGKS_HD unsigned teno_exact(const R* Q, const TenoCfg& c) {
#pragma clang fp contract(off)
  const R a = Q[0], b = Q[1], cc = Q[2], d = Q[3], e = Q[4];
  const double k13 = 13.0 / 12.0;
  R t1, t2, beta[4];
  t1 = (a - 2.0 * b) + cc;
  t2 = (a - 4.0 * b) + 3.0 * cc;
  beta[0] = k13 * (t1 * t1) + 0.25 * (t2 * t2);
  t1 = (b - 2.0 * cc) + d;
  t2 = b - d;
  beta[1] = k13 * (t1 * t1) + 0.25 * (t2 * t2);
  t1 = (cc - 2.0 * d) + e;
  t2 = (3.0 * cc - 4.0 * d) + e;
  beta[2] = k13 * (t1 * t1) + 0.25 * (t2 * t2);
  // quartic indicator (Eq. 3.7, q = 4) as a sum of squares of its derivatives
  const R P1 = (82.0 * (d - b) - 11.0 * (e - a)) * (1.0 / 120.0);
  const R P2 = ((((40.0 * b - 3.0 * a) - 74.0 * cc) + 40.0 * d) - 3.0 * e) * (1.0 / 56.0);
  const R P3 = ((e - a) - 2.0 * (d - b)) * (1.0 / 12.0);
  const R P4 = ((((a - 4.0 * b) + 6.0 * cc) - 4.0 * d) + e) * (1.0 / 24.0);
  const R s1 = P1 + P3 * (1.0 / 10.0);
  const R s2 = P2 + (123.0 / 455.0) * P4;
  beta[3] = (((s1 * s1) + (13.0 / 3.0) * (s2 * s2)) + (781.0 / 20.0) * (P3 * P3)) +
            (1421461.0 / 2275.0) * (P4 * P4);
  R g[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const R bb = beta[k] + c.eps;
    R pw;
    if (c.q == 7) {
      const R b2 = bb * bb;
      const R b4 = b2 * b2;
      pw = (b4 * b2) * bb;
    } else {
      pw = R(1.0);
      for (int r = 0; r < c.q; ++r) pw = pw * bb;
    }
    g[k] = 1.0 / pw;  // gamma_k = (beta_k + eps)^-q  (Eq. 4.5)
  }
  const R s4 = ((g[0] + g[1]) + g[2]) + g[3];
  if (!(g[3] < c.ct1 * s4)) return 1u;  // large stencil kept (Eqs. 4.6-4.7)
  const R s3 = (g[0] + g[1]) + g[2];
  unsigned f = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (!(g[k] < c.ct2 * s3)) f |= 2u << k;  // Eqs. 4.11-4.12
  return f;
}

// 2^-e for a normal x in [2^e, 2^(e+1)), e > -1023: the exponent mirrored
TGKS_HD double scale_of(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __hiloint2double(0x7fe00000 - (__double2hiint(x) & 0x7ff00000), 0);
#else
  uint64_t u;
  __builtin_memcpy(&u, &x, sizeof u);
  u = 0x7fe0000000000000ull - (u & 0x7ff0000000000000ull);
  double r;
  __builtin_memcpy(&r, &u, sizeof r);
  return r;
#endif
}

// whether x holds in every active lane of the wavefront (the host: of one)
TGKS_HD bool all_lanes(bool x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ballot_w64(!x) == 0;
#else
  return x;
#endif
}

// the certain decisions; false where the exact weights have to decide
template <int MODE>
TGKS_HD bool teno_certain(const double* Q, const TenoParts<double>& p, const TenoCfg& c, TenoSel& s) {
#pragma clang fp contract(off)
  // Y2 = 56 P2 of the quartic indicator in the oracle's order; s1 = 12 (P1 +
  // P3 / 10), s2 = 56 (P2 + 123/455 P4)
  const double Y2 = (((40.0 * Q[1] - 3.0 * Q[0]) - 74.0 * Q[2]) + 40.0 * Q[3]) - 3.0 * Q[4];
  const double s1 = fma(8.0, p.x, -p.y), s2 = fma(41.0 / 65.0, p.y4, Y2);
  const double k = 13.0 / 3.0;
  const double b0 = fma(k, p.t[0] * p.t[0], fma(p.l0, p.l0, c.eps4));
  const double b1 = fma(k, p.t[1] * p.t[1], fma(p.x, p.x, c.eps4));
  const double b2 = fma(k, p.t[2] * p.t[2], fma(p.l2, p.l2, c.eps4));
  const double b3 = fma(13.0 / 2352.0, s2 * s2,
                        fma(1.0 / 36.0, s1 * s1,
                            fma(1421461.0 / 327600.0, p.y4 * p.y4, fma(781.0 / 720.0, p.y3 * p.y3, c.eps4))));
  const double m = fmin(fmin(b0, b1), b2);
  // a NaN or an infinite input makes b3 a NaN or infinite
  const bool inr = (b3 < 1e40) & (m < 1e40);
  if (MODE == SEL_RATIO) {
    if (c.fast & TENO_RATIO_OK) {
      const double lo = 4.0 * m, hi = 8.0 * m;
      const bool k0 = b0 <= lo, k1 = b1 <= lo, k2 = b2 <= lo, keep = b3 <= lo;
      const bool sure = inr & (keep | ((b3 > 16.0 * m) & (k0 | (b0 > hi)) & (k1 | (b1 > hi)) & (k2 | (b2 > hi))));
      if (all_lanes(sure)) {
        s = TenoSel{keep, k0, k1, k2};
        return true;
      }
    }
  }
  if (!(c.fast & TENO_FILTER_OK)) return false;
  const double sc = scale_of(m);
  const double bb[4] = {b0, b1, b2, b3};
  double q[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double t = fmin(bb[i] * sc, 2048.0);
    const double t2 = t * t;
    q[i] = (t2 * t2) * (t2 * t);
  }
  const double q01 = q[0] * q[1], q12 = q[1] * q[2], q02 = q[0] * q[2];
  const double S = (q01 + q12) + q02, P = q01 * q[2];
  const double X = fma(S, q[3], P);
  const double hi = S * c.ct2_up, lo = S * c.ct2_dn;
  const bool keep = P > X * c.ct1_up, rej = P < X * c.ct1_dn;
  const bool k0 = q12 > hi, k1 = q02 > hi, k2 = q01 > hi;
  const bool sure = inr & (keep | (rej & (k0 | (q12 < lo)) & (k1 | (q02 < lo)) & (k2 | (q01 < lo))));
  s = TenoSel{keep, k0, k1, k2};
  return sure;
}

// teno_exact as a function of its own: the rare path of the kernels, called
// so that its code (four divisions, a power loop) stands once beside their
// straight-line code
__host__ __device__ __attribute__((noinline)) inline unsigned teno_exact_cold(double a, double b, double cc, double d,
                                                                              double e, double ct1, double ct2,
                                                                              double eps, int q) {
  const double Q[5] = {a, b, cc, d, e};
  TenoCfg c{};
  c.ct1 = ct1;
  c.ct2 = ct2;
  c.eps = eps;
  c.q = q;
  return teno_exact(Q, c);
}
TGKS_HD unsigned teno_exact_cold(const double* Q, const TenoCfg& c) {
  return teno_exact_cold(Q[0], Q[1], Q[2], Q[3], Q[4], c.ct1, c.ct2, c.eps, c.q);
}

// COLD: the exact weights called (for a kernel with several selections)
template <int MODE, bool COLD, class R>
TGKS_HD TenoSel teno_select(const R* Q, const TenoParts<R>& p, const TenoCfg& c) {
  if constexpr (MODE != SEL_EXACT && std::is_same_v<R, double>) {
    TenoSel s;
    if (!teno_certain<MODE>(Q, p, c, s)) s = teno_sel(COLD ? teno_exact_cold(Q, c) : teno_exact(Q, c));
    return s;
  } else {
    return teno_sel(teno_exact(Q, c));
  }
}

// the flag alone: bit0 = delta_{3,1}; if it is 0, bits 1..3 = delta_{0,2},
// delta_{1,2}, delta_{2,2}
template <int MODE = SEL_EXACT, bool COLD = false, class R>
TGKS_HD unsigned teno_flag(const R* Q, const TenoCfg& c) {
  TenoParts<R> p;
  if constexpr (MODE != SEL_EXACT && std::is_same_v<R, double>) teno_parts(Q, p);
  return teno_select<MODE, COLD>(Q, p, c).flag();
}

// Values and slopes (cell units) at x_{i-1/2} and x_{i+1/2} of the selected
// reconstruction: out = {v(-1/2), s(-1/2), v(+1/2), s(+1/2)}.
template <class R>
TGKS_HD void teno_face(const R* Q, unsigned flag, R* out) {
#pragma clang fp contract(off)
  const R a = Q[0], b = Q[1], c = Q[2], d = Q[3], e = Q[4];
  if (flag & 1u) {
    // Eq. 4.8, Eq. 4.9 and their mirror images
    // (fma with a power of two: the product is exact, so the result is that
    // of the separate multiplication and addition)
    out[2] = (((fma_(R(2.0), a, -(13.0 * b)) + 47.0 * c) + 27.0 * d) - 3.0 * e) * (1.0 / 60.0);
    out[3] = (((b - 15.0 * c) + 15.0 * d) - e) * (1.0 / 12.0);
    out[0] = fma_(R(2.0), e, ((27.0 * b - 3.0 * a) + 47.0 * c) - 13.0 * d) * (1.0 / 60.0);
    out[1] = (((a - 15.0 * b) + 15.0 * c) - d) * (1.0 / 12.0);
    return;
  }
  // surviving small stencils averaged with d_k = 1/3 (Eqs. 4.13-4.14)
  // omega_k = d_k delta_k / sum d_k delta_k with d_k = 1/3: in double
  // arithmetic (1/3)/(m/3) is exactly 1, 0.5 or (1/3) for m = 1, 2, 3
  // surviving stencils
  const int cnt = (int)((flag >> 1) & 1u) + (int)((flag >> 2) & 1u) + (int)((flag >> 3) & 1u);
  const double om = cnt == 1 ? 1.0 : (cnt == 2 ? 0.5 : 1.0 / 3.0);
  const R o0 = R((flag & 2u) ? om : 0.0), o1 = R((flag & 4u) ? om : 0.0), o2 = R((flag & 8u) ? om : 0.0);
  const R vp0 = (fma_(R(2.0), a, -(7.0 * b)) + 11.0 * c) * (1.0 / 6.0);
  const R vp1 = fma_(R(2.0), d, 5.0 * c - b) * (1.0 / 6.0);
  const R vp2 = (fma_(R(2.0), c, 5.0 * d) - e) * (1.0 / 6.0);
  const R dp0 = fma_(R(2.0), c, a - 3.0 * b);
  const R dp12 = d - c;
  const R vm0 = fma_(R(2.0), c, 5.0 * b - a) * (1.0 / 6.0);
  const R vm1 = (fma_(R(2.0), b, 5.0 * c) - d) * (1.0 / 6.0);
  const R vm2 = fma_(R(2.0), e, 11.0 * c - 7.0 * d) * (1.0 / 6.0);
  const R dm01 = c - b;
  const R dm2 = fma_(R(-2.0), c, 3.0 * d) - e;
  out[0] = (o0 * vm0 + o1 * vm1) + o2 * vm2;
  out[1] = (o0 * dm01 + o1 * dm01) + o2 * dm2;
  out[2] = (o0 * vp0 + o1 * vp1) + o2 * vp2;
  out[3] = (o0 * dp0 + o1 * dp12) + o2 * dp12;
}

// teno_face with both kinds evaluated and one selected, to the same bits: one
// straight line for a kernel whose few wavefronts wait for their own results
// (several cells' values can then be evaluated in turn).
template <class R>
TGKS_HD void teno_face_both(const R* Q, const TenoSel& s, R* out) {
  R lg[4], sm[4];
  teno_face(Q, 1u, lg);
  teno_face(Q, (s.k0 ? 2u : 0u) | (s.k1 ? 4u : 0u) | (s.k2 ? 8u : 0u), sm);
#pragma unroll
  for (int k = 0; k < 4; ++k) out[k] = s.lg ? lg[k] : sm[k];
}

// The selected polynomial at the Gauss points +-s, s = 1/(2 sqrt 3) (cell
// units): p(+-s) = base +- odd, p'(+-s) = ev +- od.
//
// s^2 = 1/12, so a quadratic with cell average c takes the values
// c +- s p'(0) there, and the quartic of the five averages the values
// c - y4 / 4320 +- s (x / 2 - 7/72 y3) with the derivatives
// (x / 2 - y3 / 12) +- s (t1 - y4 / 9): the middle quadratic (slope x / 2,
// second difference t1) plus terms in the third and fourth differences.  One
// branch-free form therefore serves both: the surviving quadratics' mean
// (large stencil: the middle one alone) plus those terms where the large
// stencil is kept.  About 35 operations, most of them on differences that
// the selection has formed; a branch per kind took 66 in wavefronts that mix
// them.  The one-sided slopes and the fourth difference are formed from the
// second differences here: constant data then has no rounding residue at
// all (the selection's own have one, in the oracle's order), so a flow that
// is uniform along the face stays so to the last bit.
template <class R>
struct TenoPoly {
  R base, odd, ev, od;
};

// l: twice the slope, t: second difference of the quadratic; y3, y4: third and
// fourth differences of the large stencil, or 0
template <class R>
TGKS_HD void teno_poly_at(R c, R l, R t, R y3, R y4, TenoPoly<R>& o) {
#pragma clang fp contract(off)
  const double h = 0.28867513459481288225;  // s = 1/(2 sqrt 3)
  o.base = fma_(y4, R(-1.0 / 4320.0), c);
  o.odd = (0.5 * h) * fma_(y3, R(-7.0 / 36.0), l);
  o.ev = 0.5 * fma_(y3, R(-1.0 / 6.0), l);
  o.od = h * fma_(y4, R(-1.0 / 9.0), t);
}

// the large stencil's, as teno_poly evaluates it (to the bit)
template <class R>
TGKS_HD void teno_poly_large(const TenoParts<R>& p, TenoPoly<R>& o) {
#pragma clang fp contract(off)
  teno_poly_at<R>(p.c, p.x, p.t[1], p.t[2] - p.t[0], fma_(R(-2.0), p.t[1], p.t[0] + p.t[2]), o);
}

template <class R>
TGKS_HD void teno_poly(const TenoParts<R>& p, const TenoSel& s, TenoPoly<R>& o) {
#pragma clang fp contract(off)
  const R z = R(0.0), one = R(1.0);
  const R o0 = !s.lg && s.k0 ? one : z, o1 = s.lg || s.k1 ? one : z, o2 = !s.lg && s.k2 ? one : z;
  const R l0 = fma_(R(2.0), p.c - p.b, p.t[0]), l2 = fma_(R(2.0), p.d - p.c, -p.t[2]);
  const R y3 = s.lg ? p.t[2] - p.t[0] : z, y4 = s.lg ? fma_(R(-2.0), p.t[1], p.t[0] + p.t[2]) : z;
  // 1/(m + 1) for m = 0 (exactly), 1, 2 further stencils: 1 - 2/3 m + m^2/6
  const R m = ((o0 + o1) + o2) - 1.0;
  const R inv = fma_(m, fma_(m, R(1.0 / 6.0), R(-2.0 / 3.0)), one);
  const R l = fma_(o2, l2, fma_(o1, p.x, o0 * l0)) * inv;
  const R t = fma_(o2, p.t[2], fma_(o1, p.t[1], o0 * p.t[0])) * inv;
  teno_poly_at<R>(p.c, l, t, y3, y4, o);
}

// Selected polynomial at the Gauss points: val[m], der[m] for m = 0 (s-) and
// 1 (s+).  The values feed only the flux.
template <class R>
TGKS_HD void teno_gauss(const R* Q, unsigned flag, R* val, R* der) {
  TenoParts<R> p;
  TenoPoly<R> o;
  teno_parts(Q, p);
  teno_poly(p, teno_sel(flag), o);
  val[0] = o.base - o.odd;
  val[1] = o.base + o.odd;
  der[0] = o.ev - o.od;
  der[1] = o.ev + o.od;
}

// teno_gauss in one fixed evaluation order without contraction: the 3-D
// first sweep's Gauss-point values are the inputs of the second sweep's
// selections, whose flags must be a deterministic function of the data.
template <class R>
TGKS_HD void teno_gauss_exact(const R* Q, unsigned flag, R* val, R* der) {
#pragma clang fp contract(off)
  const R a = Q[0], b = Q[1], c = Q[2], d = Q[3], e = Q[4];
  const double s = 0.28867513459481288225;  // 1/(2 sqrt 3)
  R c0, c1, c2, c3 = R(0.0), c4 = R(0.0);
  if (flag & 1u) {
    c0 = ((2134.0 * c - 116.0 * (d + b)) + 9.0 * (e + a)) * (1.0 / 1920.0);
    c1 = (34.0 * (d - b) - 5.0 * (e - a)) * (1.0 / 48.0);
    c2 = ((12.0 * (d + b) - 22.0 * c) - (e + a)) * (1.0 / 16.0);
    c3 = ((e - a) - 2.0 * (d - b)) * (1.0 / 12.0);
    c4 = ((((a - 4.0 * b) + 6.0 * c) - 4.0 * d) + e) * (1.0 / 24.0);
  } else {
    const bool k0 = flag & 2u, k1 = flag & 4u, k2 = flag & 8u;
    const int cnt = (int)k0 + (int)k1 + (int)k2;
    const double inv = cnt == 1 ? 1.0 : (cnt == 2 ? 0.5 : 1.0 / 3.0);
    R s0 = R(0.0), s1 = R(0.0), s2 = R(0.0);
    if (k0) {
      s0 = s0 + ((23.0 * c + 2.0 * b) - a) * (1.0 / 24.0);
      s1 = s1 + ((3.0 * c - 4.0 * b) + a) * 0.5;
      s2 = s2 + ((c - 2.0 * b) + a) * 0.5;
    }
    if (k1) {
      s0 = s0 + ((26.0 * c - d) - b) * (1.0 / 24.0);
      s1 = s1 + (d - b) * 0.5;
      s2 = s2 + ((d + b) - 2.0 * c) * 0.5;
    }
    if (k2) {
      s0 = s0 + ((23.0 * c + 2.0 * d) - e) * (1.0 / 24.0);
      s1 = s1 + ((4.0 * d - 3.0 * c) - e) * 0.5;
      s2 = s2 + ((c - 2.0 * d) + e) * 0.5;
    }
    c0 = s0 * inv;
    c1 = s1 * inv;
    c2 = s2 * inv;
  }
  const double ss = s * s;
  const R even = c0 + ss * (c2 + ss * c4);
  const R odd = s * (c1 + ss * c3);
  val[0] = even - odd;
  val[1] = even + odd;
  const R deven = c1 + (3.0 * ss) * c3;
  const R dodd = s * (2.0 * c2 + (4.0 * ss) * c4);
  der[0] = deven - dodd;
  der[1] = deven + dodd;
}

// ---------------------------------------------------------------------------
// The paper's comparison schemes on the same five values and candidate
// polynomials: WENO-AO (Sec. 3.2), TENO5 (Sec. 4.1) and WENO-Z (Sec. 3.1).
//   * WENO-AO: linear weights d3 = d_Hi, d0 = d2 = (1 - d_Hi)(1 - d_Lo)/2,
//     d1 = (1 - d_Hi) d_Lo; omega_k = d_k (1 + (tau / (beta_k + eps))^2)
//     with tau the mean of |beta3 - beta_k| (the ratio squared, as Table 2
//     requires), normalised over k = 0..3; the polynomial
//     w3 (p3/d3 - sum d_k/d3 p_k) + sum w_k p_k gives values and slopes
//     wherever they are needed (interfaces, Gauss points).
//   * WENO-Z / TENO5: small stencils only, omega_k = d_k (1 + tau /
//     (beta_k + eps)) (WENO-Z) or d_k delta_k with delta_k = 0 where
//     (1 + tau / (beta_k + eps))^q < C_T sum (TENO5), tau = |beta0 - beta2|,
//     d_k the linear weights of the evaluation point (0.1, 0.6, 0.3 at
//     x_{i+1/2}, mirrored at x_{i-1/2}, (7/36 -+ sqrt 3/1080, 11/18, ...) at
//     the Gauss points).  Interface slopes from the quadratic with the cell
//     average and the two interface values (Eq. 3.11); along a face the
//     same quadratic's derivative at the Gauss point.
// The TENO5 cut-offs and the WENO-Z / TENO5 interface values follow one
// fixed evaluation order without contraction (the interface values are the
// inputs of the tangential selections, whose flags must be a deterministic
// function of the data).
// ---------------------------------------------------------------------------
constexpr int SCHEME_TENO_D = 0, SCHEME_WENO_AO = 1, SCHEME_TENO5 = 2, SCHEME_WENO_Z = 3;

struct SchemeCfg {
  double ct, eps;      // TENO5 cut-off C_T and epsilon
  int q;               // TENO5 power
  double d[3];         // WENO-AO linear weights of p0 (and p2), p1 and p3
  double r[3];         // their ratios to that of p3; of p3: 1 / d3
  double eps_w;        // WENO-AO / WENO-Z epsilon
};

inline SchemeCfg scheme_cfg(double ct, double eps, int q, double dh, double dl, double eps_w) {
  const double d0 = (1.0 - dh) * (1.0 - dl) / 2.0, d1 = (1.0 - dh) * dl;
  return SchemeCfg{ct, eps, q, {d0, d1, dh}, {d0 / dh, d1 / dh, 1.0 / dh}, eps_w};
}

// Jiang-Shu indicators of p0..p2 and Balsara's form for p3 (the same
// arithmetic as teno_flag's)
template <class R>
TGKS_HD void indicators(const R* Q, R* beta) {
#pragma clang fp contract(off)
  const R a = Q[0], b = Q[1], cc = Q[2], d = Q[3], e = Q[4];
  const double k13 = 13.0 / 12.0;
  R t1, t2;
  t1 = (a - 2.0 * b) + cc;
  t2 = (a - 4.0 * b) + 3.0 * cc;
  beta[0] = k13 * (t1 * t1) + 0.25 * (t2 * t2);
  t1 = (b - 2.0 * cc) + d;
  t2 = b - d;
  beta[1] = k13 * (t1 * t1) + 0.25 * (t2 * t2);
  t1 = (cc - 2.0 * d) + e;
  t2 = (3.0 * cc - 4.0 * d) + e;
  beta[2] = k13 * (t1 * t1) + 0.25 * (t2 * t2);
  const R P1 = (82.0 * (d - b) - 11.0 * (e - a)) * (1.0 / 120.0);
  const R P2 = ((((40.0 * b - 3.0 * a) - 74.0 * cc) + 40.0 * d) - 3.0 * e) * (1.0 / 56.0);
  const R P3 = ((e - a) - 2.0 * (d - b)) * (1.0 / 12.0);
  const R P4 = ((((a - 4.0 * b) + 6.0 * cc) - 4.0 * d) + e) * (1.0 / 24.0);
  const R s1 = P1 + P3 * (1.0 / 10.0);
  const R s2 = P2 + (123.0 / 455.0) * P4;
  beta[3] = (((s1 * s1) + (13.0 / 3.0) * (s2 * s2)) + (781.0 / 20.0) * (P3 * P3)) +
            (1421461.0 / 2275.0) * (P4 * P4);
}

// the same of p0..p2 alone, from the shared differences
template <class R>
TGKS_HD void small_indicators(const TenoParts<R>& p, R* beta) {
#pragma clang fp contract(off)
  const double k13 = 13.0 / 12.0;
  const R l[3] = {p.l0, p.x, p.l2};
#pragma unroll
  for (int k = 0; k < 3; ++k) beta[k] = fma_(R(0.25), l[k] * l[k], k13 * (p.t[k] * p.t[k]));
}

// TENO5 cut-offs: bit k = delta_k (Eqs. 4.1-4.3)
template <class R>
TGKS_HD unsigned teno5_flags(const R* beta, const SchemeCfg& c) {
#pragma clang fp contract(off)
  const R tau = fabs(beta[0] - beta[2]);
  R g[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const R t = 1.0 + tau / (beta[k] + c.eps);
    R pw;
    if (c.q == 6) {
      const R t2 = t * t;
      const R t4 = t2 * t2;
      pw = t4 * t2;
    } else {
      pw = R(1.0);
      for (int r = 0; r < c.q; ++r) pw = pw * t;
    }
    g[k] = pw;
  }
  const R sg = (g[0] + g[1]) + g[2];
  unsigned f = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (!(g[k] < c.ct * sg)) f |= 1u << k;
  return f;
}

// ... as a function of its own, the rare path of teno5_select
__host__ __device__ __attribute__((noinline)) inline unsigned teno5_flags_cold(double b0, double b1, double b2,
                                                                               double ct, double eps, int q) {
  const double beta[3] = {b0, b1, b2};
  SchemeCfg c{};
  c.ct = ct;
  c.eps = eps;
  c.q = q;
  return teno5_flags(beta, c);
}

// The cut-offs by estimated reciprocals: each ratio is right to 2^-45, its
// q-th power (q <= 1024) to 2^-34, so a power outside the cut-off by 2^-30 on
// either side is decided; what is not (also where a power overflows, an
// indicator is huge or anything is NaN) takes the exact quotients.  Three
// estimates for three divisions: half of the selection's operations.
template <class R>
TGKS_HD unsigned teno5_select(const R* beta, const SchemeCfg& c) {
  if constexpr (std::is_same_v<R, double>) {
#pragma clang fp contract(off)
    const double tau = fabs(beta[0] - beta[2]);
    double g[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double x = beta[k] + c.eps;
      double r = rcp_approx(x);
      r = fma(r, fma(-x, r, 1.0), r);
      g[k] = fma(tau, r, 1.0);
    }
    if (c.q == 6) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double t2 = g[k] * g[k];
        g[k] = t2 * t2 * t2;
      }
    } else {
      const double t[3] = {g[0], g[1], g[2]};
      g[0] = g[1] = g[2] = 1.0;
      for (int r = 0; r < c.q; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) g[k] *= t[k];
    }
    const double sg = (g[0] + g[1]) + g[2], cut = c.ct * sg;
    const double up = cut * (1.0 + 0x1p-30), dn = cut * (1.0 - 0x1p-30);
    bool sure = (sg < 1e300) & ((beta[0] + beta[1]) + beta[2] < 1e300) & (c.q <= 1024);
    unsigned f = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const bool keep = g[k] > up;
      sure &= keep | (g[k] < dn);
      f |= keep ? 1u << k : 0u;
    }
    if (!sure) f = teno5_flags_cold(beta[0], beta[1], beta[2], c.ct, c.eps, c.q);
    return f;
  } else {
    return teno5_flags(beta, c);
  }
}

// linear weights of p0..p2 at x_{i-1/2} (where 0), x_{i+1/2} (1), the Gauss
// points -1/(2 sqrt 3) (2) and +1/(2 sqrt 3) (3)
constexpr double LIN_GW = 1.7320508075688772 / 1080.0;
constexpr double LIN_W[4][3] = {{0.3, 0.6, 0.1},
                                {0.1, 0.6, 0.3},
                                {7.0 / 36.0 + LIN_GW, 11.0 / 18.0, 7.0 / 36.0 - LIN_GW},
                                {7.0 / 36.0 - LIN_GW, 11.0 / 18.0, 7.0 / 36.0 + LIN_GW}};

// TENO5's normalised weights d_k delta_k / sum d_k delta_k of each flag at the
// four points: divided by the compiler, which rounds as the division of the
// definition does
struct Teno5Weights {
  double w[8][4][3];
};
constexpr Teno5Weights teno5_weights() {
  Teno5Weights t{};
  for (int f = 1; f < 8; ++f)
    for (int x = 0; x < 4; ++x) {
      double S = 0.0;
      for (int k = 0; k < 3; ++k) S = S + ((f >> k) & 1 ? LIN_W[x][k] : 0.0);
      for (int k = 0; k < 3; ++k) t.w[f][x][k] = (f >> k) & 1 ? LIN_W[x][k] / S : 0.0;
    }
  return t;
}
constexpr Teno5Weights TENO5_W = teno5_weights();

// tau / (beta + eps) of the WENO weights, without a division; indicators
// below 1e-300 (eps_w > 0 is smaller still) belong to differences below 1e-150,
// whose weighting no longer shows in a value.  The reciprocal and its product
// are each rounded: L1 errors of a step against the oracle, smooth, rough and
// jump data in 1-D and 2-D, 0.995 to 1.002 times those with divisions (WENO-Z
// and WENO-AO).
template <class R>
TGKS_HD R weno_ratio(R tau, R x) {
  return tau / x;
}
TGKS_HD double weno_ratio(double tau, double x) { return tau * recip(fmax(x, 1e-300)); }

// WENO-AO coefficients of p0..p2 (w[0..2]) and p3 (w[3])
template <class R>
TGKS_HD void ao_coeffs(const R* beta, const SchemeCfg& c, R* w) {
  const R tau = ((fabs(beta[3] - beta[0]) + fabs(beta[3] - beta[1])) + fabs(beta[3] - beta[2])) * (1.0 / 3.0);
  const double d[4] = {c.d[0], c.d[1], c.d[0], c.d[2]};
  R om[4], S = R(0.0);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const R r = weno_ratio(tau, beta[k] + c.eps_w);
    om[k] = d[k] * (1.0 + r * r);
    S = S + om[k];
  }
  const R iS = recip(S);
  const R o3 = om[3] * iS;
  w[3] = o3 * c.r[2];
  w[0] = om[0] * iS - o3 * c.r[0];
  w[1] = om[1] * iS - o3 * c.r[1];
  w[2] = om[2] * iS - o3 * c.r[0];
}

// interface values of p0..p2 at x_{i-1/2} (vm) and x_{i+1/2} (vp)
template <class R>
TGKS_HD void small_face(const R* Q, R* vm, R* vp) {
#pragma clang fp contract(off)
  const R a = Q[0], b = Q[1], c = Q[2], d = Q[3], e = Q[4];
  vp[0] = ((2.0 * a - 7.0 * b) + 11.0 * c) * (1.0 / 6.0);
  vp[1] = ((5.0 * c - b) + 2.0 * d) * (1.0 / 6.0);
  vp[2] = ((2.0 * c + 5.0 * d) - e) * (1.0 / 6.0);
  vm[0] = ((5.0 * b - a) + 2.0 * c) * (1.0 / 6.0);
  vm[1] = ((2.0 * b + 5.0 * c) - d) * (1.0 / 6.0);
  vm[2] = ((11.0 * c - 7.0 * d) + 2.0 * e) * (1.0 / 6.0);
}

// the WENO-Z ratios u_k = 1 + tau / (beta_k + eps) of p0..p2, and the
// normalised weights d_k u_k / sum d_k u_k at point `where`
template <class R>
TGKS_HD void wenoz_ratios(const R* beta, const SchemeCfg& c, R* u) {
  const R tau = fabs(beta[0] - beta[2]);
#pragma unroll
  for (int k = 0; k < 3; ++k) u[k] = 1.0 + weno_ratio(tau, beta[k] + c.eps_w);
}
template <class R>
TGKS_HD void wenoz_weights(const R* u, int where, R* w) {
#pragma unroll
  for (int k = 0; k < 3; ++k) w[k] = LIN_W[where][k] * u[k];
  const R iS = recip((w[0] + w[1]) + w[2]);
#pragma unroll
  for (int k = 0; k < 3; ++k) w[k] = w[k] * iS;
}

// interface values of the weighted small stencils, in one fixed order
template <class R, class W>
TGKS_HD void small_blend(const R* vm, const R* vp, const W* wm, const W* wp, R& vm_o, R& vp_o) {
#pragma clang fp contract(off)
  vm_o = (wm[0] * vm[0] + wm[1] * vm[1]) + wm[2] * vm[2];
  vp_o = (wp[0] * vp[0] + wp[1] * vp[1]) + wp[2] * vp[2];
}

// Normal reconstruction: out = {v(-1/2), s(-1/2), v(+1/2), s(+1/2)} (cell
// units); returns the flags (TENO5) or 0.  TENO5: wavefronts all of whose
// lanes keep every stencil, the smooth ones, take the linear weights as
// constants, the others load their flag's row of the table.  With a division
// per weight and per indicator, 410 in a 2-D face's code, the divisions bound
// the kernel: 500 x 310 cells, one stage's faces, 160 us; now 77.
template <int SCHEME, class R>
TGKS_HD unsigned scheme_face(const R* Q, const SchemeCfg& c, R* out) {
#pragma clang fp contract(off)
  if (SCHEME == SCHEME_WENO_AO) {
    R beta[4], w[4];
    indicators(Q, beta);
    ao_coeffs(beta, c, w);
    const R a = Q[0], b = Q[1], cc = Q[2], d = Q[3], e = Q[4];
    R vm[3], vp[3];
    small_face(Q, vm, vp);
    const R Lp = ((((2.0 * a - 13.0 * b) + 47.0 * cc) + 27.0 * d) - 3.0 * e) * (1.0 / 60.0);
    const R Lps = (((b - 15.0 * cc) + 15.0 * d) - e) * (1.0 / 12.0);
    const R Lm = ((((27.0 * b - 3.0 * a) + 47.0 * cc) - 13.0 * d) + 2.0 * e) * (1.0 / 60.0);
    const R Lms = (((a - 15.0 * b) + 15.0 * cc) - d) * (1.0 / 12.0);
    const R dp0 = (a - 3.0 * b) + 2.0 * cc, dp12 = d - cc;
    const R dm01 = cc - b, dm2 = (3.0 * d - 2.0 * cc) - e;
    out[0] = ((w[3] * Lm + w[0] * vm[0]) + w[1] * vm[1]) + w[2] * vm[2];
    out[1] = ((w[3] * Lms + w[0] * dm01) + w[1] * dm01) + w[2] * dm2;
    out[2] = ((w[3] * Lp + w[0] * vp[0]) + w[1] * vp[1]) + w[2] * vp[2];
    out[3] = ((w[3] * Lps + w[0] * dp0) + w[1] * dp12) + w[2] * dp12;
    return 0u;
  }
  TenoParts<R> p;
  R beta[3], vms[3], vps[3], vm, vp;
  teno_parts(Q, p);
  small_indicators(p, beta);
  small_face(Q, vms, vps);
  unsigned f = 0;
  if (SCHEME == SCHEME_TENO5) {
    f = teno5_select(beta, c);
    if (all_lanes(f == 7u))
      small_blend(vms, vps, TENO5_W.w[7][0], TENO5_W.w[7][1], vm, vp);
    else
      small_blend(vms, vps, TENO5_W.w[f][0], TENO5_W.w[f][1], vm, vp);
  } else {
    R u[3], wm[3], wp[3];
    wenoz_ratios(beta, c, u);
    wenoz_weights(u, 0, wm);
    wenoz_weights(u, 1, wp);
    small_blend(vms, vps, wm, wp, vm, vp);
  }
  out[0] = vm;
  out[1] = -2.0 * ((2.0 * vm + vp) - 3.0 * Q[2]);
  out[2] = vp;
  out[3] = 2.0 * ((vm + 2.0 * vp) - 3.0 * Q[2]);
  return f;
}

// monomial coefficients (x in [-1/2, 1/2]) of the large-stencil quartic (L)
// and the three quadratics (S[k][0..2])
template <class R>
TGKS_HD void cand_coeffs(const R* Q, R* L, R (*S)[3]) {
  const R a = Q[0], b = Q[1], c = Q[2], d = Q[3], e = Q[4];
  L[0] = ((2134.0 * c - 116.0 * (d + b)) + 9.0 * (e + a)) * (1.0 / 1920.0);
  L[1] = (34.0 * (d - b) - 5.0 * (e - a)) * (1.0 / 48.0);
  L[2] = ((12.0 * (d + b) - 22.0 * c) - (e + a)) * (1.0 / 16.0);
  L[3] = ((e - a) - 2.0 * (d - b)) * (1.0 / 12.0);
  L[4] = ((((a - 4.0 * b) + 6.0 * c) - 4.0 * d) + e) * (1.0 / 24.0);
  S[0][0] = (23.0 * c + 2.0 * b - a) * (1.0 / 24.0);
  S[0][1] = (3.0 * c - 4.0 * b + a) * 0.5;
  S[0][2] = (c - 2.0 * b + a) * 0.5;
  S[1][0] = (26.0 * c - d - b) * (1.0 / 24.0);
  S[1][1] = (d - b) * 0.5;
  S[1][2] = (d + b - 2.0 * c) * 0.5;
  S[2][0] = (23.0 * c + 2.0 * d - e) * (1.0 / 24.0);
  S[2][1] = (4.0 * d - 3.0 * c - e) * 0.5;
  S[2][2] = (c - 2.0 * d + e) * 0.5;
}

// Tangential reconstruction at the Gauss points s = -+1/(2 sqrt 3): val[m],
// der[m] (cell units); returns the flags (TENO5) or 0
template <int SCHEME, class R>
TGKS_HD unsigned scheme_gauss(const R* Q, const SchemeCfg& c, R* val, R* der) {
  const double s = 0.28867513459481288225;  // 1/(2 sqrt 3)
  const double ss = s * s;
  if (SCHEME == SCHEME_WENO_AO) {
    R beta[4], L[5], S[3][3], w[4];
    indicators(Q, beta);
    cand_coeffs(Q, L, S);
    ao_coeffs(beta, c, w);
    const R c0 = w[3] * L[0] + ((w[0] * S[0][0] + w[1] * S[1][0]) + w[2] * S[2][0]);
    const R c1 = w[3] * L[1] + ((w[0] * S[0][1] + w[1] * S[1][1]) + w[2] * S[2][1]);
    const R c2 = w[3] * L[2] + ((w[0] * S[0][2] + w[1] * S[1][2]) + w[2] * S[2][2]);
    const R c3 = w[3] * L[3], c4 = w[3] * L[4];
    const R even = c0 + ss * (c2 + ss * c4), odd = s * (c1 + ss * c3);
    val[0] = even - odd;
    val[1] = even + odd;
    const R deven = c1 + (3.0 * ss) * c3, dodd = s * (2.0 * c2 + (4.0 * ss) * c4);
    der[0] = deven - dodd;
    der[1] = deven + dodd;
    return 0u;
  }
  // Quadratic k has the value Q_0 +- l_k / 4 + t_k / 12 at the faces and,
  // s^2 being 1/12, Q_0 +- (s / 2) l_k at the Gauss points; the slopes are
  // those of the quadratic with the average Q_0 and the end values
  // Q_0 + vm, Q_0 + vp
  TenoParts<R> p;
  R beta[3];
  teno_parts(Q, p);
  small_indicators(p, beta);
  const R l[3] = {p.l0, p.x, -p.l2};
  auto blend = [&](const auto* wm, const auto* wp, const auto* w0, const auto* w1) {
    R am[3], ap[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const R t = p.t[k] * (1.0 / 12.0);
      am[k] = t - 0.25 * l[k];
      ap[k] = t + 0.25 * l[k];
    }
    const R vm = (wm[0] * am[0] + wm[1] * am[1]) + wm[2] * am[2];
    const R vp = (wp[0] * ap[0] + wp[1] * ap[1]) + wp[2] * ap[2];
    const R q1 = vp - vm, q2 = 3.0 * (vm + vp);
    val[0] = Q[2] - (0.5 * s) * ((w0[0] * l[0] + w0[1] * l[1]) + w0[2] * l[2]);
    val[1] = Q[2] + (0.5 * s) * ((w1[0] * l[0] + w1[1] * l[1]) + w1[2] * l[2]);
    der[0] = q1 - (2.0 * s) * q2;
    der[1] = q1 + (2.0 * s) * q2;
  };
  unsigned f = 0;
  if (SCHEME == SCHEME_TENO5) {
    f = teno5_select(beta, c);
    if (all_lanes(f == 7u)) {
      blend(TENO5_W.w[7][0], TENO5_W.w[7][1], TENO5_W.w[7][2], TENO5_W.w[7][3]);
    } else {
      blend(TENO5_W.w[f][0], TENO5_W.w[f][1], TENO5_W.w[f][2], TENO5_W.w[f][3]);
      if (f == 0u) {  // no stencil kept (a cut-off above 1/3): weights of zero
        val[0] = val[1] = R(0.0);
        der[0] = (12.0 * s) * Q[2];
        der[1] = -(12.0 * s) * Q[2];
      }
    }
  } else {
    R u[3], wm[3], wp[3], w0[3], w1[3];
    wenoz_ratios(beta, c, u);
    wenoz_weights(u, 0, wm);
    wenoz_weights(u, 1, wp);
    wenoz_weights(u, 2, w0);
    wenoz_weights(u, 3, w1);
    blend(wm, wp, w0, w1);
  }
  return f;
}

// Eq. 3.12: the equilibrium slope at x_{i+1/2} from the cells i-1 .. i+2
// (cell units)
template <class R>
TGKS_HD R eq_slope(R wm1, R w0, R w1, R w2) {
  return (-1.0 / 12.0) * (w2 - wm1) + 1.25 * (w1 - w0);
}

// ---------------------------------------------------------------------------
// Characteristic variables: an optional choice of reconstruction variables
// (the paper reconstructs the conservative ones).  At a face the reference
// state Wb is the mean of the conservative states of the two adjacent cells
// (frame order: rho, m_0..m_{D-1}, E); the fields are the eigenvectors of the
// Euler flux Jacobian along frame axis A at Wb (A = 0 normal, A = 1 along
// the face), ordered u_A - c, entropy, shear waves of the other axes in
// increasing order, u_A + c.  L holds the left eigenvectors as rows, Rm the
// right ones as columns (Rm L = I).  Entries, projections and
// back-projections follow one fixed operation order without contraction
// (dense left-to-right sums over all components), so that the projected
// values, and the stencil selections made on them, are a deterministic
// function of the input bits.  A non-physical Wb gives the identity.
// ---------------------------------------------------------------------------
template <int D, int A, class R>
TGKS_HD bool char_basis(double gamma, const R* Wb, R (*L)[D + 2], R (*Rm)[D + 2]) {
#pragma clang fp contract(off)
  constexpr int NC = D + 2, KP = D + 1;
  const R rho = Wb[0];
  const R irho = R(1.0) / rho;
  R u[D];
#pragma unroll
  for (int e = 0; e < D; ++e) u[e] = Wb[1 + e] * irho;
  R q2 = u[0] * u[0];
#pragma unroll
  for (int e = 1; e < D; ++e) q2 = q2 + u[e] * u[e];
  const R E = Wb[D + 1];
  const R p = (gamma - 1.0) * (E - 0.5 * (rho * q2));
  const R c2 = (gamma * p) * irho;
  const bool ok = (rho > 0.0) && (p > 0.0) && (c2 < INFINITY) && (E < INFINITY) && (E > -INFINITY);
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j) L[i][j] = Rm[i][j] = R(0.0);
  if (!ok) {
#pragma unroll
    for (int i = 0; i < NC; ++i) L[i][i] = Rm[i][i] = R(1.0);
    return false;
  }
  const R c = sqrt(c2);
  const R ic = R(1.0) / c;
  const R H = (E + p) * irho;
  const R b1 = (gamma - 1.0) / c2;
  const R b2 = 0.5 * (b1 * q2);
  const R un = u[A];
  const R uc = un * c;
  L[0][0] = 0.5 * (b2 + un * ic);
  L[KP][0] = 0.5 * (b2 - un * ic);
  L[1][0] = 1.0 - b2;
#pragma unroll
  for (int e = 0; e < D; ++e) {
    if (e == A) {
      L[0][1 + e] = 0.5 * (-(b1 * un) - ic);
      L[KP][1 + e] = 0.5 * (ic - b1 * un);
    } else {
      L[0][1 + e] = 0.5 * (-(b1 * u[e]));
      L[KP][1 + e] = 0.5 * (-(b1 * u[e]));
    }
    L[1][1 + e] = b1 * u[e];
  }
  L[0][D + 1] = 0.5 * b1;
  L[KP][D + 1] = 0.5 * b1;
  L[1][D + 1] = -b1;
  int k = 2;
#pragma unroll
  for (int s = 0; s < D; ++s) {
    if (s == A) continue;
    L[k][0] = -u[s];
    L[k][1 + s] = R(1.0);
    Rm[1 + s][k] = R(1.0);
    Rm[D + 1][k] = u[s];
    ++k;
  }
  Rm[0][0] = R(1.0);
  Rm[0][1] = R(1.0);
  Rm[0][KP] = R(1.0);
#pragma unroll
  for (int e = 0; e < D; ++e) {
    Rm[1 + e][0] = e == A ? un - c : u[e];
    Rm[1 + e][1] = u[e];
    Rm[1 + e][KP] = e == A ? un + c : u[e];
  }
  Rm[D + 1][0] = H - uc;
  Rm[D + 1][1] = 0.5 * q2;
  Rm[D + 1][KP] = H + uc;
  return true;
}

// y = M x with dense left-to-right sums, no contraction
template <int NC, class R>
TGKS_HD void char_mv(const R (*M)[NC], const R* x, R* y) {
#pragma clang fp contract(off)
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    R v = M[i][0] * x[0];
#pragma unroll
    for (int j = 1; j < NC; ++j) v = v + M[i][j] * x[j];
    y[i] = v;
  }
}

// one row: l . x
template <int NC, class R>
TGKS_HD R char_dot(const R* l, const R* x) {
#pragma clang fp contract(off)
  R v = l[0] * x[0];
#pragma unroll
  for (int j = 1; j < NC; ++j) v = v + l[j] * x[j];
  return v;
}

// Normal reconstruction of both sides of one face in characteristic
// variables, from the six frame-ordered cells C[0..5] = f-3 .. f+2 along the
// normal: values and slopes (slopes per unit length, idn = 1/dx) in frame
// order; fr = selection flags of the right side (cell f at its low face).
template <int D, class R>
TGKS_HD void char_recon_face(double gamma, const R (*C)[D + 2], const TenoCfg& tn, double idn, R* vl, R* sl,
                             R* vr, R* sr, unsigned* fr) {
  constexpr int NC = D + 2;
  R Wb[NC], L[NC][NC], Rm[NC][NC];
  {
#pragma clang fp contract(off)
#pragma unroll
    for (int q = 0; q < NC; ++q) Wb[q] = 0.5 * (C[2][q] + C[3][q]);
  }
  char_basis<D, 0>(gamma, Wb, L, Rm);
  R ol[NC][4], orr[NC][4];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    R V[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) V[r] = char_dot<NC>(L[k], C[r]);
    const unsigned f0 = teno_flag<SEL_FILTER, true>(V, tn);
    const unsigned f1 = teno_flag<SEL_FILTER, true>(V + 1, tn);
    teno_face(V, f0, ol[k]);
    teno_face(V + 1, f1, orr[k]);
    fr[k] = f1;
  }
  R a[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) a[k] = ol[k][2];
  char_mv<NC>(Rm, a, vl);
#pragma unroll
  for (int k = 0; k < NC; ++k) a[k] = ol[k][3];
  char_mv<NC>(Rm, a, sl);
#pragma unroll
  for (int k = 0; k < NC; ++k) a[k] = orr[k][0];
  char_mv<NC>(Rm, a, vr);
#pragma unroll
  for (int k = 0; k < NC; ++k) a[k] = orr[k][1];
  char_mv<NC>(Rm, a, sr);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    sl[q] = sl[q] * idn;
    sr[q] = sr[q] * idn;
  }
}

// ---------------------------------------------------------------------------
// Gas-kinetic flux at one Gauss point (Sec. 2.1), face frame: u1 is normal.
// ---------------------------------------------------------------------------
struct FluxCfg {
  double N;          // K + D = 2/(gamma - 1)
  double K;          // internal degrees of freedom
  double mu, pr_fix; // viscosity; (1/Pr - 1) for the energy flux, 0 if Euler
  double c1, c2;
  int tau_mode;      // 0 inviscid, 1 viscous, 2 zero
};

constexpr int NM1 = 7;  // normal moment table <u1^n>, n = 0..6

template <int D, class R>
struct Gas {
  R rho, irho, U[D], lam, h;  // h = 1/(2 lambda) = p / rho
  bool ok;
};

// 1/sqrt(x): the device's reciprocal square root in the kernels
template <class R>
TGKS_HD R rsqrt_(R x) {
  return rsqrt(x);
}
TGKS_HD double rsqrt_(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return rsqrt(x);
#else
  return 1.0 / sqrt(x);
#endif
}

// The instruction scheduler moves nothing across this point.
template <class R>
TGKS_HD void phase_end() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// An opaque copy: the compiler cannot see that the result equals the input,
// so a recomputation from it is not merged with an earlier identical one
// (whose results would otherwise stay live in registers until the later
// use).  The value is unchanged.
template <class R>
TGKS_HD R opaque(R x) {
  return x;
}
TGKS_HD double opaque(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
  return x;
}

// ... which may be moved or dropped like any other value: code after it is
// compiled from the value alone, not from how it was made
TGKS_HD double sealed(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(x));
#endif
  return x;
}

// (rho, 1/rho, U, lambda, h) of W with one reciprocal:
// re = rho (rho E) - |rho U|^2 / 2 = rho^2 e_int, inv = 1 / (rho re)
template <int D, class R>
TGKS_HD void make_gas(const R* W, double N, Gas<D, R>& g) {
  g.rho = W[0];
  R m2 = R(0.0);
#pragma unroll
  for (int d = 0; d < D; ++d) m2 += W[d + 1] * W[d + 1];
  const R re = g.rho * W[D + 1] - 0.5 * m2;
  const R inv = recip(g.rho * re);
  g.irho = re * inv;
#pragma unroll
  for (int d = 0; d < D; ++d) g.U[d] = W[d + 1] * g.irho;
  const R ir2 = g.irho * g.irho;
  g.h = ((2.0 / N) * re) * ir2;                      // p / rho = 1/(2 lambda)
  g.lam = (0.25 * N) * ((g.rho * g.rho) * (g.rho * inv));
  g.ok = (g.rho > 0.0) && (re > 0.0) && (g.rho < INFINITY) && (re < INFINITY);
}

// erfc(x) given ex2 = exp(-x^2), which the half-space moments need anyway.
// With t = |x|: erfc(t) = ex2 f(y) / (1 + 2t), where f(y) = (1 + 2t)
// exp(t^2) erfc(t) is a smooth function of y = (t - K) / (t + K) on
// [-1, 1] (K = 3.75; the form of Shepherd and Laframboise, Math. Comp. 36,
// 1981): its Chebyshev series cut after 23 terms, in powers of y, summed by
// Horner's rule as even and odd parts in y^2 (two independent chains); the
// power coefficients are small (sum of magnitudes 1.76), so the power form
// is as accurate as the series.  erfc(-t) = 2 - erfc(t).  The
// coefficients are written by paper_2309_10534_amd/erfc_coeffs.py from the
// definition (mpmath, 40 digits); in this arithmetic f / (1 + 2t) is
// within 5.6e-16 of exp(t^2) erfc(t) for t in [0, 27] (beyond, ex2
// underflows).  One reciprocal of (t + K)(1 + 2t) (estimate and two Newton
// steps, about 1 ulp) serves both divisions.  The operation-counting type
// counts one erfc.
constexpr double ERFC_POLY[23] = {
    1.2375126308378275, -0.14024059858554525, 0.0035854154854790257,
    0.08227673848999506, -0.10880393014244462, 0.09230432116428125,
    -0.05869339857664934, 0.028362277372111139, -0.0097465796832652621,
    0.0017556261651970652, 0.00029371437804495801, -0.00029015535246077655,
    5.1646529741774162e-05, 2.2387565714911816e-05, -1.1438048033346894e-05,
    -9.7926257073035231e-07, 1.7419821586224816e-06, -5.0844653786873023e-08,
    -2.4857126248016745e-07, 1.8790823223700481e-08, 3.1979266716668042e-08,
    -1.9551358868985616e-09, -2.6231073471334759e-09,
};

template <class R>
TGKS_HD R erfc_exp(R x, R ex2) {
  return erfc(x);
}
TGKS_HD double erfc_exp(double x, double ex2) {
  const double K = 3.75;
  const double t = fmin(fabs(x), 1e10);  // beyond, ex2 = 0 (x = +-inf: erfc = 0 or 2)
  const double a = t + K, q = fma(2.0, t, 1.0);
  const double d = a * q;
  double r = rcp_approx(d);
  r = fma(r, fma(-d, r, 1.0), r);
  r = fma(r, fma(-d, r, 1.0), r);
  const double y = ((t - K) * q) * r;
  const double w = a * r;  // 1 / (1 + 2t)
  const double z = y * y;
  double ev = ERFC_POLY[22], od = ERFC_POLY[21];
#pragma unroll
  for (int j = 20; j >= 0; j -= 2) ev = fma(ev, z, ERFC_POLY[j]);
#pragma unroll
  for (int j = 19; j >= 1; j -= 2) od = fma(od, z, ERFC_POLY[j]);
  const double e = ex2 * (fma(od, y, ev) * w);
  return x < 0.0 ? 2.0 - e : e;
}

// first two half-space moments: sgn = +1 (u1 > 0) or -1 (u1 < 0)
template <class R>
TGKS_HD void half_seed(R U, R lam, double sgn, R& m0, R& m1) {
  const R isl = rsqrt_(lam);
  const R sl = lam * isl;
  const R ex = exp(-(lam * U) * U);
  m0 = 0.5 * erfc_exp(-sgn * (sl * U), ex);
  m1 = U * m0 + ((sgn * 0.28209479177387814347) * ex) * isl;  // 1/(2 sqrt(pi))
}

// ---------------------------------------------------------------------------
// The Gauss-point flux.  Every moment it needs has the form <u1^j psi>,
// <u1^j psi a> or <u1^j c_t psi a> with a microscopic slope a = the
// logarithmic derivative of a Maxwellian along some direction.  They are
// evaluated in the frame that moves with the state's tangential velocity
// (c_t = u_t - U_t), where the odd moments of c_t vanish: with the derivatives
// (dr = d rho / rho, dU, dh) along the direction, h = p / rho = 1/(2 lambda),
//   a = al + be u1 + sum_t (dU_t / h) c_t + de (u1^2 + sum_t c_t^2 + xi^2),
//   de = dh / (2 h^2), be = dU_1 / h - 2 U_1 de,
// and with M_j = rho <u1^j> (over the half space for a side, the full space
// for the equilibrium) and E_j = rho <u1^j (a, its even part in c, xi)> =
// al' M_j + be M_{j+1} + de M_{j+2}, al' = al + (N-1) h de,
//   rho <u1^j psi' a>     = (E_j, E_{j+1}, dU_t M_j, (E_{j+2} + (N-1) q_j) / 2),
//   rho <u1^j c_t psi' a> = (dU_t M_j, dU_t M_{j+1}, q_j [t], dU_t (M_{j+2} + (N+1) h M_j) / 2),
// q_j = h E_j + dh M_j, psi' the collision invariants of that frame.  The
// convective sums split as u_t a_t = U_t a_t + c_t a_t, and the slope of the
// time derivative as A = B - sum_t U_t a_t, with B from the Euler equations
// of the moving frame in primitive variables; a result goes back to the face
// frame at the end.  Tables of every monomial's moments in the face frame, a
// linear solve per slope and sums of products took 209 more instructions per
// lane of the 2-D face kernel (of 2,500) and 225 registers where this takes
// 145, which is three wavefronts per SIMD instead of two (Euler; with the
// Navier-Stokes terms 165 in stage 1, and 169 in stage 2, one more than three
// wavefronts have): 20 steps of the
// 2-D four-quadrant problem at 1024^2 15.5 ms (18.2 before), 2 steps of the
// 3-D Taylor-Green vortex at 128^3 22.3 ms (24.4).
// ---------------------------------------------------------------------------
template <int D, class R>
struct Slope {
  R r, U[D], h;   // d rho / rho, dU, dh along the direction
  R al, be, de;   // al', be, de above
};

// primitive derivatives of the conservative derivative dW
template <int D, class R>
TGKS_HD void slope_prim(const Gas<D, R>& g, double N, const R* dW, Slope<D, R>& s) {
  s.r = dW[0] * g.irho;
  R e = dW[D + 1] * g.irho, u2 = R(0.0);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const R m = dW[d + 1] * g.irho;
    s.U[d] = m - g.U[d] * s.r;
    e -= g.U[d] * m;
    u2 += g.U[d] * g.U[d];
  }
  s.h = (2.0 / N) * (e + (0.5 * u2) * s.r) - g.h * s.r;
}

// the polynomial's coefficients from the primitive derivatives
template <int D, class R>
TGKS_HD void slope_poly(const Gas<D, R>& g, Slope<D, R>& s) {
  const R l2 = 2.0 * g.lam;
  s.de = s.h * (l2 * g.lam);
  const R b = s.U[0] * l2 - g.U[0] * s.de;
  s.be = b - g.U[0] * s.de;
  s.al = (s.r - g.h * s.de) - g.U[0] * b;
}

// the slope of the time derivative in the moving frame (Euler equations)
// from the slopes along the frame axes
template <int D, class R>
TGKS_HD void slope_time(const Gas<D, R>& g, double N, const Slope<D, R>* a, Slope<D, R>& b) {
  R div = a[0].U[0];
#pragma unroll
  for (int d = 1; d < D; ++d) div += a[d].U[d];
  const R u = g.U[0];
  b.r = -(u * a[0].r + div);
#pragma unroll
  for (int d = 0; d < D; ++d) b.U[d] = -(u * a[0].U[d] + (a[d].h + g.h * a[d].r));
  b.h = -(u * a[0].h + (2.0 / N) * (g.h * div));
  slope_poly<D>(g, b);
}

template <int D, class R>
TGKS_HD R slope_e(const R* M, const Slope<D, R>& s, int j) {
  return s.al * M[j] + (s.be * M[j + 1] + s.de * M[j + 2]);
}

// v = rho <u1^j psi' a>
template <int D, class R>
TGKS_HD void slope_vec(const R* M, const Gas<D, R>& g, double N, const Slope<D, R>& s, int j, R* v) {
  const R e = slope_e<D>(M, s, j);
  v[0] = e;
  v[1] = slope_e<D>(M, s, j + 1);
#pragma unroll
  for (int d = 1; d < D; ++d) v[d + 1] = s.U[d] * M[j];
  v[D + 1] = 0.5 * (slope_e<D>(M, s, j + 2) + (N - 1.0) * (g.h * e + s.h * M[j]));
}

// v += rho <u1^j c_t psi' a>
template <int D, class R>
TGKS_HD void slope_vec_c(const R* M, const Gas<D, R>& g, double N, const Slope<D, R>& s, int t, int j, R* v) {
  v[0] += s.U[t] * M[j];
  v[1] += s.U[t] * M[j + 1];
  v[t + 1] += g.h * slope_e<D>(M, s, j) + s.h * M[j];
  v[D + 1] += (0.5 * s.U[t]) * (M[j + 2] + ((N + 1.0) * g.h) * M[j]);
}

// moments of psi' to moments of psi (the face frame)
template <int D, class R>
TGKS_HD void to_face(const Gas<D, R>& g, R* v) {
#pragma unroll
  for (int t = 1; t < D; ++t) {
    v[D + 1] += g.U[t] * (v[t + 1] + (0.5 * g.U[t]) * v[0]);
    v[t + 1] += g.U[t] * v[0];
  }
}

// heat-flux moment <phi X> from <u1 psi X> (f1) and <psi X> (f0):
// phi = (u1 - c1)(psi_E - c.u + |c|^2/2) about the velocity c
template <int D, class R>
TGKS_HD R heat_combine(const R* f1, const R* f0, const R* c) {
  R c2 = R(0.0), s1 = f1[D + 1], s0 = f0[D + 1];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    c2 += c[d] * c[d];
    s1 -= c[d] * f1[d + 1];
    s0 -= c[d] * f0[d + 1];
  }
  s1 += (0.5 * c2) * f1[0];
  s0 += (0.5 * c2) * f0[0];
  return s1 - c[0] * s0;
}

// moments M[0..6] of one Maxwellian from the first two
template <class R>
TGKS_HD void moment_table(R U, R h, R m0, R m1, R* m) {
  m[0] = m0;
  m[1] = m1;
#pragma unroll
  for (int k = 1; k + 1 < NM1; ++k) m[k + 1] = U * m[k] + ((double)k * h) * m[k - 1];
}

// v2 = rho sum_d <u1 u_d psi a_d>, v3 = rho <u1 psi A>, face frame; HEAT: y2,
// y3 their heat-flux moments about the velocity c (moving frame)
template <int D, bool HEAT, class R>
TGKS_HD void slope_parts(const R* M, const Gas<D, R>& g, double N, const Slope<D, R>* a, const R* c, R* v2, R* v3,
                         R& y2, R& y3) {
  constexpr int NC = D + 2;
  Slope<D, R> b;
  slope_time<D>(g, N, a, b);
  slope_vec<D>(M, g, N, a[0], 2, v2);
  slope_vec<D>(M, g, N, b, 1, v3);
#pragma unroll
  for (int t = 1; t < D; ++t) {
    R z[NC];
    slope_vec<D>(M, g, N, a[t], 1, z);
    slope_vec_c<D>(M, g, N, a[t], t, 1, v2);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      v2[q] += g.U[t] * z[q];
      v3[q] -= g.U[t] * z[q];
    }
  }
  if (HEAT) {
    R w2[NC], w3[NC];
    slope_vec<D>(M, g, N, a[0], 1, w2);
    slope_vec<D>(M, g, N, b, 0, w3);
#pragma unroll
    for (int t = 1; t < D; ++t) {
      R z[NC];
      slope_vec<D>(M, g, N, a[t], 0, z);
      slope_vec_c<D>(M, g, N, a[t], t, 0, w2);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        w2[q] += g.U[t] * z[q];
        w3[q] -= g.U[t] * z[q];
      }
    }
    y2 = heat_combine<D>(v2, w2, c);
    y3 = heat_combine<D>(v3, w3, c);
  }
  to_face<D>(g, v2);
  to_face<D>(g, v3);
}

// ---------------------------------------------------------------------------
// The flux in three pieces, for kernels that give the two sides of a Gauss
// point to two lanes: each lane evaluates its side's share of the equilibrium
// state (side_w0) and, once W0 is known, its side's shares of the slopes of
// W0 and of the non-equilibrium moments (side_part); the two shares are
// summed and flux_combine adds the equilibrium part and the time integration.
// gp_flux below evaluates the same arithmetic in one lane.
// ---------------------------------------------------------------------------
template <int D, class R>
struct SidePart {
  R dW0[D][D + 2];          // rho_s <psi a_d>_s: share of the slopes of W0 (Eq. 2.6)
  R S1[D + 2], S2[D + 2], S3[D + 2];  // rho_s <u1 psi>, sum_d <u1 u_d psi a_d>, <u1 psi A> over the half space
  R H1, H2, H3;             // their heat-flux moments (Navier-Stokes)
};

// gas state, rho-weighted half-space seeds (M_0, M_1) and the side's share
// rho_s <psi>_s of W0; sgn = +1 for the left side (u1 > 0), -1 for the right
template <int D, class R>
TGKS_HD void side_w0(const R* Ws, const FluxCfg& P, double sgn, Gas<D, R>& gs, R& h0, R& h1, R* w0) {
  make_gas<D>(Ws, P.N, gs);
  half_seed(gs.U[0], gs.lam, sgn, h0, h1);
  h0 = gs.rho * h0;
  h1 = gs.rho * h1;
  w0[0] = h0;
  w0[1] = h1;
#pragma unroll
  for (int t = 1; t < D; ++t) w0[t + 1] = R(0.0);
  w0[D + 1] = 0.5 * (gs.U[0] * h1 + (P.N * gs.h) * h0);  // M_2 + (N-1) h M_0, M_2 = U M_1 + h M_0
  to_face<D>(gs, w0);
}

template <int D, bool NS, class R>
TGKS_HD void side_part(const Gas<D, R>& gs, R h0, R h1, const R (*dW)[D + 2], const FluxCfg& P, const Gas<D, R>& g0,
                       SidePart<D, R>& o) {
  const double N = P.N;
  R M[NM1];
  moment_table(gs.U[0], gs.h, h0, h1, M);
  Slope<D, R> a[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    slope_prim<D>(gs, N, dW[d], a[d]);
    slope_poly<D>(gs, a[d]);
    slope_vec<D>(M, gs, N, a[d], 0, o.dW0[d]);
    to_face<D>(gs, o.dW0[d]);
  }
  o.S1[0] = M[1];
  o.S1[1] = M[2];
#pragma unroll
  for (int t = 1; t < D; ++t) o.S1[t + 1] = R(0.0);
  o.S1[D + 1] = 0.5 * (M[3] + ((N - 1.0) * gs.h) * M[1]);
  R c[D];  // velocity of the equilibrium in the side's moving frame
  o.H1 = o.H2 = o.H3 = R(0.0);
  if (NS) {
    c[0] = g0.U[0];
    R f0[D + 2];
    f0[0] = M[0];
    f0[1] = M[1];
#pragma unroll
    for (int t = 1; t < D; ++t) {
      c[t] = g0.U[t] - gs.U[t];
      f0[t + 1] = R(0.0);
    }
    f0[D + 1] = 0.5 * (M[2] + ((N - 1.0) * gs.h) * M[0]);
    o.H1 = heat_combine<D>(o.S1, f0, c);
  }
  slope_parts<D, NS>(M, gs, N, a, c, o.S2, o.S3, o.H2, o.H3);
  to_face<D>(gs, o.S1);
}

// What a kernel takes from a Gauss point, w its weight:
//   FLUX_TIMES:  Fa = F(dt), Fb = F(dt/2) (w unused)
//   FLUX_STAGE1: Fa = w F(dt/2), Fb = w (8/3 F(dt/2) - 1/3 F(dt))
//   FLUX_STAGE2: Fa = w (4/3 F(dt) - 8/3 F(dt/2))
// The combinations are made of the six time coefficients, not of the fluxes.
constexpr int FLUX_TIMES = 0, FLUX_STAGE1 = 1, FLUX_STAGE2 = 2;

// Collision time (Sec. 5 preamble; dt is the full step in both stages) and em
// = expm1(-dt / (2 tau)): e^{-dt/tau} = (1 + em)^2, one exponential serves
// both intervals; -1 for tau = 0.  Evaluated before the sides' moments: its
// branches would otherwise end a basic block between them and their use, and
// the compiler moves all of them past it, where they are live at once.
template <class R>
struct FluxTime {
  R tau, em;
};

template <int D, class R>
TGKS_HD FluxTime<R> flux_time(const Gas<D, R>& g0, R pl, R pr, const FluxCfg& P, R dt) {
  const R S = pl + pr, A = fabs(pl - pr);
  R tau = R(0.0), xh = R(0.0);
  if (P.tau_mode == 1) {
    tau = P.mu * recip(g0.rho * g0.h) + (P.c2 * (A * recip(S))) * dt;
    xh = -(0.5 * dt) * recip(tau);
  } else if (P.tau_mode == 0) {
    // tau = (c1 + c2 A/S) dt = dt T/S with T = c1 S + c2 A; one reciprocal
    const R T = P.c1 * S + P.c2 * A;
    if (T > 0.0) {
      const R inv = recip(S * T);
      tau = dt * ((T * T) * inv);
      xh = -0.5 * ((S * S) * inv);
    }
  }
  R em = R(-1.0);
  if (tau != 0.0) em = expm1(xh);
  return FluxTime<R>{tau, em};
}

// Equilibrium part of Eq. 2.5 and the time integration over dt and dt/2,
// given W0, its gas state g0, the two sides' summed shares (dW0, S1..S3,
// H1..H3) and the collision time.
template <int D, bool NS, int OUT, class R>
TGKS_HD void flux_combine(const R* W0, const Gas<D, R>& g0, const SidePart<D, R>& T, const FluxTime<R>& ft,
                          const FluxCfg& P, R dt, double w, R* Fa, R* Fb) {
  constexpr int NC = D + 2;
  const double N = P.N;
  // equilibrium part of Eq. 2.5: T1 = F_1(W0), T2 = rho0 sum_d <u1 u_d psi
  // abar_d>_0, T3 = rho0 <u1 psi Abar>_0 (Abar by the compatibility
  // condition, Eq. 2.7: the Euler equations)
  R T1[NC], T2[NC], T3[NC];
  R G2 = R(0.0), G3 = R(0.0);  // heat-flux moments of the equilibrium part (the first vanishes)
  {
    const R p0 = g0.rho * g0.h;
    T1[0] = W0[1];
#pragma unroll
    for (int e = 0; e < D; ++e) T1[e + 1] = W0[1] * g0.U[e] + (e == 0 ? p0 : R(0.0));
    T1[D + 1] = g0.U[0] * (W0[D + 1] + p0);
    R M[NM1];
    moment_table(g0.U[0], g0.h, g0.rho, W0[1], M);
    Slope<D, R> a[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      slope_prim<D>(g0, N, T.dW0[d], a[d]);
      slope_poly<D>(g0, a[d]);
    }
    R c[D];
    c[0] = g0.U[0];
#pragma unroll
    for (int t = 1; t < D; ++t) c[t] = R(0.0);
    slope_parts<D, NS>(M, g0, N, a, c, T2, T3, G2, G3);
  }

  R C[2][6];
#pragma unroll
  for (int id = 0; id < 2; ++id) {
    const R dl = id == 0 ? dt : 0.5 * dt;
    const R tau = ft.tau, em = ft.em;
    const R e = id == 1 ? em + 1.0 : (em + 1.0) * (em + 1.0);
    const R ome = id == 1 ? -em : -em * (em + 2.0);
    const R tt = (tau * tau) * ome;
    C[id][0] = dl - tau * ome;
    C[id][1] = 2.0 * tt - (tau * dl) * (1.0 + e);
    C[id][2] = (0.5 * dl) * dl - tau * dl + tt;
    C[id][3] = tau * ome;
    C[id][4] = (tau * dl) * e - 2.0 * tt;
    C[id][5] = -tt;
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const R cd = C[0][k], ch = C[1][k];
    if (OUT == FLUX_STAGE1) {
      C[0][k] = w * ch;
      C[1][k] = (w * (8.0 / 3.0)) * ch - (w * (1.0 / 3.0)) * cd;
    } else if (OUT == FLUX_STAGE2) {
      C[0][k] = (w * (4.0 / 3.0)) * cd - (w * (8.0 / 3.0)) * ch;
    }
  }
#pragma unroll
  for (int id = 0; id < (OUT == FLUX_STAGE2 ? 1 : 2); ++id) {
    R* F = id == 0 ? Fa : Fb;
    const R* Ck = C[id];
#pragma unroll
    for (int q = 0; q < NC; ++q)
      F[q] = ((Ck[0] * T1[q] + Ck[1] * T2[q]) + Ck[2] * T3[q]) +
             ((Ck[3] * T.S1[q] + Ck[4] * T.S2[q]) + Ck[5] * T.S3[q]);
    if (NS) {
      const R q = (Ck[1] * G2 + Ck[2] * G3) + ((Ck[3] * T.H1 + Ck[4] * T.H2) + Ck[5] * T.H3);
      F[NC - 1] += P.pr_fix * q;
    }
  }
}

// sum of the two sides' shares (the same in either order)
template <int D, class R>
TGKS_HD void side_sum(const SidePart<D, R>& l, const SidePart<D, R>& r, SidePart<D, R>& o) {
  constexpr int NC = D + 2;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
#pragma unroll
    for (int d = 0; d < D; ++d) o.dW0[d][q] = l.dW0[d][q] + r.dW0[d][q];
    o.S1[q] = l.S1[q] + r.S1[q];
    o.S2[q] = l.S2[q] + r.S2[q];
    o.S3[q] = l.S3[q] + r.S3[q];
  }
  o.H1 = l.H1 + r.H1;
  o.H2 = l.H2 + r.H2;
  o.H3 = l.H3 + r.H3;
}

// Time-integrated fluxes at one Gauss point (FLUX_TIMES, FLUX_STAGE1, 2).
// Wl, Wr: states; dWl[d], dWr[d]: derivatives along frame axis d; sgn = 1:
// Wl is the left side (u1 > 0), -1: the right one (and Wr the left; the two
// sides' shares are added, so the order does not matter).  EQ: a separately
// reconstructed equilibrium (WENO-Z and TENO5 GKS, Sec. 3.1): the slopes of
// W0 along every frame axis are given (dW0), and so is W0 itself when W0in is
// not null (2-D: the tangential reconstruction of the face segments'
// equilibrium states); otherwise W0 is the kinetic weighting of the two sides
// (Eq. 2.6).  Returns false when a state is non-physical.
template <int D, bool NS, int OUT, bool EQ, class R>
TGKS_HD bool gp_flux_any(const R* Wl, const R* Wr, const R (*dWl)[D + 2], const R (*dWr)[D + 2], const R* W0in,
                         const R (*dW0)[D + 2], const FluxCfg& P, R dt, double w, R* Fa, R* Fb, double sgn) {
  constexpr int NC = D + 2;
  Gas<D, R> gl, gr, g0;
  R hl0, hl1, hr0, hr1, wl[NC], wr[NC], W0[NC];
  // equilibrium state by kinetic weighting (Eq. 2.6): rho_l <psi>_{>0} + rho_r <psi>_{<0}
  side_w0<D>(Wl, P, sgn, gl, hl0, hl1, wl);
  side_w0<D>(Wr, P, -sgn, gr, hr0, hr1, wr);
#pragma unroll
  for (int q = 0; q < NC; ++q) W0[q] = EQ && W0in ? W0in[q] : wl[q] + wr[q];
  make_gas<D>(W0, P.N, g0);
  const FluxTime<R> ft = flux_time<D>(g0, gl.rho * gl.h, gr.rho * gr.h, P, dt);
  // side contributions: dW0 (Eq. 2.6), A^s (Eq. 2.7), and the moments of the
  // non-equilibrium part of Eq. 2.5 over the half space.  One side is
  // finished before the other is begun: interleaved by the scheduler they
  // take more registers than three wavefronts per SIMD have.
  SidePart<D, R> L, Rt, T;
  phase_end<R>();
  side_part<D, NS>(gl, hl0, hl1, dWl, P, g0, L);
  phase_end<R>();
  side_part<D, NS>(gr, hr0, hr1, dWr, P, g0, Rt);
  side_sum<D>(L, Rt, T);
  phase_end<R>();
  if (EQ) {
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int q = 0; q < NC; ++q) T.dW0[d][q] = dW0[d][q];
  }
  flux_combine<D, NS, OUT>(W0, g0, T, ft, P, dt, w, Fa, Fb);
  return gl.ok && gr.ok && g0.ok;
}

template <int D, bool NS, int OUT = FLUX_TIMES, class R>
TGKS_HD bool gp_flux(const R* Wl, const R* Wr, const R (*dWl)[D + 2], const R (*dWr)[D + 2], const FluxCfg& P,
                     R dt, R* Fa, R* Fb, double w = 1.0, double sgn = 1.0) {
  return gp_flux_any<D, NS, OUT, false>(Wl, Wr, dWl, dWr, (const R*)nullptr, (const R(*)[D + 2]) nullptr, P, dt, w,
                                        Fa, Fb, sgn);
}

template <int D, bool NS, int OUT = FLUX_TIMES, class R>
TGKS_HD bool gp_flux_eq(const R* Wl, const R* Wr, const R (*dWl)[D + 2], const R (*dWr)[D + 2], const R* W0in,
                        const R (*dW0)[D + 2], const FluxCfg& P, R dt, R* Fa, R* Fb, double w = 1.0,
                        double sgn = 1.0) {
  return gp_flux_any<D, NS, OUT, true>(Wl, Wr, dWl, dWr, W0in, dW0, P, dt, w, Fa, Fb, sgn);
}

// ---------------------------------------------------------------------------
// Boundary index map (ghost cells): periodic, transmissive (copy of the
// nearest cell), reflective (mirror image; flip = 1: the momentum normal to
// the wall changes sign) or a no-slip adiabatic wall (mirror image; flip =
// 2: every momentum component changes sign).
// ---------------------------------------------------------------------------
constexpr int BC_NOSLIP = 3;  // boundary kind of the no-slip adiabatic wall
constexpr int BC_PRESCRIBED = 4;  // boundary kind of given states (resolved before the map)

// Selects, no division or branch: an index used by a face is at most three
// cells outside (n >= 3), so one wrap serves; what lies farther outside feeds
// no face and is clamped into the domain so that every load stays in bounds.
TGKS_HD int map_index(int i, int n, int bclo, int bchi, int& flip) {
  const bool low = i < 0, out = low || i >= n;
  const int bc = low ? bclo : bchi;
  const int wrap = low ? i + n : i - n, edge = low ? 0 : n - 1, mirror = low ? -1 - i : (n - 1) - (i - n);
  int r = bc == 0 ? wrap : (bc == 1 ? edge : mirror);
  r = out ? r : i;
  flip ^= out && bc >= 2 ? (bc == BC_NOSLIP ? 2 : 1) : 0;
  return r < 0 ? 0 : (r >= n ? n - 1 : r);
}

}  // namespace tgks
