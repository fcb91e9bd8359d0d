// Device arithmetic of the S2O4 DF-hybrid step (Zhang, Ji & Xu, arXiv:2402.10914), hand-expanded
// for gfx950.  Every function works in the local frame of an interface: component 1 is the normal
// momentum, component 2 the tangential one (y-interfaces swap rho*U and rho*V before calling,
// an exact reflection of the paper's rotation by pi/2, Section 2.1).
//
// Functions are __host__ __device__ so that the same arithmetic can be instantiated on the host
// with a counting scalar to obtain exact operation counts.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#define DFW_HD __host__ __device__ __forceinline__

namespace dfw {

// Reciprocal of a positive, finite, normal number (the WENO-Z denominators: products of the
// b_k + eps, at least eps^4, and sums of positive weights).  On the device: the hardware reciprocal
// estimate r refined once, with e = 1 - x r: r + r (e + e^2) in FP64 (cubic, one FMA less than two
// Newton steps and as accurate), r + r e in FP32; within one unit in the last place of 1/x, in 4
// (FP64) or 3 (FP32) instructions instead of the ten-instruction IEEE division sequence, whose
// scaling and fix-up steps only matter for zero, infinite or subnormal operands.
// On the host (operation counts, host-side checks): the plain division.
DFW_HD double rcp_pos(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
#else
  return 1.0 / x;
#endif
}

DFW_HD float rcp_pos(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
#else
  return 1.0f / x;
#endif
}

template <class real>
DFW_HD real rcp_pos(real x) {
  return real(1) / x;
}

// Reciprocal with IEEE results for zero, infinite and NaN operands (densities, pressures and sums of
// them on failing states, where inf and not NaN has to reach the steps that rely on it): the refined
// estimate of rcp_pos, special cases set by the division fix-up instruction; 5 instructions.
DFW_HD double rcp_any(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_div_fixup(rcp_pos(x), x, 1.0);
#else
  return 1.0 / x;
#endif
}

template <class real>
DFW_HD real rcp_any(real x) {
  return real(1) / x;
}

// n / x for a positive finite n, with IEEE results for zero, infinite and NaN x: the refined reciprocal's
// product with n corrected by its residual, so that n / n is 1; 8 instructions.
DFW_HD double quotient_any(double n, double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const double r = rcp_pos(x), q = n * r;
  return __builtin_amdgcn_div_fixup(fma(fma(-q, x, n), r, q), x, n);
#else
  return n / x;
#endif
}

template <class real>
DFW_HD real quotient_any(real n, real x) {
  return n / x;
}

// s = sqrt(x) and is = 1 / s together, with IEEE results at zero, infinity, NaN and negative x: the
// hardware estimate y of 1/sqrt(x) refined by one cubic step (e = 1 - x y^2, y + y e (1/2 + 3/8 e)),
// the root corrected by its residual; 14 instructions instead of about 30 for the library's square
// root and an IEEE division.  Zero and +inf are their own roots; a negative x leaves NaN (the
// division fix-up takes a NaN quotient for an overflow, so it serves the reciprocal only, where the
// NaN is the divisor).
DFW_HD void sqrt_inv(double x, double& s, double& is) {
#if defined(__HIP_DEVICE_COMPILE__)
  double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  y = fma(y * e, fma(e, 0.375, 0.5), y);
  const double r = x * y;
  constexpr int kZeroOrInf = 1 << 5 | 1 << 6 | 1 << 9;  // class bits: -0, +0, +inf
  s = __builtin_amdgcn_class(x, kZeroOrInf) ? x : fma(fma(-r, r, x), 0.5 * y, r);
  is = __builtin_amdgcn_div_fixup(y, s, 1.0);
#else
  s = sqrt(x);
  is = 1.0 / s;
#endif
}

template <class real>
DFW_HD void sqrt_inv(real x, real& s, real& is) {
  s = sqrt(x);
  is = real(1) / s;
}

// a b + c in one rounding (the counting scalar of the flop counts: a multiply and an add).
DFW_HD double fmadd(double a, double b, double c) { return fma(a, b, c); }
DFW_HD float fmadd(float a, float b, float c) { return fmaf(a, b, c); }
template <class real>
DFW_HD real fmadd(real a, real b, real c) {
  return a * b + c;
}

// Scheme constants in the working precision, converted once per kernel from the host values.
template <class real>
struct Coef {
  real gamma, gm1, inv_gm1, alpha_thres, eps, c1, c2, K;
  real d[4];      // WENO-AO linear weights d0..d3 (Section 3.1)
  real dr[3];     // d_k / d_3
  real inv_d3;
  real K2, k4K2;  // K + 2 and 4 / (K + 2)
  int sw_rule;    // hybrid switch: 0 max of the three DF values (eq. (42)), 1 their min, 2 the cell's own
};

// Eq. (42): the DF quadratic replaces WENO-AO for a cell when the largest DF value of the cell and
// its two neighbours along the sweep is below the threshold (strict).  Readings kept as options:
// sw_rule 1 takes the smallest of the three (a discontinuity in any of them), 2 the cell's own value.
// RULE >= 0 fixes the rule at compile time (for kernels at the register limit, where a rule read at
// run time costs spills); RULE < 0 reads k.sw_rule.
template <int RULE = -1, class real>
DFW_HD bool df_switch(real a_lo, real a_c, real a_hi, const Coef<real>& k) {
  const int rule = RULE >= 0 ? RULE : k.sw_rule;
  real mx = a_lo > a_c ? a_lo : a_c;
  mx = mx > a_hi ? mx : a_hi;
  real mn = a_lo < a_c ? a_lo : a_c;
  mn = mn < a_hi ? mn : a_hi;
  const real a = rule == 1 ? mn : (rule == 2 ? a_c : mx);
  return a < k.alpha_thres;
}

// ------------------------------------------------------------------------------------------------
// Characteristic basis (eigenvectors of the normal flux Jacobian at the arithmetic mean of the two
// cells beside the interface).  Right eigenvectors (columns): (1,u-c,v,H-uc), (1,u,v,q2/2),
// (0,0,1,v), (1,u+c,v,H+uc).  The left eigenvectors are applied in a factored closed form: with
// b1 = (gamma-1)/(2 c^2), b2 = b1 q2/2, ic = 1/(2 c) and T = b2 w0 - b1 (u w1 + v w2 - w3),
// s = (u w0 - w1) ic:  Q0 = T + s, Q1 = w0 - 2 T, Q2 = w2 - v w0, Q3 = T - s.
// ------------------------------------------------------------------------------------------------
template <class real>
struct Basis {
  real u, v, c, ic, H, hq2, b1, b2;
};

template <class real>
DFW_HD Basis<real> make_basis(const real* wa, const real* wb, const Coef<real>& k) {
  Basis<real> B;
  const real h = real(0.5);
  real r = h * (wa[0] + wb[0]);
  real m = h * (wa[1] + wb[1]);
  real n = h * (wa[2] + wb[2]);
  real e = h * (wa[3] + wb[3]);
  real ir = rcp_any(r);
  B.u = m * ir;
  B.v = n * ir;
  B.hq2 = h * (B.u * B.u + B.v * B.v);
  real p = k.gm1 * (e - r * B.hq2);
  real ic;
  sqrt_inv(k.gamma * p * ir, B.c, ic);
  B.ic = h * ic;
  B.H = (e + p) * ir;
  B.b1 = k.gm1 * (B.ic * ic);
  B.b2 = B.hq2 * B.b1;
  return B;
}

template <class real>
DFW_HD void project(const Basis<real>& B, const real* w, real* q) {
  real T = B.b2 * w[0] - B.b1 * (B.u * w[1] + B.v * w[2] - w[3]);
  real s = (B.u * w[0] - w[1]) * B.ic;
  q[0] = T + s;
  q[1] = w[0] - real(2) * T;
  q[2] = w[2] - B.v * w[0];
  q[3] = T - s;
}

template <class real>
DFW_HD void unproject(const Basis<real>& B, const real* q, real* w) {
  real w0 = q[0] + q[1] + q[3];
  real dq = q[3] - q[0];
  w[0] = w0;
  w[1] = B.u * w0 + B.c * dq;
  w[2] = B.v * w0 + q[2];
  w[3] = B.H * (q[0] + q[3]) + B.u * B.c * dq + B.hq2 * q[1] + B.v * q[2];
}

// The variables the reconstruction works on: characteristic (CHAR) or, as an ablation of that
// choice, the conservative variables themselves (component-wise reconstruction).
template <bool CHAR, class real>
DFW_HD void to_recon(const Basis<real>& B, const real* w, real* q) {
  if constexpr (CHAR) {
    project(B, w, q);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = w[c];
  }
}

template <bool CHAR, class real>
DFW_HD void from_recon(const Basis<real>& B, const real* q, real* w) {
  if constexpr (CHAR) {
    unproject(B, q, w);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) w[c] = q[c];
  }
}

template <bool CHAR, class real>
DFW_HD Basis<real> recon_basis(const real* wa, const real* wb, const Coef<real>& k) {
  if constexpr (CHAR) {
    return make_basis(wa, wb, k);
  } else {
    return Basis<real>{};
  }
}

// ------------------------------------------------------------------------------------------------
// Hybrid reconstruction of one cell (Section 3.1 and 3.3).  Q[0..4] = Q_{i-2..i+2}; the result is
// the polynomial P(xi) = sum_n P[n] xi^n on the cell, xi = (x - x_{i+1/2})/dx in [-1, 0].
//   WENO-AO: P = sum_{k<3} (wb_k - wb_3 d_k/d_3) p_k + (wb_3/d_3) p_3 with WENO-Z weights.
//   DF branch (max of the three alphas < threshold): P = Q_i + alpha_i (p_1 - Q_i), which is the
//   paper's zero-mean quadratic with x0 = -dx/2, x1 = dx^2/3 written through p_1.
// NDEG limits the coefficients produced (2 = value and slope at the edge only).
// ------------------------------------------------------------------------------------------------

// ------------------------------------------------------------------------------------------------
// Non-linear time limiter (Section 2.2, eqs. (27)-(29)).  Weight of one reconstruction:
//   a1 = 1 + (tau_Z / (beta_min + eps))^2,  a2 = 1 + (tau_Z / (beta_max + eps))^2,
//   alpha = 2 a2 / (a1 + a2)  (in (0, 1]: 1 on smooth data, -> 0 across a jump),
// beta_min, beta_max over the four indicators of eq. (38), tau_Z of eq. (37).  The weight of an
// interface is the smallest over the characteristic components of the two normal reconstructions
// beside it; ao_weights forms it from the ratios tau/(beta_k + eps) that its weights hold.
// ------------------------------------------------------------------------------------------------

// ------------------------------------------------------------------------------------------------
// Difference form of the reconstruction.  With d_m = Q_{m+1} - Q_m (four differences of the five
// averages), t_k = d_{k+1} - d_k and x01 = t_0 - t_1, x12 = t_1 - t_2, everything but Q_i itself is a
// combination of a few differences:
//   slopes of p_0, p_1, p_2 at the cell centre: h_0 = d_1 + t_0/2, h_1 = d_1 + t_1/2, h_2 = d_2 - t_2/2;
//   beta_k = h_k^2 + 13/12 t_k^2 for the quadratics; for the quartic, with u = x01 + x12 and
//   v = x01 - x12 (u_3 = -u/12, u_4 = v/24 in the Legendre-type basis above),
//   beta_3 = (h_1 + u/12)^2 + 13/12 (t_1 - 11/130 v)^2 + 781/2880 u^2 + 1421461/1310400 v^2.
// Since wb_k - wb_3 d_k/d_3 = d_k (r_k^2 - r_3^2) / sum w and the d_k sum to one, the weights of the
// combination are a_k = d_k (r_k^2 - r_3^2) and H = 1 + r_3^2 over sum w = H + a_0 + a_1 + a_2, and the
// combination is the centred quadratic p_1 corrected by x01 and x12.  a_1 only enters the sum.
// (The beta_k: Jiang-Shu forms for the quadratics, closed form for the quartic, with u_1..u_4 its
// coefficients in its Legendre-type basis on the cell.)
// The 16 reconstructions of an interface are most of the interface kernel's arithmetic, and the kernel
// is bound by instruction issue: this form takes about 76 (edge, two sides sharing t_k and
// 13/12 t_k^2 + eps) and 88 (Gauss points) instructions against 137 and 147 for the evaluation
// through separate candidates (dfw_math_f32.hpp), and rounds the increments instead of the states.
// Measured, FP64, against that form: 4096^2 GKS 13.0 -> 11.5 ms per step, 512^2 GKS 249 -> 221 us per
// step, a ragged LF batch of 48 grids 7.84 -> 6.49 ms.
// ------------------------------------------------------------------------------------------------
constexpr double kBetaU = 781.0 / 2880.0, kBetaV = 1421461.0 / 1310400.0;  // of u^2 and v^2 in beta_3

template <class real>
struct AoWeights {
  real x01, x12, u, v;
  real a0, a1, a2, H, is;   // is = 1 / sum w
  real h0, h1, h2, e1, e2;  // from here on for the reverse only
  real j0, j1, j2;          // B_3 - B_k
  real r[4], ib[4];         // r_k, 1 / B_k
};

// 13/12 t^2 + eps, the part of beta_k + eps that neighbouring reconstructions share.
template <class real>
DFW_HD real beta_curv(real t, const Coef<real>& k) {
  return fmadd(real(13.0 / 12.0) * t, t, k.eps);
}

// d1, d2: the differences beside the cell; m_k = beta_curv(t_k).  With a non-null om also the
// time-limiter weight of the stencil.  REV: also 1/B_k, which the reverse needs.
template <bool REV = false, class real>
DFW_HD AoWeights<real> ao_weights(real d1, real d2, real t0, real t1, real t2, real m0, real m1, real m2,
                                  const Coef<real>& k, real* om = nullptr) {
  AoWeights<real> A;
  A.h0 = fmadd(real(0.5), t0, d1);
  A.h1 = fmadd(real(0.5), t1, d1);
  A.h2 = fmadd(real(-0.5), t2, d2);
  A.x01 = t0 - t1;
  A.x12 = t1 - t2;
  A.u = A.x01 + A.x12;
  A.v = A.x01 - A.x12;
  A.e1 = fmadd(real(1.0 / 12.0), A.u, A.h1);
  A.e2 = fmadd(real(-11.0 / 130.0), A.v, t1);
  // B_k = beta_k + eps
  const real B0 = fmadd(A.h0, A.h0, m0), B1 = fmadd(A.h1, A.h1, m1), B2 = fmadd(A.h2, A.h2, m2);
  real B3 = fmadd(real(kBetaV) * A.v, A.v, k.eps);
  B3 = fmadd(real(kBetaU) * A.u, A.u, B3);
  B3 = fmadd(real(13.0 / 12.0) * A.e2, A.e2, B3);
  B3 = fmadd(A.e1, A.e1, B3);
  A.j0 = B3 - B0;
  A.j1 = B3 - B1;
  A.j2 = B3 - B2;
  // WENO-Z weights, eqs. (36)-(37)
  const real tau = (fabs(A.j0) + fabs(A.j1) + fabs(A.j2)) * real(1.0 / 3.0);
  // r_q = tau / B_q from products of the B_q and one reciprocal of B0 B1 B2 B3 (in FP64 a product of
  // four numbers in [eps, 1e75] stays normal)
  const real P01 = B0 * B1, P23 = B2 * B3;
  real r0, r1, r2, r3;
  if constexpr (REV) {
    const real ip = rcp_pos(P01 * P23), i23 = ip * P23, i01 = ip * P01;
    A.ib[0] = i23 * B1, A.ib[1] = i23 * B0, A.ib[2] = i01 * B3, A.ib[3] = i01 * B2;
    r0 = tau * A.ib[0], r1 = tau * A.ib[1], r2 = tau * A.ib[2], r3 = tau * A.ib[3];
    A.r[0] = r0, A.r[1] = r1, A.r[2] = r2, A.r[3] = r3;
  } else {
    const real ti = tau * rcp_pos(P01 * P23);
    const real t23 = ti * P23, t01 = ti * P01;
    r0 = t23 * B1, r1 = t23 * B0, r2 = t01 * B3, r3 = t01 * B2;
  }
  if (om) {  // tau/(beta_min + eps) and tau/(beta_max + eps) are the largest and smallest ratio
    real rmax = r0 > r1 ? r0 : r1, rmin = r0 < r1 ? r0 : r1;
    rmax = rmax > r2 ? rmax : r2;
    rmax = rmax > r3 ? rmax : r3;
    rmin = rmin < r2 ? rmin : r2;
    rmin = rmin < r3 ? rmin : r3;
    const real a1 = real(1) + rmax * rmax, a2 = real(1) + rmin * rmin;
    *om = real(2) * a2 / (a1 + a2);
  }
  const real s3 = r3 * r3;
  A.a0 = k.d[0] * fmadd(r0, r0, -s3);
  A.a1 = k.d[1] * fmadd(r1, r1, -s3);
  A.a2 = k.d[2] * fmadd(r2, r2, -s3);
  A.H = real(1) + s3;
  A.is = rcp_pos((A.H + A.a0) + (A.a1 + A.a2));
  return A;
}

// The smoothness indicators beta_0..beta_3 of five averages.
template <class real>
struct WenoTerms {
  real b[4];
};

template <class real>
DFW_HD WenoTerms<real> weno_terms(const real* Q) {
  const real d1 = Q[2] - Q[1], d2 = Q[3] - Q[2];
  const real t0 = d1 - (Q[1] - Q[0]), t1 = d2 - d1, t2 = (Q[4] - Q[3]) - d2;
  Coef<real> k{};
  k.eps = real(1);
  const AoWeights<real> A = ao_weights(d1, d2, t0, t1, t2, beta_curv(t0, k), beta_curv(t1, k), beta_curv(t2, k), k);
  const real c = real(13.0 / 12.0);
  return {{A.h0 * A.h0 + c * t0 * t0, A.h1 * A.h1 + c * t1 * t1, A.h2 * A.h2 + c * t2 * t2,
           A.e1 * A.e1 + c * A.e2 * A.e2 + real(kBetaU) * A.u * A.u + real(kBetaV) * A.v * A.v}};
}

// The hybrid reconstruction of one cell at its edge xi = 0: value minus cell average (dv) and slope
// per unit xi (sl), from the differences d1, d2 beside the cell and the second differences.
// DF branch: alpha_i times the centred quadratic's.
template <int RULE = -1, class real>
DFW_HD void recon_edge(real d1, real d2, real t0, real t1, real t2, real m0, real m1, real m2, real a_lo, real a_c,
                       real a_hi, const Coef<real>& k, real& dv, real& sl, real* om = nullptr) {
  const real v1 = fmadd(real(-1.0 / 6.0), t1, real(0.5) * d2);  // of p_1
  if (df_switch<RULE>(a_lo, a_c, a_hi, k)) {
    dv = a_c * v1;
    sl = a_c * d2;
    if (om) (void)ao_weights(d1, d2, t0, t1, t2, m0, m1, m2, k, om);
    return;
  }
  const AoWeights<real> A = ao_weights(d1, d2, t0, t1, t2, m0, m1, m2, k, om);
  const real ca = fmadd(real(1.0 / 3.0), A.a0, real(1.0 / 30.0) * A.H);
  const real cb = fmadd(real(1.0 / 6.0), A.a2, real(0.05) * A.H);
  dv = fmadd(A.is, fmadd(cb, A.x12, ca * A.x01), v1);
  sl = fmadd(A.is, fmadd(A.a0, A.x01, (real(1.0 / 12.0) * A.H) * A.x12), d2);
}

// Gauss points of a segment [-1, 0] (in units of its length): -1/2 -+ kGpDelta, kGpDelta = sqrt(3)/6.
constexpr double kGpDelta = 0.28867513459481288225;

// The hybrid reconstruction of one cell evaluated at the two Gauss points of the segment, xi =
// -1/2 - kGpDelta and -1/2 + kGpDelta (the tangential sweep), in even and odd parts: the values
// are Q_i + ev -/+ od, the slopes (per unit xi) evd -/+ odd.  The polynomial is taken in the centred
// variable zeta = xi + 1/2, where the Gauss points are zeta = -/+ delta, delta = kGpDelta, delta^2 = 1/12:
// P = D0 + D1 zeta + ... + D4 zeta^4 with D0 fixed by the cell mean (D0 = Q_i - D2/12 - D4/80), so that
//   ev = -D4/180, od = delta (D1 + D3/12), evd = D1 + D3/4, odd = delta (2 D2 + D4/3);
// in the difference form D1 = h_1 + is ((a_0 x01 + a_2 x12)/2 + 5/48 H u), D3 = -is H u/12,
// 2 D2 = t_1 + is (a_0 x01 - a_2 x12 - H v/8), D4 = is H v/24.
// DF branch: D1 = alpha_i h_1, 2 D2 = alpha_i t_1, D3 = D4 = 0.
template <int RULE = -1, class real>
DFW_HD void recon_gauss_parts(real d0, real d1, real d2, real d3, real a_lo, real a_c, real a_hi, const Coef<real>& k,
                              real& ev, real& od, real& evd, real& odd) {
  const real t0 = d1 - d0, t1 = d2 - d1, t2 = d3 - d2;
  const real h1 = fmadd(real(0.5), t1, d1), dl = real(kGpDelta);
  if (df_switch<RULE>(a_lo, a_c, a_hi, k)) {
    ev = real(0);
    evd = a_c * h1;
    od = dl * evd;
    odd = dl * (a_c * t1);
    return;
  }
  const AoWeights<real> A = ao_weights(d1, d2, t0, t1, t2, beta_curv(t0, k), beta_curv(t1, k), beta_curv(t2, k), k);
  const real p = A.a0 * A.x01, q = A.a2 * A.x12;
  const real x = p + q, y = p - q, Hu = A.H * A.u, Hv = A.H * A.v;
  const real ish = real(0.5) * A.is;
  od = dl * fmadd(ish, fmadd(real(7.0 / 36.0), Hu, x), h1);
  evd = fmadd(ish, fmadd(real(1.0 / 6.0), Hu, x), h1);
  odd = dl * fmadd(A.is, fmadd(real(-1.0 / 9.0), Hv, y), t1);
  ev = real(-1.0 / 4320.0) * (A.is * Hv);
}

// The same at the two Gauss points from the five averages: values v[g] and slopes d[g].
template <class real, int RULE = -1>
DFW_HD void recon_gauss(const real* Q, real a_lo, real a_c, real a_hi, const Coef<real>& k, real* v, real* d) {
  real ev, od, evd, odd;
  recon_gauss_parts<RULE>(Q[1] - Q[0], Q[2] - Q[1], Q[3] - Q[2], Q[4] - Q[3], a_lo, a_c, a_hi, k, ev, od, evd, odd);
  v[0] = Q[2] + (ev - od);
  v[1] = Q[2] + (ev + od);
  d[0] = evd - odd;
  d[1] = evd + odd;
}

// The polynomial's first NDEG coefficients at the edge from the five averages (NDEG = 2: value and
// slope).
template <class real, int NDEG, int RULE = -1>
DFW_HD void recon_poly(const real* Q, real a_lo, real a_c, real a_hi, const Coef<real>& k, real* P) {
  const real d0 = Q[1] - Q[0], d1 = Q[2] - Q[1], d2 = Q[3] - Q[2], d3 = Q[4] - Q[3];
  const real t0 = d1 - d0, t1 = d2 - d1, t2 = d3 - d2;
  const real m0 = beta_curv(t0, k), m1 = beta_curv(t1, k), m2 = beta_curv(t2, k);
  real dv, sl;
  recon_edge<RULE>(d1, d2, t0, t1, t2, m0, m1, m2, a_lo, a_c, a_hi, k, dv, sl);
  P[0] = Q[2] + dv;
  if (NDEG > 1) P[1] = sl;
  if (NDEG > 2) {  // from the centred coefficients: xi = zeta - 1/2
    real D2, D3 = real(0), D4 = real(0);
    if (df_switch<RULE>(a_lo, a_c, a_hi, k)) {
      D2 = real(0.5) * (a_c * t1);
    } else {
      const AoWeights<real> A = ao_weights(d1, d2, t0, t1, t2, m0, m1, m2, k);
      const real Hu = A.H * A.u, Hv = A.H * A.v;
      D2 = real(0.5) * fmadd(A.is, A.a0 * A.x01 - A.a2 * A.x12 - real(0.125) * Hv, t1);
      D3 = real(-1.0 / 12.0) * (A.is * Hu);
      D4 = real(1.0 / 24.0) * (A.is * Hv);
    }
    P[2] = D2 + real(1.5) * (D3 + D4);
    if (NDEG > 3) P[3] = D3 + real(2) * D4;
    if (NDEG > 4) P[4] = D4;
  }
}

// ------------------------------------------------------------------------------------------------
// Primitive variables and the DF of one Gauss point (Section 3.2):
//   alpha = 1/(1 + D^2), D = |pl-pr|/pl + |pl-pr|/pr + (Ma_n^l - Ma_n^r)^2 + (Ma_t^l - Ma_t^r)^2.
// ------------------------------------------------------------------------------------------------
template <class real>
struct Prim {
  real r, ir, u, v, p, c, ic;  // ir = 1/r, ic = 1/c
};

template <class real>
DFW_HD Prim<real> prim(const real* w, const Coef<real>& k) {
  Prim<real> q;
  q.r = w[0];
  q.ir = rcp_any(w[0]);
  q.u = w[1] * q.ir;
  q.v = w[2] * q.ir;
  q.p = k.gm1 * (w[3] - real(0.5) * (w[1] * q.u + w[2] * q.v));
  sqrt_inv(k.gamma * q.p * q.ir, q.c, q.ic);
  return q;
}

// 1/p as gamma/(rho c^2), from the reciprocals already formed.
template <class real>
DFW_HD real df_factor(const Prim<real>& L, const Prim<real>& R, const Coef<real>& k) {
  const real jump = fabs(L.p - R.p);
  const real dn = L.u * L.ic - R.u * R.ic;
  const real dt = L.v * L.ic - R.v * R.ic;
  const real D = k.gamma * jump * (L.ir * (L.ic * L.ic) + R.ir * (R.ic * R.ic)) + dn * dn + dt * dt;
  return rcp_any(real(1) + D * D);
}

template <class real>
DFW_HD real df_factor(const Prim<real>& L, const Prim<real>& R) {
  real jump = fabs(L.p - R.p);
  real dn = L.u * L.ic - R.u * R.ic;
  real dt = L.v * L.ic - R.v * R.ic;
  real D = jump * (rcp_any(L.p) + rcp_any(R.p)) + dn * dn + dt * dt;
  return rcp_any(real(1) + D * D);
}

// ------------------------------------------------------------------------------------------------
// Lax-Friedrichs flux (Section 2.3) and its time derivative for S2O4: the left and right time
// derivatives come from the Euler equations in primitive form (Cauchy-Kovalevskaya),
//   rho_t = -(u rho_x + rho u_x + v rho_y + rho v_y),  u_t = -(u u_x + v u_y + p_x/rho),
//   v_t = -(u v_x + v v_y + p_y/rho),  p_t = -(u p_x + v p_y + gamma p (u_x + v_y)),
// and dF/dt = (F_t^l + F_t^r)/2 - s (W_t^r - W_t^l)/2 with the LF speed s held fixed.
// ------------------------------------------------------------------------------------------------
// In the products of the density with the derivatives (a = rho u_x, ..., in the order u_x, u_y, v_x,
// v_y), which need no reciprocal: rho_t = -((rho u)_x + (rho v)_y), Au = -rho u_t, Av = -rho v_t.
template <class real>
DFW_HD void euler_time_derivs(const real* w, const Prim<real>& q, const real* wx, const real* wy,
                              const Coef<real>& k, real* wt, real* ft) {
  const real ke = real(0.5) * (q.u * q.u + q.v * q.v);
  const real ux = wx[1] - q.u * wx[0], vx = wx[2] - q.v * wx[0];
  const real uy = wy[1] - q.u * wy[0], vy = wy[2] - q.v * wy[0];
  const real px = k.gm1 * (wx[3] - q.u * wx[1] - q.v * wx[2] + ke * wx[0]);
  const real py = k.gm1 * (wy[3] - q.u * wy[1] - q.v * wy[2] + ke * wy[0]);
  const real rt = -(wx[1] + wy[2]);
  const real Au = fmadd(q.u, ux, fmadd(q.v, uy, px));
  const real Av = fmadd(q.u, vx, fmadd(q.v, vy, py));
  const real pt = -fmadd(q.u, px, fmadd(q.v, py, (k.gamma * q.p * q.ir) * (ux + vy)));
  wt[0] = rt;
  wt[1] = fmadd(rt, q.u, -Au);
  wt[2] = fmadd(rt, q.v, -Av);
  wt[3] = fmadd(pt, k.inv_gm1, fmadd(rt, ke, -fmadd(q.u, Au, q.v * Av)));
  ft[0] = wt[1];
  ft[1] = fmadd(q.u, wt[1] - Au, pt);
  ft[2] = fmadd(wt[1], q.v, -(q.u * Av));
  ft[3] = fmadd(q.u, wt[3] + pt, -(((w[3] + q.p) * q.ir) * Au));
}

template <class real, bool WANT_F>
DFW_HD void lf_flux(const real* wl, const real* wlx, const real* wly, const real* wr, const real* wrx,
                    const real* wry, const Prim<real>& ql, const Prim<real>& qr, const Coef<real>& k,
                    real* F, real* Ft) {
  real sl = fabs(ql.u) + ql.c, sr = fabs(qr.u) + qr.c;
  real s = sl >= sr ? sl : sr;
  real hs = real(0.5) * s;
  if (WANT_F) {
    real Fl[4] = {wl[1], wl[1] * ql.u + ql.p, wl[2] * ql.u, ql.u * (wl[3] + ql.p)};
    real Fr[4] = {wr[1], wr[1] * qr.u + qr.p, wr[2] * qr.u, qr.u * (wr[3] + qr.p)};
#pragma unroll
    for (int c = 0; c < 4; ++c) F[c] = real(0.5) * (Fl[c] + Fr[c]) - hs * (wr[c] - wl[c]);
  }
  real wtl[4], ftl[4], wtr[4], ftr[4];
  euler_time_derivs(wl, ql, wlx, wly, k, wtl, ftl);
  euler_time_derivs(wr, qr, wrx, wry, k, wtr, ftr);
#pragma unroll
  for (int c = 0; c < 4; ++c) Ft[c] = real(0.5) * (ftl[c] + ftr[c]) - hs * (wtr[c] - wtl[c]);
}

// ------------------------------------------------------------------------------------------------
// Gas-kinetic flux (Sections 2.2 and 3.4), Euler case: physical tau = 0 outside the exponential,
// numerical tau_n = c1 dt + c2 |(pl-pr)/(pl+pr)| dt inside it.
// Moments <u^a v^b xi^2c> of a Maxwellian (normalised by rho) factorise; mu_n are those of u.
// ------------------------------------------------------------------------------------------------
// The slopes of a Maxwellian enter the flux only through moments <(s . psi) u^a v^b psi>, and since
// rho (s . psi) g is the derivative of rho g in that direction, such a moment is the derivative of
// rho <u^a v^b psi>, a product of u-moments mu_n(U, h) with polynomials in V and h = p/rho.  So no slope s is formed: with the derivative's density r = rho_x, a = rho U_x,
// b = rho V_x and e = rho h_x, and d mu_n/dU = n mu_{n-1}, d mu_n/dh = n (n-1)/2 mu_{n-2},
//   D_n = (rho mu_n)_x = r mu_n + n a mu_{n-1} + n (n-1)/2 e mu_{n-2}
// in full space and, for n >= 2, in a half space too; there mu_0 and mu_1 have the boundary terms
//   D_0 = r mu_0 + G (a - U e/(2h)),  D_1 = r mu_1 + a mu_0 + G e/2,  G = +-exp(-U^2/(2h)) / sqrt(2 pi h).
// This took the flux of one Gauss point from about 1 200 instructions (slopes from the inverse moment
// matrix, moments up to order 6 folded per slope) to about 600, most of the rest being the exponential,
// error function and root of the two half spaces.
template <class real>
struct GasSlope {
  real r, a, b, e;
};

template <class real>
DFW_HD GasSlope<real> gas_slope(const real* w, real U, real V, real h, real ke, const Coef<real>& k) {
  GasSlope<real> s;
  s.r = w[0];
  s.a = w[1] - U * w[0];
  s.b = w[2] - V * w[0];
  s.e = fmadd(-h, w[0], k.gm1 * (w[3] - U * w[1] - V * w[2] + ke * w[0]));
  return s;
}

// D_n for n = 1 (full space) and n = 2, 3, 4 from the u-moments mu[0..4].
template <class real>
DFW_HD real slope_d1(const GasSlope<real>& s, const real* mu) { return fmadd(s.r, mu[1], s.a * mu[0]); }
template <class real>
DFW_HD real slope_d2(const GasSlope<real>& s, const real* mu) {
  return fmadd(s.r, mu[2], fmadd(real(2) * s.a, mu[1], s.e * mu[0]));
}
template <class real>
DFW_HD real slope_d3(const GasSlope<real>& s, const real* mu) {
  return fmadd(s.r, mu[3], real(3) * fmadd(s.a, mu[2], s.e * mu[1]));
}
template <class real>
DFW_HD real slope_d4(const GasSlope<real>& s, const real* mu) {
  return fmadd(s.r, mu[4], fmadd(real(4) * s.a, mu[3], (real(6) * s.e) * mu[2]));
}

// M += (rho <u^2 psi>)_x + (rho <u v psi>)_y for the slopes sx, sy of one Maxwellian (mean V, X = <v^2 +
// xi^2>, d1 = D_1 of sy); the energy component is left doubled.
template <class real>
DFW_HD void add_second_moments(const GasSlope<real>& sx, const GasSlope<real>& sy, const real* mu, real V, real h,
                               real X, real d1, const Coef<real>& k, real* M) {
  const real K1 = k.K + real(1), K3 = k.K + real(3);
  const real d2 = slope_d2(sx, mu), d3 = slope_d3(sx, mu), d4 = slope_d4(sx, mu);
  M[0] += d2;
  M[1] += d3;
  M[2] += fmadd(V, d2, sx.b * mu[2]);
  M[3] += fmadd(X, d2, fmadd(mu[2], fmadd(real(2) * V, sx.b, K1 * sx.e), d4));
  const real t2 = slope_d2(sy, mu), t3 = slope_d3(sy, mu);
  const real vb = real(2) * V * sy.b, Z = fmadd(real(2), h, X);  // Z = <v^3 + v xi^2> / V
  M[0] += fmadd(V, d1, mu[1] * sy.b);
  M[1] += fmadd(V, t2, mu[2] * sy.b);
  M[2] += fmadd(fmadd(V, V, h), d1, mu[1] * (vb + sy.e));
  M[3] += fmadd(V, fmadd(Z, d1, fmadd(mu[1], fmadd(K3, sy.e, vb), t3)), sy.b * fmadd(Z, mu[1], mu[3]));
}

// Half-space part of one side (SG = +1: left state, u > 0; -1: right state, u < 0) added to the sums; energy
// components doubled.  s2h = sqrt(2 h) and its reciprocal is.
template <int SG, class real>
DFW_HD void gks_side(const Prim<real>& q, real h, real s2h, real is, const real* wn, const real* wt,
                     const Coef<real>& k, real* Wc, real* Wcn, real* Wct, real* Flr, real* Malr) {
  const real inv_sqrt_pi = real(SG * 0.56418958354775628695);
  const real U = q.u, V = q.v, K1 = k.K + real(1);
  const real z = is * U, ex = exp(-(z * z));
  real mu[5];
  mu[0] = real(0.5) * erfc(SG > 0 ? -z : z);
  mu[1] = fmadd(U, mu[0], (real(0.5) * inv_sqrt_pi) * s2h * ex);
  mu[2] = fmadd(U, mu[1], h * mu[0]);
  mu[3] = fmadd(U, mu[2], real(2) * h * mu[1]);
  mu[4] = fmadd(U, mu[3], real(3) * h * mu[2]);
  const real G = inv_sqrt_pi * is * ex;
  const real ke = real(0.5) * (U * U + V * V), X = fmadd(V, V, K1 * h);
  const GasSlope<real> sx = gas_slope(wn, U, V, h, ke, k), sy = gas_slope(wt, U, V, h, ke, k);
  const real zi = z * is;  // U / (2 h)
  {
    const real d0 = fmadd(sx.r, mu[0], G * fmadd(-zi, sx.e, sx.a));
    Wcn[0] += d0;
    Wcn[1] += fmadd(real(0.5) * G, sx.e, slope_d1(sx, mu));
    Wcn[2] += fmadd(V, d0, sx.b * mu[0]);
    Wcn[3] += fmadd(X, d0, fmadd(mu[0], fmadd(real(2) * V, sx.b, K1 * sx.e), slope_d2(sx, mu)));
  }
  const real t0 = fmadd(sy.r, mu[0], G * fmadd(-zi, sy.e, sy.a));
  const real t1 = fmadd(real(0.5) * G, sy.e, slope_d1(sy, mu));
  Wct[0] += t0;
  Wct[1] += t1;
  Wct[2] += fmadd(V, t0, sy.b * mu[0]);
  Wct[3] += fmadd(X, t0, fmadd(mu[0], fmadd(real(2) * V, sy.b, K1 * sy.e), slope_d2(sy, mu)));
  add_second_moments(sx, sy, mu, V, h, X, t1, k, Malr);
  const real m0 = q.r * mu[0], m1 = q.r * mu[1], m2 = q.r * mu[2];
  Wc[0] += m0;
  Wc[1] += m1;
  Wc[2] = fmadd(V, m0, Wc[2]);
  Wc[3] += fmadd(X, m0, m2);
  Flr[0] += m1;
  Flr[1] += m2;
  Flr[2] = fmadd(V, m1, Flr[2]);
  Flr[3] += fmadd(X, m1, q.r * mu[3]);
}

// GKS flux at one Gauss point.  wl/wr: states; wln/wrn: normal derivatives; wlt/wrt: tangential
// derivatives.  Outputs F (if WANT_F) and dF/dt by the S2O4 fit of eqs. (23)-(25) to the time
// integrals over dt and dt/2, written in closed form:
//   F    = cf1 Fc + cf2 (Ma_c - Ma_lr) + (1 - cf1) F_lr
//   F_t  = ct1 (Fc - F_lr) + ct2 (Ma_c - Ma_lr) + MA_c
// with x = tau/dt, E2 = exp(-1/(2 x)), E1 = E2^2, z = (1 - E2) (3 - E2):
//   cf1 = 1 - x z,  cf2 = dt (x^2 z + x E2 (E2 - 2)),
//   ct1 = 4 x (1 - E2)^2 / dt,  ct2 = 4 (x E2 (1 - E2) - x^2 (1 - E2)^2).
// Fc and MA_c (the time derivative of the flux from the compatibility condition) are the Euler flux
// of the equilibrium state and its Cauchy-Kovalevskaya derivative.  isl: 1/sqrt(2 h) of the two sides.
template <bool WANT_F, class real>
DFW_HD void gks_point_flux(const real* wln, const real* wlt, const real* wrn, const real* wrt, const Prim<real>& ql,
                           const Prim<real>& qr, real dt, const Coef<real>& k, real* F, real* Ft, real* isl) {
  real Wc[4] = {0, 0, 0, 0}, Wcn[4] = {0, 0, 0, 0}, Wct[4] = {0, 0, 0, 0};
  real Flr[4] = {0, 0, 0, 0}, Malr[4] = {0, 0, 0, 0};
  real s2h;
  real h = ql.p * ql.ir;
  sqrt_inv(real(2) * h, s2h, isl[0]);
  gks_side<1>(ql, h, s2h, isl[0], wln, wlt, k, Wc, Wcn, Wct, Flr, Malr);
  h = qr.p * qr.ir;
  sqrt_inv(real(2) * h, s2h, isl[1]);
  gks_side<-1>(qr, h, s2h, isl[1], wrn, wrt, k, Wc, Wcn, Wct, Flr, Malr);
  Wc[3] *= real(0.5);
  Wcn[3] *= real(0.5);
  Wct[3] *= real(0.5);
  // equilibrium state at the interface
  Prim<real> c;
  c.r = Wc[0];
  c.ir = rcp_any(Wc[0]);
  c.u = Wc[1] * c.ir;
  c.v = Wc[2] * c.ir;
  c.p = k.gm1 * (Wc[3] - real(0.5) * (Wc[1] * c.u + Wc[2] * c.v));
  h = c.p * c.ir;
  real Mac[4] = {0, 0, 0, 0}, MAc[4], wt[4];
  {
    const real U = c.u, V = c.v, K1 = k.K + real(1);
    real mu[5];
    mu[0] = real(1);
    mu[1] = U;
    mu[2] = fmadd(U, U, h);
    mu[3] = fmadd(U, mu[2], real(2) * h * U);
    mu[4] = fmadd(U, mu[3], real(3) * h * mu[2]);
    const real ke = real(0.5) * (U * U + V * V);
    const GasSlope<real> sx = gas_slope(Wcn, U, V, h, ke, k), sy = gas_slope(Wct, U, V, h, ke, k);
    add_second_moments(sx, sy, mu, V, h, fmadd(V, V, K1 * h), slope_d1(sy, mu), k, Mac);
  }
  euler_time_derivs(Wc, c, Wcn, Wct, k, wt, MAc);
  const real Fc[4] = {Wc[1], fmadd(Wc[1], c.u, c.p), Wc[2] * c.u, c.u * (Wc[3] + c.p)};
  // time coefficients
  const real x = k.c1 + k.c2 * fabs((ql.p - qr.p) * rcp_any(ql.p + qr.p));
  const real E2 = exp(real(-0.5) * rcp_any(x));
  const real om = real(1) - E2, xo = x * om;
  const real ct1 = (real(4) * xo * om) * rcp_any(dt), ct2 = real(4) * xo * (E2 - xo);
  const real z = om * (real(3) - E2);
  const real cf1 = real(1) - x * z, cf2 = dt * (x * fmadd(x, z, E2 * (E2 - real(2))));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const real half = i == 3 ? real(0.5) : real(1);
    const real dM = half * (Mac[i] - Malr[i]), flr = half * Flr[i], dF = Fc[i] - flr;
    Ft[i] = fmadd(ct1, dF, fmadd(ct2, dM, MAc[i]));
    if (WANT_F) F[i] = fmadd(cf1, dF, fmadd(cf2, dM, flr));
  }
}

template <class real, bool WANT_F>
DFW_HD void gks_flux(const real* wl, const real* wln, const real* wlt, const real* wr, const real* wrn,
                     const real* wrt, const Prim<real>& ql, const Prim<real>& qr, real dt,
                     const Coef<real>& k, real* F, real* Ft) {
  (void)wl;
  (void)wr;
  real isl[2];
  gks_point_flux<WANT_F>(wln, wlt, wrn, wrt, ql, qr, dt, k, F, Ft, isl);
}

// The DF of a Gauss point from isl = 1/sqrt(2 h) of its two sides, which the gas-kinetic flux has:
// 1/p = 2 isl^2/rho, 1/c = isl sqrt(2/gamma); gamma D is formed, and 1/(1 + D^2) = gamma^2/(gamma^2 + (gamma D)^2).
template <class real>
DFW_HD real df_factor_gks(const Prim<real>& L, const Prim<real>& R, const real* isl, const Coef<real>& k) {
  const real dn = L.u * isl[0] - R.u * isl[1], dt = L.v * isl[0] - R.v * isl[1];
  const real jp = fabs(L.p - R.p) * (L.ir * (isl[0] * isl[0]) + R.ir * (isl[1] * isl[1]));
  const real D = real(2) * fmadd(k.gamma, jp, fmadd(dn, dn, dt * dt));
  const real g2 = k.gamma * k.gamma;
  return quotient_any(g2, fmadd(D, D, g2));  // 1 in uniform flow, for any gamma
}

// ------------------------------------------------------------------------------------------------
// One interface segment, normal sweep (Section 3.1, Algorithm 1): from the six cells along the
// normal (cells f-3..f+2 around interface f) and the DF of cells f-2..f+1, the line values of the
// left state (cell f-1 at its right edge) and the right state (cell f at its left edge, mirrored
// stencil) and their normal derivatives, in conservative variables.  B: the basis of the interface.
// The five differences of neighbouring cells are projected (not the six cells), and the increments
// over the cell averages projected back; the mirrored stencil's differences are the same five in
// reverse with the opposite sign.
// ------------------------------------------------------------------------------------------------
template <bool CHAR, class real>
DFW_HD void normal_sweep_basis(const Basis<real>& B, const real (*cell)[4], real a0, real a1, real a2, real a3,
                               real inv_dn, const Coef<real>& k, real* wl, real* wr, real* wln, real* wrn,
                               real* om = nullptr) {
  real D[5][4];
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    real w[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) w[c] = cell[m + 1][c] - cell[m][c];
    to_recon<CHAR>(B, w, D[m]);
  }
  real ql[4], qld[4], qr[4], qrd[4];
  real omin = real(1), wk = real(1);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const real d1 = D[1][c], d2 = D[2][c], d3 = D[3][c];
    const real t0 = d1 - D[0][c], t1 = d2 - d1, t2 = d3 - d2, t3 = D[4][c] - d3;
    const real m0 = beta_curv(t0, k), m1 = beta_curv(t1, k), m2 = beta_curv(t2, k), m3 = beta_curv(t3, k);
    real dv, sl;
    recon_edge(d1, d2, t0, t1, t2, m0, m1, m2, a0, a1, a2, k, dv, sl, om ? &wk : nullptr);
    if (om) omin = omin < wk ? omin : wk;
    ql[c] = dv;
    qld[c] = sl * inv_dn;
    recon_edge(d3, d2, -t3, -t2, -t1, m3, m2, m1, a3, a2, a1, k, dv, sl, om ? &wk : nullptr);
    if (om) omin = omin < wk ? omin : wk;
    qr[c] = -dv;
    qrd[c] = sl * inv_dn;
  }
  from_recon<CHAR>(B, ql, wl);
  from_recon<CHAR>(B, qr, wr);
  from_recon<CHAR>(B, qld, wln);
  from_recon<CHAR>(B, qrd, wrn);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    wl[c] += cell[2][c];
    wr[c] += cell[3][c];
  }
  if (om) *om = omin;  // time-limiter weight of the interface (eq. (29)): both sides, all components
}

template <class real, bool CHAR = true>
DFW_HD void normal_sweep(const real (*cell)[4], real a0, real a1, real a2, real a3, real inv_dn,
                         const Coef<real>& k, real* wl, real* wr, real* wln, real* wrn, real* om = nullptr) {
  normal_sweep_basis<CHAR>(recon_basis<CHAR>(cell[2], cell[3], k), cell, a0, a1, a2, a3, inv_dn, k, wl, wr, wln,
                                 wrn, om);
}

// ------------------------------------------------------------------------------------------------
// One interface segment, tangential sweep: B is the basis of the segment (of its two cells);
// line(side, m, c) returns component c of the side's line value on segment row m-2..m+2;
// alpha[side][0..2] are the DF of the same-side cells on rows -1, 0, +1.  Produces the states and
// their tangential derivatives at the Gauss points, [side][gauss point][component].
// ------------------------------------------------------------------------------------------------
template <bool CHAR, class LineFn, class real>
DFW_HD void segment_states(const Basis<real>& B, LineFn line, const real (*alpha)[3], real inv_dt,
                           const Coef<real>& k, real (*gw)[2][4], real (*gwt)[2][4]) {
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    real D[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      real w[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) w[c] = line(side, m + 1, c) - line(side, m, c);
      to_recon<CHAR>(B, w, D[m]);
    }
    real ev[4], od[4], evd[4], odd[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      recon_gauss_parts(D[0][c], D[1][c], D[2][c], D[3][c], alpha[side][0], alpha[side][1], alpha[side][2], k, ev[c],
                        od[c], evd[c], odd[c]);
      evd[c] *= inv_dt;
      odd[c] *= inv_dt;
    }
    // even and odd parts back to conservative variables, then the two Gauss points
    real e[4], o[4];
    from_recon<CHAR>(B, ev, e);
    from_recon<CHAR>(B, od, o);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const real m = line(side, 2, c) + e[c];
      gw[side][0][c] = m - o[c];
      gw[side][1][c] = m + o[c];
    }
    from_recon<CHAR>(B, evd, e);
    from_recon<CHAR>(B, odd, o);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      gwt[side][0][c] = e[c] - o[c];
      gwt[side][1][c] = e[c] + o[c];
    }
  }
}

// The sums over the two Gauss points of the flux and its time derivative (quadrature weights applied
// by the caller) and the product of the two Gauss-point DF values.
template <int FLUX, bool WANT_F, bool WANT_DF, class real>
DFW_HD void segment_point_fluxes(const real (*gw)[2][4], const real (*gwt)[2][4], const real* wln, const real* wrn,
                                 real dt, const Coef<real>& k, real* Fs, real* Fts, real& dfp) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    Fs[c] = real(0);
    Fts[c] = real(0);
  }
  dfp = real(1);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    Prim<real> ql = prim(gw[0][g], k), qr = prim(gw[1][g], k);
    real F[4], Ft[4];
    real df;
    if (FLUX == 0) {
      lf_flux<real, WANT_F>(gw[0][g], wln, gwt[0][g], gw[1][g], wrn, gwt[1][g], ql, qr, k, F, Ft);
      if (WANT_DF) df = df_factor(ql, qr, k);
    } else {
      real isl[2];
      gks_point_flux<WANT_F>(wln, gwt[0][g], wrn, gwt[1][g], ql, qr, dt, k, F, Ft, isl);
      if (WANT_DF) df = df_factor_gks(ql, qr, isl, k);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (WANT_F) Fs[c] += F[c];
      Fts[c] += Ft[c];
    }
    if (WANT_DF) dfp *= df;
  }
}

template <class real, int FLUX, bool WANT_F, bool WANT_DF, bool CHAR = true, class LineFn>
DFW_HD void segment_fluxes(const real* wa, const real* wb, LineFn line, const real (*alpha)[3],
                           const real* wln, const real* wrn, real dt, real inv_dt, const Coef<real>& k,
                           real* Fs, real* Fts, real& dfp) {
  real gw[2][2][4], gwt[2][2][4];
  segment_states<CHAR>(recon_basis<CHAR>(wa, wb, k), line, alpha, inv_dt, k, gw, gwt);
  segment_point_fluxes<FLUX, WANT_F, WANT_DF>(gw, gwt, wln, wrn, dt, k, Fs, Fts, dfp);
}

}  // namespace dfw
