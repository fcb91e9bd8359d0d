// Hand-written reverse-mode (adjoint) counterparts of the device arithmetic in dfw_math.hpp.
//
// Convention: for y = f(x), f_adj(x, ..., ly, lx) adds (dy/dx)^T ly into lx (accumulates; callers
// zero the adjoint arrays).  Each adjoint recomputes the forward intermediates it needs from the
// primal inputs.  Kinks follow a fixed subgradient convention: d|x| = sign(x) with sign(0) = 0;
// max(a, b) routes to a when a >= b; the hybrid switch of eq. (42) has zero derivative (the branch
// taken is differentiated); dt is held fixed.
#pragma once

#include "dfw_math.hpp"

namespace dfw {

template <class real>
DFW_HD real sgn(real x) {
  return x > real(0) ? real(1) : (x < real(0) ? real(-1) : real(0));
}

// ------------------------------------------------------------------------------------------------
// Characteristic basis.
// ------------------------------------------------------------------------------------------------
template <class real>
struct BasisAdj {
  real u, v, c, ic, H, hq2, b1, b2;
  DFW_HD void zero() { u = v = c = ic = H = hq2 = b1 = b2 = real(0); }
};

template <class real>
DFW_HD void make_basis_adj(const real* wa, const real* wb, const Coef<real>& k, const BasisAdj<real>& lB, real* lwa,
                           real* lwb) {
  const real h = real(0.5);
  real r = h * (wa[0] + wb[0]), m = h * (wa[1] + wb[1]), n = h * (wa[2] + wb[2]), e = h * (wa[3] + wb[3]);
  real ir = real(1) / r;
  real u = m * ir, v = n * ir;
  real hq2 = h * (u * u + v * v);
  real p = k.gm1 * (e - r * hq2);
  real c2 = k.gamma * p * ir;
  real c = sqrt(c2);
  real ic = real(1) / c;
  real b1 = real(0.5) * k.gm1 / c2;
  real l_hq2 = lB.hq2 + lB.b2 * b1;
  real l_b1 = lB.b1 + lB.b2 * hq2;
  real l_c2 = -l_b1 * b1 / c2;
  real l_e = lB.H * ir, l_p = lB.H * ir, l_ir = lB.H * (e + p);
  real l_c = lB.c - real(0.5) * lB.ic * ic * ic;
  l_c2 += l_c * real(0.5) / c;
  l_p += l_c2 * k.gamma * ir;
  l_ir += l_c2 * k.gamma * p;
  l_e += l_p * k.gm1;
  real l_r = -l_p * k.gm1 * hq2;
  l_hq2 += -l_p * k.gm1 * r;
  real l_u = lB.u + l_hq2 * u, l_v = lB.v + l_hq2 * v;
  real l_m = l_u * ir, l_n = l_v * ir;
  l_ir += l_u * m + l_v * n;
  l_r += -l_ir * ir * ir;
  real lw[4] = {h * l_r, h * l_m, h * l_n, h * l_e};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    lwa[i] += lw[i];
    lwb[i] += lw[i];
  }
}

template <class real>
DFW_HD void project_adj(const Basis<real>& B, const real* w, const real* lq, real* lw, BasisAdj<real>& lB) {
  real lT = lq[0] - real(2) * lq[1] + lq[3];
  real ls = lq[0] - lq[3];
  lw[0] += lq[1] - B.v * lq[2];
  lw[2] += lq[2];
  lB.v += -w[0] * lq[2];
  // s = (u w0 - w1) ic
  lB.u += ls * w[0] * B.ic;
  lw[0] += ls * B.u * B.ic;
  lw[1] += -ls * B.ic;
  lB.ic += ls * (B.u * w[0] - w[1]);
  // T = b2 w0 - b1 X, X = u w1 + v w2 - w3
  real X = B.u * w[1] + B.v * w[2] - w[3];
  lB.b2 += lT * w[0];
  lw[0] += lT * B.b2;
  lB.b1 += -lT * X;
  real lX = -lT * B.b1;
  lB.u += lX * w[1];
  lw[1] += lX * B.u;
  lB.v += lX * w[2];
  lw[2] += lX * B.v;
  lw[3] += -lX;
}

// unproject_adj in two parts: lq += R^T lw does not depend on q; the basis part does.
template <class real>
DFW_HD void unproject_adj_q(const Basis<real>& B, const real* lw, real* lq) {
  real lw0 = lw[0] + B.u * lw[1] + B.v * lw[2];
  real ldq = B.c * lw[1] + B.u * B.c * lw[3];
  lq[0] += lw0 - ldq + lw[3] * B.H;
  lq[1] += lw0 + lw[3] * B.hq2;
  lq[2] += lw[2] + lw[3] * B.v;
  lq[3] += lw0 + ldq + lw[3] * B.H;
}

template <class real>
DFW_HD void unproject_adj_B(const Basis<real>& B, const real* q, const real* lw, BasisAdj<real>& lB) {
  real w0 = q[0] + q[1] + q[3];
  real dq = q[3] - q[0];
  lB.u += lw[1] * w0 + lw[3] * B.c * dq;
  lB.c += lw[1] * dq + lw[3] * B.u * dq;
  lB.v += lw[2] * w0 + lw[3] * q[2];
  lB.H += lw[3] * (q[0] + q[3]);
  lB.hq2 += lw[3] * q[1];
}

template <class real>
DFW_HD void unproject_adj(const Basis<real>& B, const real* q, const real* lw, real* lq, BasisAdj<real>& lB) {
  unproject_adj_B(B, q, lw, lB);
  unproject_adj_q(B, lw, lq);
}

template <class real>
DFW_HD void basis_adj_add(BasisAdj<real>& a, const BasisAdj<real>& b) {
  a.u += b.u;
  a.v += b.v;
  a.c += b.c;
  a.ic += b.ic;
  a.H += b.H;
  a.hq2 += b.hq2;
  a.b1 += b.b1;
  a.b2 += b.b2;
}

// Component C of R^T lw (the part of unproject_adj that does not depend on q).
template <int C, class real>
DFW_HD real unproject_adj_q_comp(const Basis<real>& B, const real* lw) {
  if (C == 2) return lw[2] + lw[3] * B.v;
  const real lw0 = lw[0] + B.u * lw[1] + B.v * lw[2];
  if (C == 1) return lw0 + lw[3] * B.hq2;
  const real ldq = B.c * lw[1] + B.u * B.c * lw[3];
  return C == 0 ? lw0 - ldq + lw[3] * B.H : lw0 + ldq + lw[3] * B.H;
}

// Basis part of unproject_adj for component C of q alone (the four parts sum to unproject_adj_B).
template <int C, class real>
DFW_HD void unproject_adj_B_comp(const Basis<real>& B, real qc, const real* lw, BasisAdj<real>& lB) {
  if (C == 0) {
    lB.u += lw[1] * qc - lw[3] * B.c * qc;
    lB.c += -lw[1] * qc - lw[3] * B.u * qc;
    lB.v += lw[2] * qc;
    lB.H += lw[3] * qc;
  } else if (C == 1) {
    lB.u += lw[1] * qc;
    lB.v += lw[2] * qc;
    lB.hq2 += lw[3] * qc;
  } else if (C == 2) {
    lB.v += lw[3] * qc;
  } else {
    lB.u += lw[1] * qc + lw[3] * B.c * qc;
    lB.c += lw[1] * qc + lw[3] * B.u * qc;
    lB.v += lw[2] * qc;
    lB.H += lw[3] * qc;
  }
}

// ------------------------------------------------------------------------------------------------
// Hybrid reconstruction in the difference form of dfw_math.hpp, reversed.  ao_weights_adj takes the
// weights back to the differences: from the adjoints of a_0, a_2, H, is, x01, x12 (those of the
// combination) to those of d_1, d_2, t_0, t_1, t_2 (accumulated).  About 60 instructions; the reverse
// through separate candidates and five averages took about 220.
// ------------------------------------------------------------------------------------------------
// y with the sign of x, zero at x = 0.
template <class real>
DFW_HD real signed_by(real y, real x) {
  return x > real(0) ? y : (x < real(0) ? -y : real(0));
}

template <class real>
DFW_HD void ao_weights_adj(const AoWeights<real>& A, real t0, real t1, real t2, const Coef<real>& k, real la0, real la2,
                           real lH, real lis, real lx01, real lx12, real& ld1, real& ld2, real& lt0, real& lt1,
                           real& lt2) {
  const real lS = -(lis * A.is) * A.is;
  const real c0 = k.d[0] * (la0 + lS), c1 = k.d[1] * lS, c2 = k.d[2] * (la2 + lS);
  const real c3 = (lH + lS) - (c0 + c1 + c2);  // of r_3^2
  // half the adjoints of r_k, over B_k
  const real g0 = (c0 * A.r[0]) * A.ib[0], g1 = (c1 * A.r[1]) * A.ib[1], g2 = (c2 * A.r[2]) * A.ib[2];
  const real g3 = (c3 * A.r[3]) * A.ib[3];
  const real T = real(4.0 / 3.0) * ((g0 + g1) + (g2 + g3));  // twice the adjoint of each |B_3 - B_k|
  const real s0 = signed_by(T, A.j0), s1 = signed_by(T, A.j1), s2 = signed_by(T, A.j2);
  // twice the adjoints of B_k
  const real w0 = fmadd(real(-4) * g0, A.r[0], -s0), w1 = fmadd(real(-4) * g1, A.r[1], -s1);
  const real w2 = fmadd(real(-4) * g2, A.r[2], -s2), w3 = fmadd(real(-4) * g3, A.r[3], s0 + s1 + s2);
  const real k1312 = real(13.0 / 12.0);
  const real le1 = A.e1 * w3, le2 = (k1312 * A.e2) * w3;
  const real lu = fmadd(real(kBetaU) * A.u, w3, real(1.0 / 12.0) * le1);
  const real lv = fmadd(real(kBetaV) * A.v, w3, real(-11.0 / 130.0) * le2);
  lx01 += lu + lv;
  lx12 += lu - lv;
  const real lh0 = A.h0 * w0, lh1 = fmadd(A.h1, w1, le1), lh2 = A.h2 * w2;
  lt0 += fmadd(k1312 * t0, w0, fmadd(real(0.5), lh0, lx01));
  lt1 += fmadd(k1312 * t1, w1, fmadd(real(0.5), lh1, le2)) + (lx12 - lx01);
  lt2 += fmadd(k1312 * t2, w2, fmadd(real(-0.5), lh2, -lx12));
  ld1 += lh0 + lh1;
  ld2 += lh2;
}

// Adjoints of d_1, d_2 and t_k -> those of the four differences.
template <class real>
DFW_HD void differences_adj(real ld1, real ld2, real lt0, real lt1, real lt2, real* ld) {
  ld[0] = -lt0;
  ld[1] = ld1 + (lt0 - lt1);
  ld[2] = ld2 + (lt1 - lt2);
  ld[3] = lt2;
}

// Reverse of recon_edge on the differences d[0..3]: ldv, lsl -> ld (overwrites d, which is not needed
// any more) and the DF of the centre cell (DF branch); also the forward dv and sl.
template <int RULE = -1, class real>
DFW_HD void recon_edge_adj(real* d, real a_lo, real a_c, real a_hi, const Coef<real>& k, real ldv, real lsl,
                           real& la_c, real& dv, real& sl) {
  const real d1 = d[1], d2 = d[2];
  const real t0 = d1 - d[0], t1 = d2 - d1, t2 = d[3] - d2;
  const real v1 = fmadd(real(-1.0 / 6.0), t1, real(0.5) * d2);
  if (df_switch<RULE>(a_lo, a_c, a_hi, k)) {
    dv = a_c * v1;
    sl = a_c * d2;
    la_c += ldv * v1 + lsl * d2;
    const real lv = a_c * ldv;
    differences_adj(real(0), fmadd(real(0.5), lv, a_c * lsl), real(0), real(-1.0 / 6.0) * lv, real(0), d);
    return;
  }
  const AoWeights<real> A = ao_weights<true>(d1, d2, t0, t1, t2, beta_curv(t0, k), beta_curv(t1, k), beta_curv(t2, k), k);
  const real ca = fmadd(real(1.0 / 3.0), A.a0, real(1.0 / 30.0) * A.H);
  const real cb = fmadd(real(1.0 / 6.0), A.a2, real(0.05) * A.H);
  const real H12 = real(1.0 / 12.0) * A.H;
  const real Y = fmadd(cb, A.x12, ca * A.x01), X = fmadd(A.a0, A.x01, H12 * A.x12);
  dv = fmadd(A.is, Y, v1);
  sl = fmadd(A.is, X, d2);
  const real lY = ldv * A.is, lX = lsl * A.is;
  const real la0 = A.x01 * fmadd(real(1.0 / 3.0), lY, lX), la2 = A.x12 * (real(1.0 / 6.0) * lY);
  const real lH = fmadd(A.x12, fmadd(real(1.0 / 12.0), lX, real(0.05) * lY), A.x01 * (real(1.0 / 30.0) * lY));
  real ld1 = real(0), ld2 = fmadd(real(0.5), ldv, lsl), lt0 = real(0), lt1 = real(-1.0 / 6.0) * ldv, lt2 = real(0);
  ao_weights_adj(A, t0, t1, t2, k, la0, la2, lH, fmadd(ldv, Y, lsl * X), fmadd(lY, ca, lX * A.a0),
                 fmadd(lY, cb, lX * H12), ld1, ld2, lt0, lt1, lt2);
  differences_adj(ld1, ld2, lt0, lt1, lt2, d);
}

// Reverse of recon_gauss_parts on the differences d[0..3]: lev, lod, levd, lodd -> ld (overwrites d) and
// the DF of the centre cell (DF branch); also the forward parts.
template <int RULE = -1, class real>
DFW_HD void recon_gauss_parts_adj(real* d, real a_lo, real a_c, real a_hi, const Coef<real>& k, real lev, real lod,
                                  real levd, real lodd, real& la_c, real& ev, real& od, real& evd, real& odd) {
  const real d1 = d[1], d2 = d[2];
  const real t0 = d1 - d[0], t1 = d2 - d1, t2 = d[3] - d2;
  const real dl = real(kGpDelta);
  const real lo = dl * lod, lod2 = dl * lodd;  // of od/delta, odd/delta
  if (df_switch<RULE>(a_lo, a_c, a_hi, k)) {
    const real h1 = fmadd(real(0.5), t1, d1);
    ev = real(0);
    evd = a_c * h1;
    od = dl * evd;
    odd = dl * (a_c * t1);
    const real s = lo + levd;
    la_c += h1 * s + t1 * lod2;
    const real lh1 = a_c * s;
    differences_adj(lh1, real(0), real(0), fmadd(real(0.5), lh1, a_c * lod2), real(0), d);
    return;
  }
  const AoWeights<real> A = ao_weights<true>(d1, d2, t0, t1, t2, beta_curv(t0, k), beta_curv(t1, k), beta_curv(t2, k), k);
  const real p = A.a0 * A.x01, q = A.a2 * A.x12, Hu = A.H * A.u, Hv = A.H * A.v;
  const real x = p + q, ish = real(0.5) * A.is;
  const real E1 = fmadd(real(7.0 / 36.0), Hu, x), E2 = fmadd(real(1.0 / 6.0), Hu, x);
  const real E3 = fmadd(real(-1.0 / 9.0), Hv, p - q), zv = real(-1.0 / 4320.0) * Hv;
  od = dl * fmadd(ish, E1, A.h1);
  evd = fmadd(ish, E2, A.h1);
  odd = dl * fmadd(A.is, E3, t1);
  ev = A.is * zv;
  const real lis = fmadd(real(0.5), fmadd(lo, E1, levd * E2), fmadd(lod2, E3, lev * zv));
  const real lE1 = ish * lo, lE2 = ish * levd, lE3 = A.is * lod2;
  const real lp = (lE1 + lE2) + lE3, lq = (lE1 + lE2) - lE3;
  const real lHu = fmadd(real(7.0 / 36.0), lE1, real(1.0 / 6.0) * lE2);
  const real lHv = fmadd(real(-1.0 / 9.0), lE3, real(-1.0 / 4320.0) * (A.is * lev));
  const real lh1 = lo + levd;
  real ld1 = lh1, ld2 = real(0), lt0 = real(0), lt1 = fmadd(real(0.5), lh1, lod2), lt2 = real(0);
  ao_weights_adj(A, t0, t1, t2, k, lp * A.x01, lq * A.x12, fmadd(lHu, A.u, lHv * A.v), lis,
                 fmadd(lp, A.a0, A.H * (lHu + lHv)), fmadd(lq, A.a2, A.H * (lHu - lHv)), ld1, ld2, lt0, lt1, lt2);
  differences_adj(ld1, ld2, lt0, lt1, lt2, d);
}

// The reverses on the five averages: lQ += (d of the differences), plus the average's own share.
template <class real>
DFW_HD void averages_adj(const real* ld, real lQ2, real* lQ) {
  lQ[0] -= ld[0];
  lQ[1] += ld[0] - ld[1];
  lQ[2] += ld[1] - ld[2] + lQ2;
  lQ[3] += ld[2] - ld[3];
  lQ[4] += ld[3];
}

template <class real>
DFW_HD void average_differences(const real* Q, real* d) {
#pragma unroll
  for (int m = 0; m < 4; ++m) d[m] = Q[m + 1] - Q[m];
}

// Reverse of recon_poly (NDEG coefficients at the edge).
template <class real, int NDEG, int RULE = -1>
DFW_HD void recon_poly_adj(const real* Q, real a_lo, real a_c, real a_hi, const Coef<real>& k, const real* lP, real* lQ,
                           real& la_c) {
  real d[4], dv, sl;
  average_differences(Q, d);
  recon_edge_adj<RULE>(d, a_lo, a_c, a_hi, k, lP[0], NDEG > 1 ? lP[1] : real(0), la_c, dv, sl);
  averages_adj(d, lP[0], lQ);
  if (NDEG > 2) {  // P2 = D2 + 3/2 (D3 + D4), P3 = D3 + 2 D4, P4 = D4
    const real l3 = NDEG > 3 ? lP[3] : real(0), l4 = NDEG > 4 ? lP[4] : real(0);
    const real lD2 = lP[2], lD3 = real(1.5) * lP[2] + l3, lD4 = real(1.5) * lP[2] + real(2) * l3 + l4;
    average_differences(Q, d);
    const real t0 = d[1] - d[0], t1 = d[2] - d[1], t2 = d[3] - d[2];
    real ld1 = real(0), ld2 = real(0), lt0 = real(0), lt1 = real(0), lt2 = real(0);
    if (df_switch<RULE>(a_lo, a_c, a_hi, k)) {
      la_c += real(0.5) * lD2 * t1;
      lt1 = real(0.5) * a_c * lD2;
    } else {
      const AoWeights<real> A =
          ao_weights<true>(d[1], d[2], t0, t1, t2, beta_curv(t0, k), beta_curv(t1, k), beta_curv(t2, k), k);
      const real h = real(0.5) * lD2;  // D2 = (t1 + is y)/2, D3 = -is H u/12, D4 = is H v/24
      const real y = A.a0 * A.x01 - A.a2 * A.x12 - real(0.125) * A.H * A.v;
      const real lHu = real(-1.0 / 12.0) * lD3 * A.is;
      const real lHv = (real(1.0 / 24.0) * lD4 - real(0.125) * h) * A.is;
      const real lis = h * y - real(1.0 / 12.0) * lD3 * A.H * A.u + real(1.0 / 24.0) * lD4 * A.H * A.v;
      lt1 = h;
      ao_weights_adj(A, t0, t1, t2, k, h * A.is * A.x01, -h * A.is * A.x12, lHu * A.u + lHv * A.v, lis,
                     h * A.is * A.a0 + A.H * (lHu + lHv), -h * A.is * A.a2 + A.H * (lHu - lHv), ld1, ld2, lt0, lt1, lt2);
    }
    differences_adj(ld1, ld2, lt0, lt1, lt2, d);
    averages_adj(d, real(0), lQ);
  }
}

// Reverse of recon_gauss: lv, ld (values and slopes at the two Gauss points) -> lQ, la_c; also the
// forward v and dd.
template <class real, int RULE = -1>
DFW_HD void recon_gauss_adj(const real* Q, real a_lo, real a_c, real a_hi, const Coef<real>& k, const real* lv,
                            const real* ld, real* lQ, real& la_c, real* v, real* dd) {
  real d[4], ev, od, evd, odd;
  average_differences(Q, d);
  recon_gauss_parts_adj<RULE>(d, a_lo, a_c, a_hi, k, lv[0] + lv[1], lv[1] - lv[0], ld[0] + ld[1], ld[1] - ld[0], la_c,
                              ev, od, evd, odd);
  averages_adj(d, lv[0] + lv[1], lQ);
  v[0] = Q[2] + (ev - od);
  v[1] = Q[2] + (ev + od);
  dd[0] = evd - odd;
  dd[1] = evd + odd;
}

// ------------------------------------------------------------------------------------------------
// Primitive variables and the DF of one Gauss point.
// ------------------------------------------------------------------------------------------------
template <class real>
struct PrimAdj {
  real r, ir, u, v, p, c;
  DFW_HD void zero() { r = ir = u = v = p = c = real(0); }
};

// With the adjoints of p and 1/rho given (the speed of sound's share already in them).
template <class real>
DFW_HD void prim_adj(const real* w, const Prim<real>& q, const Coef<real>& k, const PrimAdj<real>& lq, real l_p,
                     real l_ir, real* lw) {
  const real hg = real(0.5) * k.gm1 * l_p;
  const real l_u = lq.u - hg * w[1], l_v = lq.v - hg * w[2];
  lw[3] += k.gm1 * l_p;
  lw[1] += l_u * q.ir - hg * q.u;
  lw[2] += l_v * q.ir - hg * q.v;
  l_ir += l_u * w[1] + l_v * w[2];
  lw[0] += lq.r - l_ir * q.ir * q.ir;
}

template <class real>
DFW_HD void prim_adj(const real* w, const Prim<real>& q, const Coef<real>& k, const PrimAdj<real>& lq, real* lw) {
  const real hc = lq.c * k.gamma * real(0.5) * q.ic;
  prim_adj(w, q, k, lq, lq.p + hc * q.ir, lq.ir + hc * q.p, lw);
}

template <class real>
DFW_HD void df_factor_adj(const Prim<real>& L, const Prim<real>& R, real lalpha, PrimAdj<real>& lL, PrimAdj<real>& lR) {
  const real jump = fabs(L.p - R.p);
  const real ipl = rcp_any(L.p), ipr = rcp_any(R.p);
  const real dn = L.u * L.ic - R.u * R.ic;
  const real dt = L.v * L.ic - R.v * R.ic;
  const real D = jump * (ipl + ipr) + dn * dn + dt * dt;
  const real a = rcp_any(real(1) + D * D);
  const real lD = -real(2) * D * (a * a) * lalpha;
  const real sj = signed_by(lD * (ipl + ipr), L.p - R.p), lj = lD * jump;
  lL.p += sj - lj * (ipl * ipl);
  lR.p += -sj - lj * (ipr * ipr);
  const real ldn = real(2) * dn * lD, ldt = real(2) * dt * lD;
  lL.u += ldn * L.ic;
  lR.u -= ldn * R.ic;
  lL.v += ldt * L.ic;
  lR.v -= ldt * R.ic;
  lL.c -= (ldn * L.u + ldt * L.v) * (L.ic * L.ic);
  lR.c += (ldn * R.u + ldt * R.v) * (R.ic * R.ic);
}

// ------------------------------------------------------------------------------------------------
// Lax-Friedrichs flux with the Cauchy-Kovalevskaya time derivative.
// ------------------------------------------------------------------------------------------------
// In the products of the density with the derivatives, as the forward.  lwt: adjoints of W_t, null
// for zero.
template <class real>
DFW_HD void euler_time_derivs_adj(const real* w, const Prim<real>& q, const real* wx, const real* wy,
                                  const Coef<real>& k, const real* lwt, const real* lft, real* lw, PrimAdj<real>& lq,
                                  real* lwx, real* lwy) {
  // forward
  const real u = q.u, v = q.v;
  const real ke = real(0.5) * (u * u + v * v);
  const real ux = wx[1] - u * wx[0], vx = wx[2] - v * wx[0];
  const real uy = wy[1] - u * wy[0], vy = wy[2] - v * wy[0];
  const real px = k.gm1 * (wx[3] - u * wx[1] - v * wx[2] + ke * wx[0]);
  const real py = k.gm1 * (wy[3] - u * wy[1] - v * wy[2] + ke * wy[0]);
  const real rt = -(wx[1] + wy[2]), dv = ux + vy;
  const real Au = fmadd(u, ux, fmadd(v, uy, px)), Av = fmadd(u, vx, fmadd(v, vy, py));
  const real c2 = k.gamma * q.p * q.ir, Ht = (w[3] + q.p) * q.ir;
  const real pt = -fmadd(u, px, fmadd(v, py, c2 * dv));
  const real wt1 = fmadd(rt, u, -Au);
  const real wt3 = fmadd(pt, k.inv_gm1, fmadd(rt, ke, -fmadd(u, Au, v * Av)));
  // reverse: wt_n, ft_n -> rt, Au, Av, pt
  real l1 = lft[0] + u * lft[1] + v * lft[2], l2 = real(0), l3 = u * lft[3], lrt = real(0);
  if (lwt) {
    l1 += lwt[1];
    l2 += lwt[2];
    l3 += lwt[3];
    lrt = lwt[0] + v * l2;
  }
  lrt += u * l1 + ke * l3;
  const real lAu = -(u * lft[1] + Ht * lft[3] + l1 + u * l3), lAv = -(u * lft[2] + l2 + v * l3);
  const real lpt = lft[1] + u * lft[3] + k.inv_gm1 * l3;
  real lu = (wt1 - Au) * lft[1] - Av * lft[2] + (wt3 + pt) * lft[3] + rt * l1 - Au * l3;
  real lv = wt1 * lft[2] + rt * l2 - Av * l3;
  real lke = rt * l3;
  const real lHt = -Au * lft[3], lc2 = -dv * lpt;
  lw[3] += lHt * q.ir;
  lq.p += lHt * q.ir + lc2 * k.gamma * q.ir;
  lq.ir += lHt * (w[3] + q.p) + lc2 * k.gamma * q.p;
  const real ldv = -c2 * lpt;
  const real gpx = k.gm1 * (lAu - u * lpt), gpy = k.gm1 * (lAv - v * lpt);  // gm1 times those of px, py
  const real lux = u * lAu + ldv, luy = v * lAu, lvx = u * lAv, lvy = v * lAv + ldv;
  lu += ux * lAu + vx * lAv - px * lpt - (wx[1] * gpx + wy[1] * gpy) - (wx[0] * lux + wy[0] * luy);
  lv += uy * lAu + vy * lAv - py * lpt - (wx[2] * gpx + wy[2] * gpy) - (wx[0] * lvx + wy[0] * lvy);
  lke += wx[0] * gpx + wy[0] * gpy;
  lwx[0] += ke * gpx - u * lux - v * lvx;
  lwx[1] += lux - u * gpx - lrt;
  lwx[2] += lvx - v * gpx;
  lwx[3] += gpx;
  lwy[0] += ke * gpy - u * luy - v * lvy;
  lwy[1] += luy - u * gpy;
  lwy[2] += lvy - v * gpy - lrt;
  lwy[3] += gpy;
  lq.u += lu + lke * u;
  lq.v += lv + lke * v;
}

// lF: adjoint of the flux, null where the flux itself is not used (the second stage).
template <class real>
DFW_HD void lf_flux_adj(const real* wl, const real* wlx, const real* wly, const real* wr, const real* wrx,
                        const real* wry, const Prim<real>& ql, const Prim<real>& qr, const Coef<real>& k,
                        const real* lF, const real* lFt, real* lwl, real* lwlx, real* lwly, real* lwr, real* lwrx,
                        real* lwry, PrimAdj<real>& lql, PrimAdj<real>& lqr) {
  real sl = fabs(ql.u) + ql.c, sr = fabs(qr.u) + qr.c;
  const bool left = sl >= sr;
  real s = left ? sl : sr;
  real hs = real(0.5) * s;
  real wtl[4], ftl[4], wtr[4], ftr[4];
  euler_time_derivs(wl, ql, wlx, wly, k, wtl, ftl);
  euler_time_derivs(wr, qr, wrx, wry, k, wtr, ftr);
  real lhs = real(0);
  real lwtl[4], lwtr[4], lfth[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    lhs -= lFt[c] * (wtr[c] - wtl[c]);
    lwtr[c] = -hs * lFt[c];
    lwtl[c] = hs * lFt[c];
    lfth[c] = real(0.5) * lFt[c];
  }
  if (lF) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lhs -= lF[c] * (wr[c] - wl[c]);
      lwr[c] -= hs * lF[c];
      lwl[c] += hs * lF[c];
    }
    // F = (w1, w1 u + p, w2 u, u (w3 + p)) on each side
    const real h[4] = {real(0.5) * lF[0], real(0.5) * lF[1], real(0.5) * lF[2], real(0.5) * lF[3]};
    lwl[1] += h[0] + h[1] * ql.u;
    lql.u += h[1] * wl[1] + h[2] * wl[2] + h[3] * (wl[3] + ql.p);
    lql.p += h[1] + h[3] * ql.u;
    lwl[2] += h[2] * ql.u;
    lwl[3] += h[3] * ql.u;
    lwr[1] += h[0] + h[1] * qr.u;
    lqr.u += h[1] * wr[1] + h[2] * wr[2] + h[3] * (wr[3] + qr.p);
    lqr.p += h[1] + h[3] * qr.u;
    lwr[2] += h[2] * qr.u;
    lwr[3] += h[3] * qr.u;
  }
  const real ls = real(0.5) * lhs;
  if (left) {
    lql.u += signed_by(ls, ql.u);
    lql.c += ls;
  } else {
    lqr.u += signed_by(ls, qr.u);
    lqr.c += ls;
  }
  euler_time_derivs_adj(wl, ql, wlx, wly, k, lwtl, lfth, lwl, lql, lwlx, lwly);
  euler_time_derivs_adj(wr, qr, wrx, wry, k, lwtr, lfth, lwr, lqr, lwrx, lwry);
}

// ------------------------------------------------------------------------------------------------
// Gas-kinetic flux.
// ------------------------------------------------------------------------------------------------
// The flux goes through derivatives of moments (gks_side, add_second_moments of dfw_math.hpp); its
// reverse goes back through them.  About 12 000 flops per Gauss point went into the reverse of the
// moments folded with micro-slopes; this one takes about 1 500.
// ------------------------------------------------------------------------------------------------
template <class real>
struct GasAdj {  // adjoints of a Maxwellian's mean U, V, of h = p/rho, X = <v^2 + xi^2> and mu[0..4]
  real U, V, h, X, mu[5];
};

template <class real>
DFW_HD void gas_slope_adj(const real* w, real U, real V, real h, real ke, const GasSlope<real>& l,
                          const Coef<real>& k, real* lw, GasAdj<real>& g, real& lke) {
  const real lP = k.gm1 * l.e;
  lw[0] += l.r - U * l.a - V * l.b - h * l.e + ke * lP;
  lw[1] += l.a - U * lP;
  lw[2] += l.b - V * lP;
  lw[3] += lP;
  g.U -= l.a * w[0] + lP * w[1];
  g.V -= l.b * w[0] + lP * w[2];
  g.h -= l.e * w[0];
  lke += lP * w[0];
}

template <class real>
DFW_HD void slope_d1_adj(const GasSlope<real>& s, const real* mu, real l, GasSlope<real>& ls, GasAdj<real>& g) {
  ls.r += l * mu[1];
  ls.a += l * mu[0];
  g.mu[1] += l * s.r;
  g.mu[0] += l * s.a;
}
template <class real>
DFW_HD void slope_d2_adj(const GasSlope<real>& s, const real* mu, real l, GasSlope<real>& ls, GasAdj<real>& g) {
  const real l2 = real(2) * l;
  ls.r += l * mu[2];
  ls.a += l2 * mu[1];
  ls.e += l * mu[0];
  g.mu[2] += l * s.r;
  g.mu[1] += l2 * s.a;
  g.mu[0] += l * s.e;
}
template <class real>
DFW_HD void slope_d3_adj(const GasSlope<real>& s, const real* mu, real l, GasSlope<real>& ls, GasAdj<real>& g) {
  const real l3 = real(3) * l;
  ls.r += l * mu[3];
  ls.a += l3 * mu[2];
  ls.e += l3 * mu[1];
  g.mu[3] += l * s.r;
  g.mu[2] += l3 * s.a;
  g.mu[1] += l3 * s.e;
}
template <class real>
DFW_HD void slope_d4_adj(const GasSlope<real>& s, const real* mu, real l, GasSlope<real>& ls, GasAdj<real>& g) {
  const real l4 = real(4) * l, l6 = real(6) * l;
  ls.r += l * mu[4];
  ls.a += l4 * mu[3];
  ls.e += l6 * mu[2];
  g.mu[4] += l * s.r;
  g.mu[3] += l4 * s.a;
  g.mu[2] += l6 * s.e;
}

// Reverse of add_second_moments for the adjoint l of M (energy component doubled); the adjoint of d1 is
// added to ld1.
template <class real>
DFW_HD void second_moments_adj(const GasSlope<real>& sx, const GasSlope<real>& sy, const real* mu, real V, real h,
                               real X, real d1, const Coef<real>& k, const real* l, GasSlope<real>& lx,
                               GasSlope<real>& ly, GasAdj<real>& g, real& ld1) {
  const real K1 = k.K + real(1), K3 = k.K + real(3);
  const real d2 = slope_d2(sx, mu), t2 = slope_d2(sy, mu), t3 = slope_d3(sy, mu);
  const real vb = real(2) * V * sy.b, Z = fmadd(real(2), h, X), Vl3 = V * l[3];
  const real mz = fmadd(K3, sy.e, vb);
  slope_d2_adj(sx, mu, fmadd(X, l[3], fmadd(V, l[2], l[0])), lx, g);
  slope_d3_adj(sx, mu, l[1], lx, g);
  slope_d4_adj(sx, mu, l[3], lx, g);
  slope_d2_adj(sy, mu, V * l[1], ly, g);
  slope_d3_adj(sy, mu, Vl3, ly, g);
  ld1 += fmadd(Z, Vl3, fmadd(fmadd(V, V, h), l[2], V * l[0]));
  g.mu[1] += sy.b * l[0] + (vb + sy.e) * l[2] + (V * mz + sy.b * Z) * l[3];
  g.mu[2] += sy.b * l[1] + sx.b * l[2] + fmadd(real(2) * V, sx.b, K1 * sx.e) * l[3];
  g.mu[3] += sy.b * l[3];
  const real lvb = mu[1] * (l[2] + Vl3);
  ly.b += mu[1] * l[0] + mu[2] * l[1] + fmadd(Z, mu[1], mu[3]) * l[3] + real(2) * V * lvb;
  lx.b += mu[2] * fmadd(real(2), Vl3, l[2]);
  lx.e += K1 * mu[2] * l[3];
  ly.e += mu[1] * fmadd(K3, Vl3, l[2]);
  g.V += d1 * l[0] + t2 * l[1] + (d2 + real(2) * V * d1) * l[2] + real(2) * sy.b * lvb +
         (real(2) * sx.b * mu[2] + Z * d1 + mu[1] * mz + t3) * l[3];
  const real lZ = l[3] * fmadd(V, d1, sy.b * mu[1]);
  g.X += fmadd(d2, l[3], lZ);
  g.h += fmadd(d1, l[2], real(2) * lZ);
}

// mu_2..mu_4 by the recursion mu_{n+2} = U mu_{n+1} + (n + 1) h mu_n, reversed into U, h, mu_0, mu_1.
template <class real>
DFW_HD void moments_adj(const real* mu, real U, real h, GasAdj<real>& g) {
  g.U += g.mu[4] * mu[3];
  g.mu[3] += g.mu[4] * U;
  g.h += real(3) * g.mu[4] * mu[2];
  g.mu[2] += real(3) * g.mu[4] * h;
  g.U += g.mu[3] * mu[2];
  g.mu[2] += g.mu[3] * U;
  g.h += real(2) * g.mu[3] * mu[1];
  g.mu[1] += real(2) * g.mu[3] * h;
  g.U += g.mu[2] * mu[1];
  g.mu[1] += g.mu[2] * U;
  g.h += g.mu[2] * mu[0];
  g.mu[0] += g.mu[2] * h;
}

// Adjoint of the GKS flux (lF null where the flux itself is not used), in two halves.  The first
// recomputes the flux and reverses its time coefficients and the equilibrium-state part, down to the
// adjoints of the half-space sums (Wc, Wcn, Wct, Flr, Malr, with doubled energy components) and the
// pressure-jump term of tau; the second reverses the two half-space sides.  A caller short of
// registers can keep the handover in memory between them; gks_flux_adj runs both in turn.
template <class real>
struct GksEqAdj {
  real lWc[4], lWcn[4], lWct[4], lFlr[4], lMalr[4];
  real lpl, lpr;  // the tau term's adjoints of the left and right pressure
};

template <class real>
DFW_HD void gks_flux_adj_eq(const real* wln, const real* wlt, const real* wrn, const real* wrt, const Prim<real>& ql,
                            const Prim<real>& qr, real dt, const Coef<real>& k, const real* lF, const real* lFt,
                            GksEqAdj<real>& e) {
  // ---- forward recompute
  real Wc[4] = {0, 0, 0, 0}, Wcn[4] = {0, 0, 0, 0}, Wct[4] = {0, 0, 0, 0};
  real Flr[4] = {0, 0, 0, 0}, Malr[4] = {0, 0, 0, 0};
  real s2h, is;
  real h = ql.p * ql.ir;
  sqrt_inv(real(2) * h, s2h, is);
  gks_side<1>(ql, h, s2h, is, wln, wlt, k, Wc, Wcn, Wct, Flr, Malr);
  h = qr.p * qr.ir;
  sqrt_inv(real(2) * h, s2h, is);
  gks_side<-1>(qr, h, s2h, is, wrn, wrt, k, Wc, Wcn, Wct, Flr, Malr);
  Wc[3] *= real(0.5);
  Wcn[3] *= real(0.5);
  Wct[3] *= real(0.5);
  Prim<real> c;
  c.r = Wc[0];
  c.ir = rcp_any(Wc[0]);
  c.u = Wc[1] * c.ir;
  c.v = Wc[2] * c.ir;
  c.p = k.gm1 * (Wc[3] - real(0.5) * (Wc[1] * c.u + Wc[2] * c.v));
  h = c.p * c.ir;
  const real U = c.u, V = c.v, K1 = k.K + real(1);
  real mu[5];
  mu[0] = real(1);
  mu[1] = U;
  mu[2] = fmadd(U, U, h);
  mu[3] = fmadd(U, mu[2], real(2) * h * U);
  mu[4] = fmadd(U, mu[3], real(3) * h * mu[2]);
  const real ke = real(0.5) * (U * U + V * V), X = fmadd(V, V, K1 * h);
  const GasSlope<real> sx = gas_slope(Wcn, U, V, h, ke, k), sy = gas_slope(Wct, U, V, h, ke, k);
  const real d1 = slope_d1(sy, mu);
  real Mac[4] = {0, 0, 0, 0};
  add_second_moments(sx, sy, mu, V, h, X, d1, k, Mac);
  const real Fc[4] = {Wc[1], fmadd(Wc[1], U, c.p), Wc[2] * U, U * (Wc[3] + c.p)};
  // ---- time coefficients, forward and reverse
  const real isum = rcp_any(ql.p + qr.p), pq = (ql.p - qr.p) * isum;
  const real x = k.c1 + k.c2 * fabs(pq), ix = rcp_any(x), idt = rcp_any(dt);
  const real E2 = exp(real(-0.5) * ix), om = real(1) - E2, xo = x * om;
  const real ct1 = (real(4) * xo * om) * idt, ct2 = real(4) * xo * (E2 - xo);
  const real z = om * (real(3) - E2), ee = E2 * (E2 - real(2));
  const real cf1 = real(1) - x * z, cf2 = dt * (x * fmadd(x, z, ee));
  real lFc[4], lMac[4];
  real lct1 = real(0), lct2 = real(0), lcf1 = real(0), lcf2 = real(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const real half = i == 3 ? real(0.5) : real(1);
    const real dM = half * (Mac[i] - Malr[i]), dF = Fc[i] - half * Flr[i];
    real ldF = ct1 * lFt[i], ldM = ct2 * lFt[i], lflr = real(0);
    lct1 += lFt[i] * dF;
    lct2 += lFt[i] * dM;
    if (lF) {
      lcf1 += lF[i] * dF;
      lcf2 += lF[i] * dM;
      ldF += cf1 * lF[i];
      ldM += cf2 * lF[i];
      lflr = lF[i];
    }
    lFc[i] = ldF;
    lMac[i] = half * ldM;
    e.lFlr[i] = half * (lflr - ldF);
    e.lMalr[i] = -lMac[i];
  }
  e.lpl = e.lpr = real(0);
  if (x > real(0)) {
    const real dE2 = real(0.5) * E2 * (ix * ix), dxo = om - x * dE2;
    const real dct1 = real(4) * idt * (dxo * om - xo * dE2);
    const real dct2 = real(4) * (dxo * (E2 - xo) + xo * (dE2 - dxo));
    const real dz = (real(2) * E2 - real(4)) * dE2;
    const real dcf1 = -(z + x * dz), dcf2 = dt * (real(2) * x * z + ee + x * (x * dz - real(2) * om * dE2));
    const real lx = lct1 * dct1 + lct2 * dct2 + lcf1 * dcf1 + lcf2 * dcf2;
    const real lpq = signed_by(lx * k.c2, pq) * isum;
    e.lpl = lpq * (real(1) - pq);
    e.lpr = lpq * (real(-1) - pq);
  }
  // ---- equilibrium state: Fc, MA_c and Ma_c -> Wc and its derivatives
#pragma unroll
  for (int i = 0; i < 4; ++i) e.lWc[i] = e.lWcn[i] = e.lWct[i] = real(0);
  PrimAdj<real> lq;
  lq.zero();
  e.lWc[1] += lFc[0] + lFc[1] * U;
  e.lWc[2] += lFc[2] * U;
  e.lWc[3] += lFc[3] * U;
  lq.u += lFc[1] * Wc[1] + lFc[2] * Wc[2] + lFc[3] * (Wc[3] + c.p);
  lq.p += lFc[1] + lFc[3] * U;
  euler_time_derivs_adj(Wc, c, Wcn, Wct, k, (const real*)nullptr, lFt, e.lWc, lq, e.lWcn, e.lWct);
  GasSlope<real> lx{0, 0, 0, 0}, ly{0, 0, 0, 0};
  GasAdj<real> g{};
  real ld1 = real(0), lke = real(0);
  second_moments_adj(sx, sy, mu, V, h, X, d1, k, lMac, lx, ly, g, ld1);
  slope_d1_adj(sy, mu, ld1, ly, g);
  gas_slope_adj(Wcn, U, V, h, ke, lx, k, e.lWcn, g, lke);
  gas_slope_adj(Wct, U, V, h, ke, ly, k, e.lWct, g, lke);
  moments_adj(mu, U, h, g);
  lq.u += g.U + g.mu[1] + lke * U;
  lq.v += g.V + real(2) * V * g.X + lke * V;
  const real lh = fmadd(K1, g.X, g.h);
  prim_adj(Wc, c, k, lq, lq.p + lh * c.ir, lq.ir + lh * c.p, e.lWc);
  e.lWc[3] *= real(0.5);
  e.lWcn[3] *= real(0.5);
  e.lWct[3] *= real(0.5);
}

// Reverse of the first moments of one direction, M = [d0, d1, V d0 + b mu0, X d0 + mu0 (2 V b + K1 e) + D_2] with
// the half-space d0, d1 (boundary term G, zi = U/(2h)), for the adjoint l of M; ld1 adds to d1's.  lG, lzi
// accumulate.
template <class real>
DFW_HD void first_moments_adj(const GasSlope<real>& s, const real* mu, real V, real X, real G, real zi,
                              const Coef<real>& k, const real* l, real ld1, GasSlope<real>& ls, GasAdj<real>& g,
                              real& lG, real& lzi) {
  const real K1 = k.K + real(1);
  const real az = fmadd(-zi, s.e, s.a), d0 = fmadd(s.r, mu[0], G * az);
  const real ld0 = fmadd(X, l[3], fmadd(V, l[2], l[0])), lq = mu[0] * l[3];
  ld1 += l[1];
  g.V += d0 * l[2] + real(2) * s.b * lq;
  g.X += d0 * l[3];
  g.mu[0] += s.b * l[2] + fmadd(real(2) * V, s.b, K1 * s.e) * l[3] + ld0 * s.r;
  ls.b += mu[0] * l[2] + real(2) * V * lq;
  const real lGa = ld0 * G;
  ls.r += ld0 * mu[0];
  ls.a += lGa;
  ls.e += K1 * lq - lGa * zi + real(0.5) * ld1 * G;
  lG += ld0 * az + real(0.5) * ld1 * s.e;
  lzi -= lGa * s.e;
  slope_d1_adj(s, mu, ld1, ls, g);
  slope_d2_adj(s, mu, l[3], ls, g);
}

// One half-space side.
template <int SG, class real>
DFW_HD void gks_side_adj(const Prim<real>& q, const real* wn, const real* wt, const Coef<real>& k,
                         const GksEqAdj<real>& e, real* lwn, real* lwt, PrimAdj<real>& lq) {
  // ---- forward recompute
  const real inv_sqrt_pi = real(SG * 0.56418958354775628695);
  const real U = q.u, V = q.v, h = q.p * q.ir, K1 = k.K + real(1);
  real s2h, is, mu[5];
  sqrt_inv(real(2) * h, s2h, is);
  const real z = is * U, ex = exp(-(z * z));
  mu[0] = real(0.5) * erfc(SG > 0 ? -z : z);
  mu[1] = fmadd(U, mu[0], (real(0.5) * inv_sqrt_pi) * s2h * ex);
  mu[2] = fmadd(U, mu[1], h * mu[0]);
  mu[3] = fmadd(U, mu[2], real(2) * h * mu[1]);
  mu[4] = fmadd(U, mu[3], real(3) * h * mu[2]);
  const real G = inv_sqrt_pi * is * ex, zi = z * is;
  const real ke = real(0.5) * (U * U + V * V), X = fmadd(V, V, K1 * h);
  const GasSlope<real> sx = gas_slope(wn, U, V, h, ke, k), sy = gas_slope(wt, U, V, h, ke, k);
  const real t1 = fmadd(real(0.5) * G, sy.e, slope_d1(sy, mu));
  // ---- reverse
  GasSlope<real> lx{0, 0, 0, 0}, ly{0, 0, 0, 0};
  GasAdj<real> g{};
  real ld1 = real(0), lG = real(0), lzi = real(0), lke = real(0);
  second_moments_adj(sx, sy, mu, V, h, X, t1, k, e.lMalr, lx, ly, g, ld1);
  first_moments_adj(sx, mu, V, X, G, zi, k, e.lWcn, real(0), lx, g, lG, lzi);
  first_moments_adj(sy, mu, V, X, G, zi, k, e.lWct, ld1, ly, g, lG, lzi);
  // Wc = r [mu0, mu1, V mu0, X mu0 + mu2], Flr = r [mu1, mu2, V mu1, X mu1 + mu3]
  const real m0 = fmadd(X, e.lWc[3], fmadd(V, e.lWc[2], e.lWc[0]));
  const real m1 = e.lWc[1] + fmadd(X, e.lFlr[3], fmadd(V, e.lFlr[2], e.lFlr[0]));
  const real m2 = e.lWc[3] + e.lFlr[1], m3 = e.lFlr[3];
  lq.r += m0 * mu[0] + m1 * mu[1] + m2 * mu[2] + m3 * mu[3];
  g.mu[0] += q.r * m0;
  g.mu[1] += q.r * m1;
  g.mu[2] += q.r * m2;
  g.mu[3] += q.r * m3;
  g.V += q.r * (mu[0] * e.lWc[2] + mu[1] * e.lFlr[2]);
  g.X += q.r * (mu[0] * e.lWc[3] + mu[1] * e.lFlr[3]);
  gas_slope_adj(wn, U, V, h, ke, lx, k, lwn, g, lke);
  gas_slope_adj(wt, U, V, h, ke, ly, k, lwt, g, lke);
  moments_adj(mu, U, h, g);
  // d mu0 = G (dU - zi dh), d mu1 = mu0 dU + G/2 dh, dG = G (-2 zi dU + (2 zi^2 - is^2) dh),
  // dzi = is^2 (dU - 2 zi dh)
  const real is2 = is * is, lz = lzi * is2, lg0 = g.mu[0] * G, lGG = lG * G;
  lq.u += g.U + lg0 + g.mu[1] * mu[0] - real(2) * zi * lGG + lz + lke * U;
  lq.v += g.V + real(2) * V * g.X + lke * V;
  const real lh = fmadd(K1, g.X, g.h) - lg0 * zi + real(0.5) * g.mu[1] * G + lGG * (real(2) * zi * zi - is2) -
                  real(2) * zi * lz;
  lq.p += lh * q.ir;
  lq.ir += lh * q.p;
}

template <class real>
DFW_HD void gks_flux_adj_sides(const real* wln, const real* wlt, const real* wrn, const real* wrt,
                               const Prim<real>& ql, const Prim<real>& qr, const Coef<real>& k,
                               const GksEqAdj<real>& e, real* lwln, real* lwlt, real* lwrn, real* lwrt,
                               PrimAdj<real>& lql, PrimAdj<real>& lqr) {
  lql.p += e.lpl;
  lqr.p += e.lpr;
  gks_side_adj<1>(ql, wln, wlt, k, e, lwln, lwlt, lql);
  gks_side_adj<-1>(qr, wrn, wrt, k, e, lwrn, lwrt, lqr);
}

template <class real>
DFW_HD void gks_flux_adj(const real* wl, const real* wln, const real* wlt, const real* wr, const real* wrn,
                         const real* wrt, const Prim<real>& ql, const Prim<real>& qr, real dt, const Coef<real>& k,
                         const real* lF, const real* lFt, real* lwl, real* lwln, real* lwlt, real* lwr, real* lwrn,
                         real* lwrt, PrimAdj<real>& lql, PrimAdj<real>& lqr) {
  GksEqAdj<real> e;
  gks_flux_adj_eq(wln, wlt, wrn, wrt, ql, qr, dt, k, lF, lFt, e);
  gks_flux_adj_sides(wln, wlt, wrn, wrt, ql, qr, k, e, lwln, lwlt, lwrn, lwrt, lql, lqr);
  (void)wl;
  (void)wr;
  (void)lwl;
  (void)lwr;
}

// ------------------------------------------------------------------------------------------------
// One side of the normal sweep and of an interface segment, forward and reverse.
//
// The interface kernels split the work of an interface segment over two threads, one per side:
// side 0 reconstructs cell f-1 (left state), side 1 cell f (right state).  The two sides share the
// characteristic basis of the segment (cells f-1 and f); they meet only in the flux and DF of each
// Gauss point and in the adjoint of the basis.
// ------------------------------------------------------------------------------------------------

// Normal sweep, one side.  cs[0..4]: the side's stencil, ordered away from the interface's far
// side (side 0: cells f-3..f+1; side 1: cells f+2..f-2); (a_lo, a_c, a_hi) the DF of the stencil's
// cells 1..3 in the same order; sgn_inv_dn = +1/dn (side 0) or -1/dn (side 1).  Gives the line
// value w and its normal derivative wn.
template <int RULE = -1, class real>
DFW_HD void normal_side(const Basis<real>& B, const real (*cs)[4], real a_lo, real a_c, real a_hi, real sgn_inv_dn,
                        const Coef<real>& k, real* w, real* wn) {
  real D[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    real x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = cs[m + 1][c] - cs[m][c];
    project(B, x, D[m]);
  }
  real q[4], qd[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const real t0 = D[1][c] - D[0][c], t1 = D[2][c] - D[1][c], t2 = D[3][c] - D[2][c];
    recon_edge<RULE>(D[1][c], D[2][c], t0, t1, t2, beta_curv(t0, k), beta_curv(t1, k), beta_curv(t2, k), a_lo, a_c, a_hi,
                     k, q[c], qd[c]);
    qd[c] *= sgn_inv_dn;
  }
  unproject(B, q, w);
  unproject(B, qd, wn);
#pragma unroll
  for (int c = 0; c < 4; ++c) w[c] += cs[2][c];
}

// One characteristic component C of the reverse: D[m][C] -> its adjoint, in place.
template <int C, int RULE, class real>
DFW_HD void normal_side_adj_comp(const Basis<real>& B, real (*D)[4], real a_lo, real a_c, real a_hi, real sgn_inv_dn,
                                 const Coef<real>& k, const real* lw, const real* lwn, BasisAdj<real>& lB, real& la_c) {
  real d[4] = {D[0][C], D[1][C], D[2][C], D[3][C]}, q, qd;
  recon_edge_adj<RULE>(d, a_lo, a_c, a_hi, k, unproject_adj_q_comp<C>(B, lw), unproject_adj_q_comp<C>(B, lwn) * sgn_inv_dn,
                       la_c, q, qd);
  unproject_adj_B_comp<C>(B, q, lw, lB);
  unproject_adj_B_comp<C>(B, qd * sgn_inv_dn, lwn, lB);
#pragma unroll
  for (int m = 0; m < 4; ++m) D[m][C] = d[m];
}

// Reverse of normal_side; cell(m, c) gives component c of stencil cell m.  The stencil cells'
// adjoints go to lc_add(m, c, v) (add v to cell m, component c); the basis adjoint lB and la_c (the
// DF of the reconstructed cell, DF branch only) accumulate.  One characteristic component at a
// time, its differences replaced by their adjoints; then the projection of each difference is reversed.
template <int RULE = -1, class real, class CellFn, class AddFn>
DFW_HD void normal_side_adj(const Basis<real>& B, CellFn cell, real a_lo, real a_c, real a_hi, real sgn_inv_dn,
                            const Coef<real>& k, const real* lw, const real* lwn, AddFn lc_add, BasisAdj<real>& lB,
                            real& la_c) {
  real D[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    real x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = cell(m + 1, c) - cell(m, c);
    project(B, x, D[m]);
  }
  normal_side_adj_comp<0, RULE>(B, D, a_lo, a_c, a_hi, sgn_inv_dn, k, lw, lwn, lB, la_c);
  normal_side_adj_comp<1, RULE>(B, D, a_lo, a_c, a_hi, sgn_inv_dn, k, lw, lwn, lB, la_c);
  normal_side_adj_comp<2, RULE>(B, D, a_lo, a_c, a_hi, sgn_inv_dn, k, lw, lwn, lB, la_c);
  normal_side_adj_comp<3, RULE>(B, D, a_lo, a_c, a_hi, sgn_inv_dn, k, lw, lwn, lB, la_c);
#pragma unroll
  for (int c = 0; c < 4; ++c) lc_add(2, c, lw[c]);
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    real x[4], d[4] = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = cell(m + 1, c) - cell(m, c);
    project_adj(B, x, D[m], d, lB);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lc_add(m + 1, c, d[c]);
      lc_add(m, c, -d[c]);
    }
  }
}

// Segment, one side: line(m, c) = component c of the side's line value on segment row m-2;
// al = DF of the side's cell on rows -1, 0, +1.  Gives the states and their tangential derivatives
// at the two Gauss points (as segment_states computes them).
template <int RULE = -1, class real, class LineFn>
DFW_HD void segment_side(const Basis<real>& B, LineFn line, const real* al, real inv_dt, const Coef<real>& k,
                         real (*gw)[4], real (*gwt)[4]) {
  real D[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    real x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = line(m + 1, c) - line(m, c);
    project(B, x, D[m]);
  }
  real ev[4], od[4], evd[4], odd[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    recon_gauss_parts<RULE>(D[0][c], D[1][c], D[2][c], D[3][c], al[0], al[1], al[2], k, ev[c], od[c], evd[c], odd[c]);
    evd[c] *= inv_dt;
    odd[c] *= inv_dt;
  }
  real e[4], o[4];
  unproject(B, ev, e);
  unproject(B, od, o);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const real m = line(2, c) + e[c];
    gw[0][c] = m - o[c];
    gw[1][c] = m + o[c];
  }
  unproject(B, evd, e);
  unproject(B, odd, o);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    gwt[0][c] = e[c] - o[c];
    gwt[1][c] = e[c] + o[c];
  }
}

// One characteristic component C of the reverse of segment_side: D[m][C] -> its adjoint, in place.
// se, so: even and odd sums (point 0 + point 1, point 1 - point 0) of the adjoints of the Gauss-point
// states, te, to those of their tangential derivatives.
template <int C, int RULE, class real>
DFW_HD void segment_side_adj_comp(const Basis<real>& B, real (*D)[4], const real* al, real inv_dt,
                                  const Coef<real>& k, const real* se, const real* so, const real* te, const real* to,
                                  BasisAdj<real>& lB, real& la_c) {
  real d[4] = {D[0][C], D[1][C], D[2][C], D[3][C]}, ev, od, evd, odd;
  recon_gauss_parts_adj<RULE>(d, al[0], al[1], al[2], k, unproject_adj_q_comp<C>(B, se), unproject_adj_q_comp<C>(B, so),
                              unproject_adj_q_comp<C>(B, te) * inv_dt, unproject_adj_q_comp<C>(B, to) * inv_dt, la_c, ev,
                              od, evd, odd);
  unproject_adj_B_comp<C>(B, ev, se, lB);
  unproject_adj_B_comp<C>(B, od, so, lB);
  unproject_adj_B_comp<C>(B, evd * inv_dt, te, lB);
  unproject_adj_B_comp<C>(B, odd * inv_dt, to, lB);
#pragma unroll
  for (int m = 0; m < 4; ++m) D[m][C] = d[m];
}

// Reverse of segment_side for the adjoints lgw, lgwt of the Gauss-point states: the adjoints of the
// side's line values go to ll_put(m, v) (row m, all four components, each row once); lB and la_c
// accumulate.
template <int RULE = -1, class real, class LineFn, class PutFn>
DFW_HD void segment_side_adj_rows(const Basis<real>& B, LineFn line, const real* al, real inv_dt, const Coef<real>& k,
                                  const real (*lgw)[4], const real (*lgwt)[4], PutFn ll_put, BasisAdj<real>& lB,
                                  real& la_c) {
  real se[4], so[4], te[4], to[4], D[4][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    se[c] = lgw[0][c] + lgw[1][c];
    so[c] = lgw[1][c] - lgw[0][c];
    te[c] = lgwt[0][c] + lgwt[1][c];
    to[c] = lgwt[1][c] - lgwt[0][c];
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    real x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = line(m + 1, c) - line(m, c);
    project(B, x, D[m]);
  }
  segment_side_adj_comp<0, RULE>(B, D, al, inv_dt, k, se, so, te, to, lB, la_c);
  segment_side_adj_comp<1, RULE>(B, D, al, inv_dt, k, se, so, te, to, lB, la_c);
  segment_side_adj_comp<2, RULE>(B, D, al, inv_dt, k, se, so, te, to, lB, la_c);
  segment_side_adj_comp<3, RULE>(B, D, al, inv_dt, k, se, so, te, to, lB, la_c);
  real prev[4] = {0, 0, 0, 0};  // adjoint of the difference below the row
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    real d[4] = {0, 0, 0, 0}, v[4];
    if (m < 4) {
      real x[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) x[c] = line(m + 1, c) - line(m, c);
      project_adj(B, x, D[m], d, lB);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      v[c] = prev[c] - d[c] + (m == 2 ? se[c] : real(0));
      prev[c] = d[c];
    }
    ll_put(m, v);
  }
}

// The same with each component added by ll_add(m, c, v).
template <int RULE = -1, class real, class LineFn, class AddFn>
DFW_HD void segment_side_adj(const Basis<real>& B, LineFn line, const real* al, real inv_dt, const Coef<real>& k,
                             const real (*lgw)[4], const real (*lgwt)[4], AddFn ll_add, BasisAdj<real>& lB,
                             real& la_c) {
  segment_side_adj_rows<RULE>(B, line, al, inv_dt, k, lgw, lgwt,
                              [&](int m, const real* v) {
#pragma unroll
                                for (int c = 0; c < 4; ++c) ll_add(m, c, v[c]);
                              },
                              lB, la_c);
}

// Reverse of the flux, its time derivative and the DF at one Gauss point (left state wl with normal
// and tangential derivatives wln, wlt; right state likewise): lF, lFt are the adjoints of the
// Gauss point's flux and time derivative, ldf that of its DF value.  Outputs accumulate.
template <class real, int FLUX>
DFW_HD void gp_flux_adj(const real* wl, const real* wln, const real* wlt, const real* wr, const real* wrn,
                        const real* wrt, real dt, const Coef<real>& k, const real* lF, const real* lFt, real ldf,
                        real* lwl, real* lwln, real* lwlt, real* lwr, real* lwrn, real* lwrt) {
  const Prim<real> ql = prim(wl, k), qr = prim(wr, k);
  PrimAdj<real> lql, lqr;
  lql.zero();
  lqr.zero();
  if (FLUX == 0)
    lf_flux_adj(wl, wln, wlt, wr, wrn, wrt, ql, qr, k, lF, lFt, lwl, lwln, lwlt, lwr, lwrn, lwrt, lql, lqr);
  else
    gks_flux_adj(wl, wln, wlt, wr, wrn, wrt, ql, qr, dt, k, lF, lFt, lwl, lwln, lwlt, lwr, lwrn, lwrt, lql, lqr);
  df_factor_adj(ql, qr, ldf, lql, lqr);
  prim_adj(wl, ql, k, lql, lwl);
  prim_adj(wr, qr, k, lqr, lwr);
}

}  // namespace dfw
