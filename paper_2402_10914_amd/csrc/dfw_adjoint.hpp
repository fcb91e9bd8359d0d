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

template <class real>
DFW_HD void prim_adj(const real* w, const Prim<real>& q, const Coef<real>& k, const PrimAdj<real>& lq, real* lw) {
  real l_p = lq.p + lq.c * k.gamma * q.ir * real(0.5) / q.c;
  real l_ir = lq.ir + lq.c * k.gamma * q.p * real(0.5) / q.c;
  real l_u = lq.u - real(0.5) * k.gm1 * w[1] * l_p;
  real l_v = lq.v - real(0.5) * k.gm1 * w[2] * l_p;
  lw[3] += k.gm1 * l_p;
  lw[1] += -real(0.5) * k.gm1 * q.u * l_p + l_u * q.ir;
  lw[2] += -real(0.5) * k.gm1 * q.v * l_p + l_v * q.ir;
  l_ir += l_u * w[1] + l_v * w[2];
  lw[0] += lq.r - l_ir * q.ir * q.ir;
}

template <class real>
DFW_HD void df_factor_adj(const Prim<real>& L, const Prim<real>& R, real lalpha, PrimAdj<real>& lL, PrimAdj<real>& lR) {
  real jump = fabs(L.p - R.p);
  real icl = real(1) / L.c, icr = real(1) / R.c;
  real dn = L.u * icl - R.u * icr;
  real dt = L.v * icl - R.v * icr;
  real D = jump * (real(1) / L.p + real(1) / R.p) + dn * dn + dt * dt;
  real a = real(1) / (real(1) + D * D);
  real lD = -real(2) * D * a * a * lalpha;
  real ljump = lD * (real(1) / L.p + real(1) / R.p);
  lL.p += -lD * jump / (L.p * L.p);
  lR.p += -lD * jump / (R.p * R.p);
  real s = sgn(L.p - R.p);
  lL.p += s * ljump;
  lR.p -= s * ljump;
  real ldn = real(2) * dn * lD, ldt = real(2) * dt * lD;
  lL.u += ldn * icl;
  lR.u -= ldn * icr;
  lL.v += ldt * icl;
  lR.v -= ldt * icr;
  real licl = ldn * L.u + ldt * L.v;
  real licr = -(ldn * R.u + ldt * R.v);
  lL.c += -licl * icl * icl;
  lR.c += -licr * icr * icr;
}

// ------------------------------------------------------------------------------------------------
// Lax-Friedrichs flux with the Cauchy-Kovalevskaya time derivative.
// ------------------------------------------------------------------------------------------------
template <class real>
DFW_HD void euler_time_derivs_adj(const real* w, const Prim<real>& q, const real* wx, const real* wy,
                                  const Coef<real>& k, const real* lwt_in, const real* lft, real* lw, PrimAdj<real>& lq,
                                  real* lwx, real* lwy) {
  // forward
  real ke = real(0.5) * (q.u * q.u + q.v * q.v);
  real ux = (wx[1] - q.u * wx[0]) * q.ir, vx = (wx[2] - q.v * wx[0]) * q.ir;
  real px = k.gm1 * (wx[3] - q.u * wx[1] - q.v * wx[2] + ke * wx[0]);
  real uy = (wy[1] - q.u * wy[0]) * q.ir, vy = (wy[2] - q.v * wy[0]) * q.ir;
  real py = k.gm1 * (wy[3] - q.u * wy[1] - q.v * wy[2] + ke * wy[0]);
  real rt = -(q.u * wx[0] + q.r * ux + q.v * wy[0] + q.r * vy);
  real ut = -(q.u * ux + q.v * uy + px * q.ir);
  real vt = -(q.u * vx + q.v * vy + py * q.ir);
  real pt = -(q.u * px + q.v * py + k.gamma * q.p * (ux + vy));
  real wt1 = rt * q.u + q.r * ut;
  real wt3 = pt * k.inv_gm1 + rt * ke + q.r * (q.u * ut + q.v * vt);
  // reverse
  real lwt[4] = {lwt_in[0], lwt_in[1], lwt_in[2], lwt_in[3]};
  real lut = real(0), lvt = real(0), lpt = real(0), lrt = real(0), lke = real(0);
  // ft3 = ut (w3 + p) + u (wt3 + pt)
  lut += lft[3] * (w[3] + q.p);
  lw[3] += lft[3] * ut;
  lq.p += lft[3] * ut;
  lq.u += lft[3] * (wt3 + pt);
  lwt[3] += lft[3] * q.u;
  lpt += lft[3] * q.u;
  // ft2 = wt1 v + w1 vt
  lwt[1] += lft[2] * q.v;
  lq.v += lft[2] * wt1;
  lw[1] += lft[2] * vt;
  lvt += lft[2] * w[1];
  // ft1 = wt1 u + w1 ut + pt
  lwt[1] += lft[1] * q.u;
  lq.u += lft[1] * wt1;
  lw[1] += lft[1] * ut;
  lut += lft[1] * w[1];
  lpt += lft[1];
  // ft0 = wt1
  lwt[1] += lft[0];
  // wt3 = pt/gm1 + rt ke + r (u ut + v vt)
  lpt += lwt[3] * k.inv_gm1;
  lrt += lwt[3] * ke;
  lke += lwt[3] * rt;
  lq.r += lwt[3] * (q.u * ut + q.v * vt);
  lq.u += lwt[3] * q.r * ut;
  lut += lwt[3] * q.r * q.u;
  lq.v += lwt[3] * q.r * vt;
  lvt += lwt[3] * q.r * q.v;
  // wt2 = rt v + r vt
  lrt += lwt[2] * q.v;
  lq.v += lwt[2] * rt;
  lq.r += lwt[2] * vt;
  lvt += lwt[2] * q.r;
  // wt1 = rt u + r ut
  lrt += lwt[1] * q.u;
  lq.u += lwt[1] * rt;
  lq.r += lwt[1] * ut;
  lut += lwt[1] * q.r;
  // wt0 = rt
  lrt += lwt[0];
  // pt = -(u px + v py + gamma p (ux + vy))
  real lux = -lpt * k.gamma * q.p, lvy = -lpt * k.gamma * q.p;
  real lpx = -lpt * q.u, lpy = -lpt * q.v;
  lq.u += -lpt * px;
  lq.v += -lpt * py;
  lq.p += -lpt * k.gamma * (ux + vy);
  // vt = -(u vx + v vy + py ir)
  lq.u -= lvt * vx;
  real lvx = -lvt * q.u;
  lq.v -= lvt * vy;
  lvy -= lvt * q.v;
  lpy -= lvt * q.ir;
  lq.ir -= lvt * py;
  // ut = -(u ux + v uy + px ir)
  lq.u -= lut * ux;
  lux -= lut * q.u;
  lq.v -= lut * uy;
  real luy = -lut * q.v;
  lpx -= lut * q.ir;
  lq.ir -= lut * px;
  // rt = -(u wx0 + r ux + v wy0 + r vy)
  lq.u -= lrt * wx[0];
  lwx[0] -= lrt * q.u;
  lq.r -= lrt * (ux + vy);
  lux -= lrt * q.r;
  lq.v -= lrt * wy[0];
  lwy[0] -= lrt * q.v;
  lvy -= lrt * q.r;
  // py, px
  lwy[3] += k.gm1 * lpy;
  lq.u -= k.gm1 * lpy * wy[1];
  lwy[1] -= k.gm1 * lpy * q.u;
  lq.v -= k.gm1 * lpy * wy[2];
  lwy[2] -= k.gm1 * lpy * q.v;
  lke += k.gm1 * lpy * wy[0];
  lwy[0] += k.gm1 * lpy * ke;
  lwx[3] += k.gm1 * lpx;
  lq.u -= k.gm1 * lpx * wx[1];
  lwx[1] -= k.gm1 * lpx * q.u;
  lq.v -= k.gm1 * lpx * wx[2];
  lwx[2] -= k.gm1 * lpx * q.v;
  lke += k.gm1 * lpx * wx[0];
  lwx[0] += k.gm1 * lpx * ke;
  // vy, uy, vx, ux
  lwy[2] += lvy * q.ir;
  lq.v -= lvy * wy[0] * q.ir;
  lwy[0] -= lvy * q.v * q.ir;
  lq.ir += lvy * (wy[2] - q.v * wy[0]);
  lwy[1] += luy * q.ir;
  lq.u -= luy * wy[0] * q.ir;
  lwy[0] -= luy * q.u * q.ir;
  lq.ir += luy * (wy[1] - q.u * wy[0]);
  lwx[2] += lvx * q.ir;
  lq.v -= lvx * wx[0] * q.ir;
  lwx[0] -= lvx * q.v * q.ir;
  lq.ir += lvx * (wx[2] - q.v * wx[0]);
  lwx[1] += lux * q.ir;
  lq.u -= lux * wx[0] * q.ir;
  lwx[0] -= lux * q.u * q.ir;
  lq.ir += lux * (wx[1] - q.u * wx[0]);
  // ke
  lq.u += lke * q.u;
  lq.v += lke * q.v;
}

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
  real lwtl[4], lwtr[4], lftl[4], lftr[4];
  real lFl[4], lFr[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    lhs -= lF[c] * (wr[c] - wl[c]) + lFt[c] * (wtr[c] - wtl[c]);
    lwr[c] -= hs * lF[c];
    lwl[c] += hs * lF[c];
    lFl[c] = real(0.5) * lF[c];
    lFr[c] = real(0.5) * lF[c];
    lwtr[c] = -hs * lFt[c];
    lwtl[c] = hs * lFt[c];
    lftl[c] = real(0.5) * lFt[c];
    lftr[c] = real(0.5) * lFt[c];
  }
  real ls = real(0.5) * lhs;
  if (left) {
    lql.u += sgn(ql.u) * ls;
    lql.c += ls;
  } else {
    lqr.u += sgn(qr.u) * ls;
    lqr.c += ls;
  }
  // F = (w1, w1 u + p, w2 u, u (w3 + p)) on each side
  lwl[1] += lFl[0] + lFl[1] * ql.u;
  lql.u += lFl[1] * wl[1] + lFl[2] * wl[2] + lFl[3] * (wl[3] + ql.p);
  lql.p += lFl[1] + lFl[3] * ql.u;
  lwl[2] += lFl[2] * ql.u;
  lwl[3] += lFl[3] * ql.u;
  lwr[1] += lFr[0] + lFr[1] * qr.u;
  lqr.u += lFr[1] * wr[1] + lFr[2] * wr[2] + lFr[3] * (wr[3] + qr.p);
  lqr.p += lFr[1] + lFr[3] * qr.u;
  lwr[2] += lFr[2] * qr.u;
  lwr[3] += lFr[3] * qr.u;
  euler_time_derivs_adj(wl, ql, wlx, wly, k, lwtl, lftl, lwl, lql, lwlx, lwly);
  euler_time_derivs_adj(wr, qr, wrx, wry, k, lwtr, lftr, lwr, lqr, lwrx, lwry);
}

// ------------------------------------------------------------------------------------------------
// Gas-kinetic flux.
// ------------------------------------------------------------------------------------------------
template <class real>
struct MomAdj {
  real mu[7], mv[6], mx[3];
  DFW_HD void zero() {
#pragma unroll
    for (int i = 0; i < 7; ++i) mu[i] = real(0);
#pragma unroll
    for (int i = 0; i < 6; ++i) mv[i] = real(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) mx[i] = real(0);
  }
};

template <class real>
DFW_HD void mom_adj(const Mom<real>& M, int a, int b, int c, real l, MomAdj<real>& lM) {
  lM.mu[a] += l * M.mv[b] * M.mx[c];
  lM.mv[b] += l * M.mu[a] * M.mx[c];
  lM.mx[c] += l * M.mu[a] * M.mv[b];
}

// <(s.psi) u^a v^b xi^2c>: adjoint into the slope and the moments
template <class real>
DFW_HD void mom_s_adj(const Mom<real>& M, const real* s, int a, int b, int c, real l, real* ls, MomAdj<real>& lM) {
  ls[0] += l * mom(M, a, b, c);
  ls[1] += l * mom(M, a + 1, b, c);
  ls[2] += l * mom(M, a, b + 1, c);
  ls[3] += l * real(0.5) * (mom(M, a + 2, b, c) + mom(M, a, b + 2, c) + mom(M, a, b, c + 1));
  mom_adj(M, a, b, c, l * s[0], lM);
  mom_adj(M, a + 1, b, c, l * s[1], lM);
  mom_adj(M, a, b + 1, c, l * s[2], lM);
  const real h3 = real(0.5) * s[3] * l;
  mom_adj(M, a + 2, b, c, h3, lM);
  mom_adj(M, a, b + 2, c, h3, lM);
  mom_adj(M, a, b, c + 1, h3, lM);
}

template <class real>
DFW_HD void mom_s_psi_adj(const Mom<real>& M, const real* s, int a, int b, const real* l, real* ls, MomAdj<real>& lM) {
  mom_s_adj(M, s, a, b, 0, l[0], ls, lM);
  mom_s_adj(M, s, a + 1, b, 0, l[1], ls, lM);
  mom_s_adj(M, s, a, b + 1, 0, l[2], ls, lM);
  const real h = real(0.5) * l[3];
  mom_s_adj(M, s, a + 2, b, 0, h, ls, lM);
  mom_s_adj(M, s, a, b + 2, 0, h, ls, lM);
  mom_s_adj(M, s, a, b, 1, h, ls, lM);
}

template <class real>
DFW_HD void mom_psi_adj(const Mom<real>& M, int a, int b, const real* l, MomAdj<real>& lM) {
  mom_adj(M, a, b, 0, l[0], lM);
  mom_adj(M, a + 1, b, 0, l[1], lM);
  mom_adj(M, a, b + 1, 0, l[2], lM);
  const real h = real(0.5) * l[3];
  mom_adj(M, a + 2, b, 0, h, lM);
  mom_adj(M, a, b + 2, 0, h, lM);
  mom_adj(M, a, b, 1, h, lM);
}

// Reverse of maxwell_moments: -> adjoints of U, V, lambda.
template <class real>
DFW_HD void maxwell_moments_adj(const Mom<real>& M, int side, const Coef<real>& k, MomAdj<real> lM, real& lU, real& lV,
                                real& llam) {
  const real U = M.U, V = M.V, lam = M.lam;
  const real h = real(0.5) / lam;
  real lh = lM.mx[1] * k.K + lM.mx[2] * real(2) * k.K * (k.K + real(2)) * h;
#pragma unroll
  for (int n = 3; n >= 0; --n) {  // mv[n+2] = V mv[n+1] + (n+1) h mv[n]
    const real l = lM.mv[n + 2];
    lV += l * M.mv[n + 1];
    lM.mv[n + 1] += l * V;
    lh += l * real(n + 1) * M.mv[n];
    lM.mv[n] += l * real(n + 1) * h;
  }
  lV += lM.mv[1];
#pragma unroll
  for (int n = 4; n >= 0; --n) {
    const real l = lM.mu[n + 2];
    lU += l * M.mu[n + 1];
    lM.mu[n + 1] += l * U;
    lh += l * real(n + 1) * M.mu[n];
    lM.mu[n] += l * real(n + 1) * h;
  }
  if (side == 0) {
    lU += lM.mu[1];
  } else {
    const real inv_sqrt_pi = real(0.56418958354775628695);
    const real sg = side > 0 ? real(1) : real(-1);
    real sl = sqrt(lam);
    real ex = exp(-lam * U * U);
    real g = real(0.5) * ex * inv_sqrt_pi / sl;
    // mu1 = U mu0 +- g
    lU += lM.mu[1] * M.mu[0];
    real lmu0 = lM.mu[0] + lM.mu[1] * U;
    real lg = sg * lM.mu[1];
    // mu0 = erfc(-sg sl U)/2: d/dz erfc(z)/2 = -exp(-z^2)/sqrt(pi), z = -sg sl U
    real dmu0 = -inv_sqrt_pi * ex;
    lU += lmu0 * dmu0 * (-sg * sl);
    real lsl = lmu0 * dmu0 * (-sg * U);
    // g = exp(-lam U^2) / (2 sqrt(pi) sl)
    lU += lg * g * (real(-2) * lam * U);
    llam += lg * g * (-U * U);
    lsl += -lg * g / sl;
    llam += lsl * real(0.5) / sl;
  }
  llam += -lh * real(0.5) / (lam * lam);
}

template <class real>
DFW_HD void micro_slope_adj(const real* g, real U, real V, real lam, const Coef<real>& k, const real* ls_in, real* lg,
                            real& lU, real& lV, real& llam) {
  const real K2 = k.K2;
  const real ilam = real(1) / lam;
  real B = U * U + V * V + K2 * real(0.5) * ilam;
  real R4 = real(2) * g[3] - B * g[0];
  real R3 = g[2] - V * g[0];
  real R2 = g[1] - U * g[0];
  real kap = k.k4K2 * (lam * lam);
  real Z = R4 - real(2) * U * R2 - real(2) * V * R3;
  real s3 = kap * Z;
  real s2 = real(2) * lam * R3 - V * s3;
  real s1 = real(2) * lam * R2 - U * s3;
  // s0 = g0 - U s1 - V s2 - s3 B / 2
  real ls1 = ls_in[1] - U * ls_in[0];
  real ls2 = ls_in[2] - V * ls_in[0];
  real ls3 = ls_in[3] - real(0.5) * B * ls_in[0];
  lg[0] += ls_in[0];
  lU -= ls_in[0] * s1;
  lV -= ls_in[0] * s2;
  real lB = -real(0.5) * s3 * ls_in[0];
  // s1 = 2 lam R2 - U s3 ; s2 = 2 lam R3 - V s3
  llam += real(2) * R2 * ls1 + real(2) * R3 * ls2;
  real lR2 = real(2) * lam * ls1, lR3 = real(2) * lam * ls2;
  lU -= s3 * ls1;
  lV -= s3 * ls2;
  ls3 -= U * ls1 + V * ls2;
  // s3 = kap Z
  llam += ls3 * Z * real(2) * lam * k.k4K2;
  real lZ = ls3 * kap;
  real lR4 = lZ;
  lU -= real(2) * R2 * lZ;
  lR2 -= real(2) * U * lZ;
  lV -= real(2) * R3 * lZ;
  lR3 -= real(2) * V * lZ;
  lg[1] += lR2;
  lU -= g[0] * lR2;
  lg[0] -= U * lR2;
  lg[2] += lR3;
  lV -= g[0] * lR3;
  lg[0] -= V * lR3;
  lg[3] += real(2) * lR4;
  lB -= g[0] * lR4;
  lg[0] -= B * lR4;
  lU += real(2) * U * lB;
  lV += real(2) * V * lB;
  llam += -K2 * real(0.5) * (ilam * ilam) * lB;
}

// Adjoint of gks_flux (lF may be null when the flux itself was not requested), in two halves.  The first recomputes the flux and reverses its time
// coefficients and the equilibrium-state part, down to the adjoints of the half-space sums
// (Wc, Wcn, Wct, Flr, Malr) and the pressure-jump term of tau; the second reverses the two
// half-space sides.  A caller short of registers can keep the handover in memory between them;
// gks_flux_adj runs both in turn.
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
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const real* wn = side == 0 ? wln : wrn;
    const real* wt = side == 0 ? wlt : wrt;
    const Prim<real>& q = side == 0 ? ql : qr;
    real lam = real(0.5) * q.r / q.p;
    Mom<real> M;
    maxwell_moments(q.u, q.v, lam, side == 0 ? 1 : -1, k, M);
    real g[4], a[4], b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) g[c] = wn[c] * q.ir;
    micro_slope(g, q.u, q.v, lam, real(0.5) / lam, k, a);
#pragma unroll
    for (int c = 0; c < 4; ++c) g[c] = wt[c] * q.ir;
    micro_slope(g, q.u, q.v, lam, real(0.5) / lam, k, b);
    real t0[4], t1[4], t2[4];
    mom_psi(M, 0, 0, t0);
    mom_s_psi(M, a, 0, 0, t1);
    mom_s_psi(M, b, 0, 0, t2);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      Wc[c] += q.r * t0[c];
      Wcn[c] += q.r * t1[c];
      Wct[c] += q.r * t2[c];
    }
    mom_psi(M, 1, 0, t0);
    mom_s_psi(M, a, 2, 0, t1);
    mom_s_psi(M, b, 1, 1, t2);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      Flr[c] += q.r * t0[c];
      Malr[c] += q.r * (t1[c] + t2[c]);
    }
  }
  real irc = real(1) / Wc[0];
  real Uc = Wc[1] * irc, Vc = Wc[2] * irc;
  real pc = k.gm1 * (Wc[3] - real(0.5) * (Wc[1] * Uc + Wc[2] * Vc));
  real lamc = real(0.5) * Wc[0] / pc;
  Mom<real> Mc;
  maxwell_moments(Uc, Vc, lamc, 0, k, Mc);
  real gn[4], gt[4], ac[4], bc[4], Ac[4], gA[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    gn[c] = Wcn[c] * irc;
    gt[c] = Wct[c] * irc;
  }
  micro_slope(gn, Uc, Vc, lamc, real(0.5) / lamc, k, ac);
  micro_slope(gt, Uc, Vc, lamc, real(0.5) / lamc, k, bc);
  real y1[4], y2[4];
  mom_s_psi(Mc, ac, 1, 0, y1);
  mom_s_psi(Mc, bc, 0, 1, y2);
#pragma unroll
  for (int c = 0; c < 4; ++c) gA[c] = -(y1[c] + y2[c]);
  micro_slope(gA, Uc, Vc, lamc, real(0.5) / lamc, k, Ac);
  real fc[4], x1[4], x2[4], xA[4];
  mom_psi(Mc, 1, 0, fc);
  mom_s_psi(Mc, ac, 2, 0, x1);
  mom_s_psi(Mc, bc, 1, 1, x2);
  mom_s_psi(Mc, Ac, 1, 0, xA);
  real Fc[4], Mac[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    Fc[c] = Wc[0] * fc[c];
    Mac[c] = Wc[0] * (x1[c] + x2[c]);
  }
  const real pq = (ql.p - qr.p) / (ql.p + qr.p);
  real tau = k.c1 * dt + k.c2 * fabs(pq) * dt;
  real E2 = exp(-real(0.5) * dt / tau);
  real E1 = E2 * E2;
  real om = real(1) - E2;
  real idt = real(1) / dt;
  real ct1 = real(4) * tau * om * om * idt * idt;
  real ct2 = real(4) * (tau * dt * E2 * om - tau * tau * om * om) * idt * idt;
  real z = real(3) - real(4) * E2 + E1;
  real cf1 = real(1) - tau * idt * z;
  real cf2 = tau * tau * idt * z + tau * (E1 - real(2) * E2);
  // ---- reverse: time coefficients
  real lFc[4], lMac[4], lMAc[4];
  real* lFlr = e.lFlr;
  real* lMalr = e.lMalr;
  e.lpl = e.lpr = real(0);
  real lct1 = real(0), lct2 = real(0), lcf1 = real(0), lcf2 = real(0);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const real MA = Wc[0] * xA[c];
    (void)MA;
    lct1 += lFt[c] * (Fc[c] - Flr[c]);
    lct2 += lFt[c] * (Mac[c] - Malr[c]);
    lFc[c] = ct1 * lFt[c];
    lFlr[c] = -ct1 * lFt[c];
    lMac[c] = ct2 * lFt[c];
    lMalr[c] = -ct2 * lFt[c];
    lMAc[c] = lFt[c];
    if (lF) {
      lcf1 += lF[c] * (Fc[c] - Flr[c]);
      lcf2 += lF[c] * (Mac[c] - Malr[c]);
      lFc[c] += cf1 * lF[c];
      lFlr[c] += (real(1) - cf1) * lF[c];
      lMac[c] += cf2 * lF[c];
      lMalr[c] -= cf2 * lF[c];
    }
  }
  if (tau > real(0)) {
    real dE2 = E2 * real(0.5) * dt / (tau * tau);
    real dct1 = real(4) * idt * idt * (om * om - real(2) * tau * om * dE2);
    real dct2 = real(4) * idt * idt *
                (dt * E2 * om + tau * dt * (dE2 * om - E2 * dE2) - real(2) * tau * om * om + real(2) * tau * tau * om * dE2);
    real dz = (real(-4) + real(2) * E2) * dE2;
    real dcf1 = -idt * (z + tau * dz);
    real dcf2 = real(2) * tau * idt * z + tau * tau * idt * dz + (E1 - real(2) * E2) + tau * (real(2) * E2 - real(2)) * dE2;
    real ltau = lct1 * dct1 + lct2 * dct2 + lcf1 * dcf1 + lcf2 * dcf2;
    real lpq = ltau * k.c2 * dt * sgn(pq);
    real isum = real(1) / (ql.p + qr.p);
    e.lpl = lpq * (real(1) - pq) * isum;
    e.lpr = lpq * (real(-1) - pq) * isum;
  }
  // ---- reverse: equilibrium-state fluxes
  MomAdj<real> lMc;
  lMc.zero();
  real* lWc = e.lWc;
  real* lWcn = e.lWcn;
  real* lWct = e.lWct;
#pragma unroll
  for (int c = 0; c < 4; ++c) lWc[c] = lWcn[c] = lWct[c] = real(0);
  real lac[4] = {0, 0, 0, 0}, lbc[4] = {0, 0, 0, 0}, lAc[4] = {0, 0, 0, 0};
  real lx[4], lfc[4], lxA[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    lWc[0] += lFc[c] * fc[c] + lMac[c] * (x1[c] + x2[c]) + lMAc[c] * xA[c];
    lfc[c] = Wc[0] * lFc[c];
    lx[c] = Wc[0] * lMac[c];
    lxA[c] = Wc[0] * lMAc[c];
  }
  mom_psi_adj(Mc, 1, 0, lfc, lMc);
  mom_s_psi_adj(Mc, ac, 2, 0, lx, lac, lMc);
  mom_s_psi_adj(Mc, bc, 1, 1, lx, lbc, lMc);
  mom_s_psi_adj(Mc, Ac, 1, 0, lxA, lAc, lMc);
  real lUc = real(0), lVc = real(0), llamc = real(0);
  real lgA[4] = {0, 0, 0, 0};
  micro_slope_adj(gA, Uc, Vc, lamc, k, lAc, lgA, lUc, lVc, llamc);
  real ly[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) ly[c] = -lgA[c];
  mom_s_psi_adj(Mc, ac, 1, 0, ly, lac, lMc);
  mom_s_psi_adj(Mc, bc, 0, 1, ly, lbc, lMc);
  real lgn[4] = {0, 0, 0, 0}, lgt[4] = {0, 0, 0, 0};
  micro_slope_adj(gn, Uc, Vc, lamc, k, lac, lgn, lUc, lVc, llamc);
  micro_slope_adj(gt, Uc, Vc, lamc, k, lbc, lgt, lUc, lVc, llamc);
  real lirc = real(0);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    lWcn[c] += lgn[c] * irc;
    lWct[c] += lgt[c] * irc;
    lirc += lgn[c] * Wcn[c] + lgt[c] * Wct[c];
  }
  maxwell_moments_adj(Mc, 0, k, lMc, lUc, lVc, llamc);
  // lamc = Wc0 / (2 pc), pc = gm1 (Wc3 - (Wc1 Uc + Wc2 Vc)/2), Uc = Wc1 irc, Vc = Wc2 irc, irc = 1/Wc0
  lWc[0] += llamc * real(0.5) / pc;
  real lpc = -llamc * lamc / pc;
  lWc[3] += lpc * k.gm1;
  lWc[1] += -lpc * k.gm1 * real(0.5) * Uc;
  lWc[2] += -lpc * k.gm1 * real(0.5) * Vc;
  lUc += -lpc * k.gm1 * real(0.5) * Wc[1];
  lVc += -lpc * k.gm1 * real(0.5) * Wc[2];
  lWc[1] += lUc * irc;
  lWc[2] += lVc * irc;
  lirc += lUc * Wc[1] + lVc * Wc[2];
  lWc[0] += -lirc * irc * irc;
}

template <class real>
DFW_HD void gks_flux_adj_sides(const real* wln, const real* wlt, const real* wrn, const real* wrt,
                               const Prim<real>& ql, const Prim<real>& qr, const Coef<real>& k,
                               const GksEqAdj<real>& e, real* lwln, real* lwlt, real* lwrn, real* lwrt,
                               PrimAdj<real>& lql, PrimAdj<real>& lqr) {
  const real* lWc = e.lWc;
  const real* lWcn = e.lWcn;
  const real* lWct = e.lWct;
  const real* lFlr = e.lFlr;
  const real* lMalr = e.lMalr;
  lql.p += e.lpl;
  lqr.p += e.lpr;
  // ---- reverse: the two half-space sides
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const real* wn = side == 0 ? wln : wrn;
    const real* wt = side == 0 ? wlt : wrt;
    real* lwn = side == 0 ? lwln : lwrn;
    real* lwt = side == 0 ? lwlt : lwrt;
    const Prim<real>& q = side == 0 ? ql : qr;
    PrimAdj<real>& lq = side == 0 ? lql : lqr;
    real lam = real(0.5) * q.r / q.p;
    Mom<real> M;
    maxwell_moments(q.u, q.v, lam, side == 0 ? 1 : -1, k, M);
    real g1[4], g2[4], a[4], b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      g1[c] = wn[c] * q.ir;
      g2[c] = wt[c] * q.ir;
    }
    micro_slope(g1, q.u, q.v, lam, real(0.5) / lam, k, a);
    micro_slope(g2, q.u, q.v, lam, real(0.5) / lam, k, b);
    MomAdj<real> lM;
    lM.zero();
    real la[4] = {0, 0, 0, 0}, lb[4] = {0, 0, 0, 0};
    real lt[4];
    real t[4];
    // Wc += r <psi>, Wcn += r <(a.psi) psi>, Wct += r <(b.psi) psi>
    mom_psi(M, 0, 0, t);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lq.r += lWc[c] * t[c];
      lt[c] = q.r * lWc[c];
    }
    mom_psi_adj(M, 0, 0, lt, lM);
    mom_s_psi(M, a, 0, 0, t);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lq.r += lWcn[c] * t[c];
      lt[c] = q.r * lWcn[c];
    }
    mom_s_psi_adj(M, a, 0, 0, lt, la, lM);
    mom_s_psi(M, b, 0, 0, t);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lq.r += lWct[c] * t[c];
      lt[c] = q.r * lWct[c];
    }
    mom_s_psi_adj(M, b, 0, 0, lt, lb, lM);
    // Flr += r <u psi>, Malr += r (<(a.psi) u^2 psi> + <(b.psi) u v psi>)
    mom_psi(M, 1, 0, t);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lq.r += lFlr[c] * t[c];
      lt[c] = q.r * lFlr[c];
    }
    mom_psi_adj(M, 1, 0, lt, lM);
    real t2[4];
    mom_s_psi(M, a, 2, 0, t);
    mom_s_psi(M, b, 1, 1, t2);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lq.r += lMalr[c] * (t[c] + t2[c]);
      lt[c] = q.r * lMalr[c];
    }
    mom_s_psi_adj(M, a, 2, 0, lt, la, lM);
    mom_s_psi_adj(M, b, 1, 1, lt, lb, lM);
    real lU = real(0), lV = real(0), llam = real(0);
    real lg1[4] = {0, 0, 0, 0}, lg2[4] = {0, 0, 0, 0};
    micro_slope_adj(g1, q.u, q.v, lam, k, la, lg1, lU, lV, llam);
    micro_slope_adj(g2, q.u, q.v, lam, k, lb, lg2, lU, lV, llam);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      lwn[c] += lg1[c] * q.ir;
      lwt[c] += lg2[c] * q.ir;
      lq.ir += lg1[c] * wn[c] + lg2[c] * wt[c];
    }
    maxwell_moments_adj(M, side == 0 ? 1 : -1, k, lM, lU, lV, llam);
    lq.u += lU;
    lq.v += lV;
    // lam = r / (2 p)
    lq.r += llam * real(0.5) / q.p;
    lq.p += -llam * lam / q.p;
  }
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
