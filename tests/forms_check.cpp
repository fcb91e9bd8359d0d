// Host check of the forms of dfw_math.hpp (the FP64 kernels) against
// the candidate form (dfw_math_f32.hpp, here in FP64 too) through the functions that the interface
// kernel calls: the normal sweep (line values, normal derivatives and time-limiter weight) and the
// tangential sweep with the fluxes, on smooth and discontinuous data, both branches of the hybrid
// switch, characteristic and component-wise; and the Gauss-point fluxes, time derivatives and DF, the
// gas-kinetic ones through derivatives of moments against the micro-slopes.  Prints one line per property: name, worst deviation
// relative to the data.  Built and run by tests/test_forms.py.
#include <cmath>
#include <cstdio>
#include <random>

#include "../paper_2402_10914_amd/csrc/dfw_math.hpp"
#include "../paper_2402_10914_amd/csrc/dfw_math_f32.hpp"

using namespace dfw;

static Coef<double> coef() {
  Coef<double> k;
  const double g = 1.4, dh = 0.85, dl = 0.85;
  k.gamma = g; k.gm1 = g - 1; k.inv_gm1 = 1 / (g - 1); k.alpha_thres = 0.5; k.eps = 1e-6;
  k.c1 = 0.01; k.c2 = 5.0; k.K = (4 - 2 * g) / (g - 1);
  const double d[4] = {(1 - dh) * (1 - dl) / 2, (1 - dh) * dl, (1 - dh) * (1 - dl) / 2, dh};
  for (int i = 0; i < 4; ++i) k.d[i] = d[i];
  for (int i = 0; i < 3; ++i) k.dr[i] = d[i] / d[3];
  k.inv_d3 = 1 / d[3]; k.K2 = k.K + 2; k.k4K2 = 4 / (k.K + 2); k.sw_rule = 0;
  return k;
}

static std::mt19937_64 rng(7);
static double U(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }

static void state(double r, double u, double v, double p, double* w) {
  w[0] = r; w[1] = r * u; w[2] = r * v; w[3] = p / 0.4 + 0.5 * r * (u * u + v * v);
}

// n states along a line: kind 0 smooth, 1 a jump, 2 independent
static void fill(int kind, int n, double (*w)[4]) {
  double a[4], b[4];
  const double ra = U(0.3, 2), rb = U(0.3, 2), pa = std::pow(10.0, U(-1, 1)), pb = std::pow(10.0, U(-1, 1));
  state(ra, U(-1, 1), U(-1, 1), pa, a);
  state(rb, U(-1, 1), U(-1, 1), pb, b);
  const double ph = U(0, 6), amp = std::pow(10.0, U(-8, -0.5));
  const int at = 1 + int(rng() % (n - 1));
  for (int m = 0; m < n; ++m) {
    if (kind == 0) state(ra * (1 + amp * std::sin(ph + 0.4 * m)), 0.3 + amp * std::cos(ph + 0.3 * m), -0.2, pa * (1 + amp * std::cos(ph + 0.5 * m)), w[m]);
    else if (kind == 1) for (int c = 0; c < 4; ++c) w[m][c] = m < at ? a[c] : b[c];
    else state(U(0.3, 2), U(-1, 1), U(-1, 1), std::pow(10.0, U(-1, 1)), w[m]);
  }
}

static double worst(const double* x, const double* y, int n, double scale) {
  double e = 0;
  for (int i = 0; i < n; ++i) e = std::fmax(e, std::fabs(x[i] - y[i]) / scale);
  return e;
}

template <bool CHAR>
static void sweeps(const Coef<double>& k, double* e) {
  for (int it = 0; it < 20000; ++it) {
    const int kind = it % 3;
    const bool df = it % 5 == 0;
    double cell[6][4];
    fill(kind, 6, cell);
    double s = 0;
    for (int m = 0; m < 6; ++m) for (int c = 0; c < 4; ++c) s = std::fmax(s, std::fabs(cell[m][c]));
    double al[4];
    for (double& x : al) x = df ? U(0, 0.45) : U(0.6, 1);
    double x[16], y[16], ox = 1, oy = 1;
    normal_sweep<double, CHAR>(cell, al[0], al[1], al[2], al[3], 1.0, k, x, x + 4, x + 8, x + 12, &ox);
    cand::normal_sweep<CHAR>(cell, al[0], al[1], al[2], al[3], 1.0, k, y, y + 4, y + 8, y + 12, &oy);
    e[0] = std::fmax(e[0], worst(x, y, 16, s));
    // the weight is a ratio of indicators: on data that is smooth to rounding it is ill-conditioned
    if (kind != 0) e[1] = std::fmax(e[1], std::fabs(ox - oy));
    double lines[2][5][4], alpha[2][3], wln[4], wrn[4];
    for (int side = 0; side < 2; ++side) {
      fill(kind, 5, lines[side]);
      for (double& a : alpha[side]) a = df ? U(0, 0.45) : U(0.6, 1);
    }
    for (int side = 0; side < 2; ++side)
      for (int m = 0; m < 5; ++m)
        for (int c = 0; c < 4; ++c) s = std::fmax(s, std::fabs(lines[side][m][c]));
    auto line = [&](int side, int m, int c) -> double { return lines[side][m][c]; };
    const Basis<double> B = recon_basis<CHAR>(cell[2], cell[3], k);
    double gw[2][2][4], gt[2][2][4];
    segment_states<CHAR>(B, line, alpha, 1.0, k, gw, gt);
    // the candidate form's Gauss-point states, component by component
    for (int side = 0; side < 2; ++side) {
      double q[5][4], v[2][4], d[2][4], w[4];
      for (int m = 0; m < 5; ++m) to_recon<CHAR>(B, lines[side][m], q[m]);
      for (int c = 0; c < 4; ++c) {
        const double st[5] = {q[0][c], q[1][c], q[2][c], q[3][c], q[4][c]};
        double vv[2], dd[2];
        cand::recon_gauss(st, alpha[side][0], alpha[side][1], alpha[side][2], k, vv, dd);
        for (int g = 0; g < 2; ++g) { v[g][c] = vv[g]; d[g][c] = dd[g]; }
      }
      for (int g = 0; g < 2; ++g) {
        from_recon<CHAR>(B, v[g], w);
        e[2] = std::fmax(e[2], worst(gw[side][g], w, 4, s));
        from_recon<CHAR>(B, d[g], w);
        e[2] = std::fmax(e[2], worst(gt[side][g], w, 4, s));
      }
    }
  }
}

// Fluxes, time derivatives and DF of one Gauss point; the second form's Prim is its own.
static void fluxes(double* e) {
  for (int it = 0; it < 20000; ++it) {
    Coef<double> k = coef();
    if (it % 4 == 3) k.c1 = k.c2 = 0;  // zero collision time: exp(-inf)
    double w[2][4], wn[2][4], wt[2][4];
    for (int s = 0; s < 2; ++s) {
      state(U(0.3, 2), U(-2, 2), U(-2, 2), std::pow(10.0, U(-0.5, 0.5)), w[s]);
      for (int c = 0; c < 4; ++c) { wn[s][c] = U(-1, 1); wt[s][c] = U(-1, 1); }
    }
    if (it % 2) for (int c = 0; c < 4; ++c) w[1][c] = w[0][c] * (1 + 1e-3 * U(-1, 1));
    const double dt = std::pow(10.0, U(-4, 0));
    const Prim<double> l = prim(w[0], k), r = prim(w[1], k);
    const cand::Prim<double> cl = cand::prim(w[0], k), cr = cand::prim(w[1], k);
    double x[8], y[8], isl[2];
    lf_flux<double, true>(w[0], wn[0], wt[0], w[1], wn[1], wt[1], l, r, k, x, x + 4);
    cand::lf_flux<double, true>(w[0], wn[0], wt[0], w[1], wn[1], wt[1], cl, cr, k, y, y + 4);
    double s = 1;
    for (double v : y) s = std::fmax(s, std::fabs(v));
    e[0] = std::fmax(e[0], worst(x, y, 8, s));
    gks_point_flux<true>(wn[0], wt[0], wn[1], wt[1], l, r, dt, k, x, x + 4, isl);
    cand::gks_flux<double, true>(w[0], wn[0], wt[0], w[1], wn[1], wt[1], cl, cr, dt, k, y, y + 4);
    s = 1;
    for (double v : y) s = std::fmax(s, std::fabs(v));
    e[1] = std::fmax(e[1], worst(x, y, 8, s));
    const double df = cand::df_factor(cl, cr);
    const double d[3] = {df_factor(l, r), df_factor(l, r, k), df_factor_gks(l, r, isl, k)}, ref[3] = {df, df, df};
    e[2] = std::fmax(e[2], worst(d, ref, 3, 1.0));
  }
}

int main() {
  const Coef<double> k = coef();
  double g[3] = {0, 0, 0};
  fluxes(g);
  std::printf("flux_lf %.3e\nflux_gks %.3e\nflux_df %.3e\n", g[0], g[1], g[2]);
  double e[3] = {0, 0, 0}, f[3] = {0, 0, 0};
  sweeps<true>(k, e);
  sweeps<false>(k, f);
  std::printf("normal_char %.3e\nomega_char %.3e\ntangential_char %.3e\n", e[0], e[1], e[2]);
  std::printf("normal_comp %.3e\nomega_comp %.3e\ntangential_comp %.3e\n", f[0], f[1], f[2]);
  return 0;
}
