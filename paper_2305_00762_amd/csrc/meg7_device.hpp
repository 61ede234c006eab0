// Device-side building blocks of the MEG7 scheme (Chamarthi, arXiv
// 2305.00762) for gfx950, in a frame rotated to the interface normal:
// primitive vector W = (rho, un, ut, p), conservative (rho, rho un, rho ut, E).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gbr {

// Constants of the scheme.
constexpr double kAlphaV = 4.0;   // alpha-damping coefficient, Sec. 2.1 eq. (eqn:alphad)
constexpr double kXiMP = 7.0;     // MP parameter xi, Sec. 2.3 eq. (eqn:alpha)
constexpr double kMPTol = 1e-40;  // MP activation threshold, eq. (eqn:hocus/mp5Condition)
constexpr double kPsiC = 0.5;     // detector threshold psi_c, Sec. 2.4 eq. (buffer)
constexpr double kXiDet = 1e-3;   // detector xi, eq. (buffer)
// eq. (buffer): eps = 0.9 psi_c / (1 - 0.9 psi_c) xi^2 (folded with IEEE rounding)
constexpr double kDetEps = (0.9 * kPsiC) / (1.0 - 0.9 * kPsiC) * (kXiDet * kXiDet);

// Reciprocal and reciprocal square root: hardware estimate refined by two
// Newton steps (full FP64 accuracy up to the last bit or two; positive,
// normal arguments only).  Used for the Riemann-solver arithmetic, never
// for the detector decision.
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
__device__ __forceinline__ double rsq_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double e = fma(-x * y, y, 1.0);
  y = fma(0.5 * y, e, y);
  e = fma(-x * y, y, 1.0);
  return fma(0.5 * y, e, y);
}
__device__ __forceinline__ double sqrt_nr(double x) {
  const double y = rsq_nr(x);
  const double s = x * y;
  return fma(0.5 * y, fma(-s, s, x), s);
}

// The same from one third-order step, for the Riemann solver: with the
// estimate's relative error e (about 2^-24), 1/x = r (1 + e + e^2) and
// 1/sqrt(x) = y (1 + e/2 + 3 e^2/8) up to e^3 < 2^-70, so one such step
// reaches the last bit or two of FP64 in 3 (6, 5) dependent operations where
// two Newton steps take 4 (8, 11).
__device__ __forceinline__ double rcp_c3(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ double rsq_c3(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ double sqrt_c3(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double t = x * y;
  const double e = fma(-t, y, 1.0);
  return fma(t * e, fma(0.375, e, 0.5), t);
}

// fl(a / b) from rb = rcp_nr(b): the quotient a rb and one correction by the
// exact residual.  These are the steps of the hardware's IEEE division after
// its scaling step (reciprocal estimate, two Newton steps, quotient, fused
// correction), and that step leaves operands unchanged when both magnitudes
// lie in [2^-300, 2^300] or the numerator is zero (div_rb_ok): there the
// result is the IEEE quotient bit for bit, up to the sign of a zero result
// (gbr_selftest_division checks it on the device).  One reciprocal then
// serves the three quotients of a cell.
__device__ __forceinline__ double div_rb(double a, double b, double rb) {
#pragma clang fp contract(off)
  const double q = a * rb;
  return fma(fma(-b, q, a), rb, q);
}
__device__ __forceinline__ bool div_rb_ok(double a) {
  const double m = fabs(a);
  return m <= 0x1p300 && (m >= 0x1p-300 || m == 0.0);
}

// The compiler would issue all of a long walk's loads first and its sums last,
// which needs several times the register file: pin() makes a running sum's
// value due here, hold() keeps the loads on either side apart.
template <class T>
__device__ __forceinline__ void pin(T& v) { __asm__ volatile("" : "+v"(v)); }
__device__ __forceinline__ void hold() { __asm__ volatile("" ::: "memory"); }

// Sixth-order central first derivative, eq. (eqn:six), scaled by the
// spacing: returns dx * dPhi/dx from Phi_{-3..3} (pm3 .. p3).
__device__ __forceinline__ double grad6(double pm3, double pm2, double pm1, double p1,
                                        double p2, double p3) {
  return (45.0 * (p1 - pm1) - 9.0 * (p2 - pm2) + (p3 - pm3)) * (1.0 / 60.0);
}

// Density detector of Sec. 2.4, eps in numerator and denominator: the decision
// psi < psi_c (= 1/2) of psi = fl(num / den), num = 2ab + eps, den = a^2 + b^2 +
// eps (both positive), every operation rounded on its own in a fixed order so
// that it is reproducible bit for bit, but without the division:
// fl(num / den) < 1/2 holds exactly when num / den < 1/2 - 2^-55 (the rounding
// boundary below 1/2; a tie rounds to 1/2, whose significand is even), i.e.
// when den - 2 num > den 2^-54.  That is 2 num < den: let 2^e <= 2 num < 2^(e+1)
// be below den.  Where den < 2^(e+2) both are multiples of 2^(e-52), so
// den - 2 num >= 2^(e-52) > den 2^-54; where den >= 2^(e+2), den - 2 num >
// den / 2.  And 2 num = fl(4 ab + 2 eps) (scaling by 2 is exact), one fused
// operation on fl(ab).
// em, ep: the density jumps r0 - rm1 and rp1 - r0.
static_assert(kPsiC == 0.5, "the division-free decision assumes psi_c = 1/2");
__device__ __forceinline__ bool detector_flag_jumps(double rm2, double rm1, double r0, double rp1,
                                                    double rp2, double em, double ep) {
#pragma clang fp contract(off)
  double a = fabs(em) + fabs(fma(-2.0, rm1, r0) + rm2);
  double b = fabs(ep) + fabs(fma(-2.0, rp1, r0) + rp2);
  double den = (a * a + b * b) + kDetEps;
  return fma(4.0, a * b, 2.0 * kDetEps) < den;
}
__device__ __forceinline__ bool detector_flag(double rm2, double rm1, double r0, double rp1,
                                              double rp2) {
#pragma clang fp contract(off)
  return detector_flag_jumps(rm2, rm1, r0, rp1, rp2, r0 - rm1, rp1 - r0);
}

// (sign a + sign b)/2 min(|a|,|b|), eq. (eqn:alpha): one of the two terms is zero
__device__ __forceinline__ double minmod(double a, double b) {
  return fmax(fmin(a, b), 0.0) + fmin(fmax(a, b), 0.0);
}

// GRB interface states, eq. (eqn:grb).  v[k] = Phi_{j+k-2} (k=0..5),
// g[k] = Phi'_{j+k-2} (Phi' = dx dPhi/dx).
__device__ __forceinline__ double grb_left(const double* v, const double* g) {
  constexpr double s = 1.0 / 840.0;
  return (3.0 * s) * (v[0] + v[4]) + (178.0 * s) * (v[1] + v[3]) + (478.0 * s) * v[2] +
         (420.0 * s) * g[2] + (60.0 * s) * (g[1] - g[3]);
}
__device__ __forceinline__ double grb_right(const double* v, const double* g) {
  constexpr double s = 1.0 / 840.0;
  return (3.0 * s) * (v[1] + v[5]) + (178.0 * s) * (v[2] + v[4]) + (478.0 * s) * v[3] -
         (420.0 * s) * g[3] + (60.0 * s) * (g[2] - g[4]);
}

// Fourth-order GRB states: the subset alpha = 4, beta = 0 of eqs.
// (good_6tth-order_scheme_flux), (alpha-beta) put into eq. (eqn:lingrb),
//   Phi^L = (4 (Phi_{j-1} + Phi_{j+1}) + 16 Phi_j + Phi'_{j-1} + 12 Phi'_j - Phi'_{j+1}) / 24
// and its mirror image for Phi^R at j+1/2.  Same v, g layout as grb_left.
__device__ __forceinline__ double grb4_left(const double* v, const double* g) {
  constexpr double s = 1.0 / 24.0;
  return (4.0 * s) * (v[1] + v[3]) + (16.0 * s) * v[2] + (12.0 * s) * g[2] + s * (g[1] - g[3]);
}
__device__ __forceinline__ double grb4_right(const double* v, const double* g) {
  constexpr double s = 1.0 / 24.0;
  return (4.0 * s) * (v[2] + v[4]) + (16.0 * s) * v[3] - (12.0 * s) * g[3] + s * (g[2] - g[4]);
}

// GRB states of the selected order: 7 (eq. eqn:grb) or 4 (the subset above).
template <int ORD>
__device__ __forceinline__ double grb_l(const double* v, const double* g) {
  return ORD == 4 ? grb4_left(v, g) : grb_left(v, g);
}
template <int ORD>
__device__ __forceinline__ double grb_r(const double* v, const double* g) {
  return ORD == 4 ? grb4_right(v, g) : grb_right(v, g);
}

// Mean of the reconstructed cell fluxes, (F(f_L) + F(f_R))/2 at j+1/2, from
// f[q] = f_{j+q-4} (q = 0..9).  The sum of a left stencil and its mirror image
// is symmetric about the interface, so pairs are added first:
//   order 7, eqs. (flux-full), (flux-right): (1052, -250, 38, 1, -1) / 1680;
//   order 4, eq. (fourth) and its mirror:    (1821, -461, 85, -4, -1) / 2880.
template <int ORD>
__device__ __forceinline__ double flux_mean(const double* f) {
  if (ORD == 4) {
    constexpr double s = 1.0 / 2880.0;
    return (1821.0 * s) * (f[4] + f[5]) - (461.0 * s) * (f[3] + f[6]) +
           (85.0 * s) * (f[2] + f[7]) - (4.0 * s) * (f[1] + f[8]) - s * (f[0] + f[9]);
  }
  constexpr double s = 1.0 / 1680.0;
  return (1052.0 * s) * (f[4] + f[5]) - (250.0 * s) * (f[3] + f[6]) +
         (38.0 * s) * (f[2] + f[7]) + s * (f[1] + f[8]) - s * (f[0] + f[9]);
}

// MP curvature d of eq. (eqn:mp-procedure) at the centre of v[-1..1], g[-1..1].
__device__ __forceinline__ double mp_curv(double vm, double v0, double vp, double gm,
                                          double gp) {
  return 2.0 * (vp - 2.0 * v0 + vm) - 0.5 * (gp - gm);
}

// MEG7 left and right values at j+1/2 of one characteristic component
// (Sec. 2.3): GRB value (of order ORD), the activation test, and the MP
// bounds.  v, g hold offsets -2..3 around cell j.  The right value is the
// mirror image.
template <int ORD = 7>
__device__ __forceinline__ void meg7_pair(const double* v, const double* g, double& outL,
                                          double& outR) {
  const double dm1 = mp_curv(v[0], v[1], v[2], g[0], g[2]);
  const double d0 = mp_curv(v[1], v[2], v[3], g[1], g[3]);
  const double dp1 = mp_curv(v[2], v[3], v[4], g[2], g[4]);
  const double dp2 = mp_curv(v[3], v[4], v[5], g[3], g[5]);
  const double md = 0.5 * (v[2] + v[3]) - 0.5 * minmod(d0, dp1);
  {
    double phi = grb_l<ORD>(v, g);
    double pmp = v[2] + minmod(v[3] - v[2], kXiMP * (v[2] - v[1]));
    if ((phi - v[2]) * (phi - pmp) > kMPTol) {
      double ul = v[2] + kXiMP * (v[2] - v[1]);
      double lc = 0.5 * (3.0 * v[2] - v[1]) + (4.0 / 3.0) * minmod(d0, dm1);
      double lo = fmax(fmin(v[2], fmin(v[3], md)), fmin(v[2], fmin(ul, lc)));
      double hi = fmin(fmax(v[2], fmax(v[3], md)), fmax(v[2], fmax(ul, lc)));
      phi = phi + minmod(lo - phi, hi - phi);
    }
    outL = phi;
  }
  {
    double phi = grb_r<ORD>(v, g);
    double pmp = v[3] + minmod(v[2] - v[3], kXiMP * (v[3] - v[4]));
    if ((phi - v[3]) * (phi - pmp) > kMPTol) {
      double ul = v[3] + kXiMP * (v[3] - v[4]);
      double lc = 0.5 * (3.0 * v[3] - v[4]) + (4.0 / 3.0) * minmod(dp1, dp2);
      double lo = fmax(fmin(v[3], fmin(v[2], md)), fmin(v[3], fmin(ul, lc)));
      double hi = fmin(fmax(v[3], fmax(v[2], md)), fmax(v[3], fmax(ul, lc)));
      phi = phi + minmod(lo - phi, hi - phi);
    }
    outR = phi;
  }
}

// Characteristic MEG7 states at an interface (Secs. 2.3, 2.4, flagged
// branch).  Wf(q, f) returns rotated primitive field f at offset q-2
// (q = 0..5) from cell j; CG(fa, fb, ca, cb, cg) writes the normal gradients
// (spacing-scaled) of the combination ca * field fa + cb * field fb at the
// same six offsets.  Eigenvectors of the primitive normal Jacobian are taken
// at the mean density and pressure of cells j, j+1.  Each characteristic
// field combines two primitive fields (rows of L: (u_n, p), (rho, p), (u_t),
// (u_n, p)); the four fields are limited one at a time in a rolled loop that
// reads only its two primitive fields, which keeps the register footprint
// small, and are projected back by accumulating the columns of R.
template <int ORD = 7, class FW, class FC>
__device__ __forceinline__ void meg7_char_states_comb(FW Wf, FC CG, double gamma, double WLo[4],
                                                      double WRo[4]) {
  const double rb = 0.5 * (Wf(2, 0) + Wf(3, 0));
  const double pb = 0.5 * (Wf(2, 3) + Wf(3, 3));
  const double irb = rcp_nr(rb);
  const double cb = sqrt_nr(gamma * pb * irb);
  const double icb = rcp_nr(cb);
  const double h2c = 0.5 * icb, ic2 = icb * icb, h2c2 = 0.5 * ic2;
  const double cor = cb * irb, c2 = cb * cb;
#pragma unroll
  for (int m = 0; m < 4; ++m) { WLo[m] = 0.0; WRo[m] = 0.0; }
#pragma unroll 1
  for (int m = 0; m < 4; ++m) {
    // row m of L as ca * field fa + cb_ * field fb
    const int fa = (m == 1) ? 0 : ((m == 2) ? 2 : 1);
    const int fb = (m == 2) ? 2 : 3;
    const double ca = (m == 0) ? -rb * h2c : ((m == 3) ? rb * h2c : 1.0);
    const double cbv = (m == 1) ? -ic2 : ((m == 2) ? 0.0 : h2c2);
    double cv[6], cg[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) cv[q] = ca * Wf(q, fa) + cbv * Wf(q, fb);
    CG(fa, fb, ca, cbv, cg);
    double cl, cr;
    meg7_pair<ORD>(cv, cg, cl, cr);
    // column m of R = L^{-1}: (1,-c/rho,0,c^2), (1,0,0,0), (0,0,1,0), (1,c/rho,0,c^2)
    const double b0 = (m == 2) ? 0.0 : 1.0;
    const double b1 = (m == 0) ? -cor : ((m == 3) ? cor : 0.0);
    const double b2 = (m == 2) ? 1.0 : 0.0;
    const double b3 = (m == 0 || m == 3) ? c2 : 0.0;
    WLo[0] += b0 * cl; WLo[1] += b1 * cl; WLo[2] += b2 * cl; WLo[3] += b3 * cl;
    WRo[0] += b0 * cr; WRo[1] += b1 * cr; WRo[2] += b2 * cr; WRo[3] += b3 * cr;
  }
}

// The same with staged gradients: Gf(q, f) is the normal gradient of rotated
// field f at offset q-2.
template <int ORD = 7, class FW, class FG>
__device__ __forceinline__ void meg7_char_states(FW Wf, FG Gf, double gamma, double WLo[4],
                                                 double WRo[4]) {
  meg7_char_states_comb<ORD>(
      Wf,
      [&](int fa, int fb, double ca, double cb, double cg[6]) {
#pragma unroll
        for (int q = 0; q < 6; ++q) cg[q] = ca * Gf(q, fa) + cb * Gf(q, fb);
      },
      gamma, WLo, WRo);
}

// The same from the cells alone, for NV = 4 fields (rho, u_n, u_t, p) or 5
// (rho, u_n, u_t1, u_t2, p: an identity row and column for the second
// tangential velocity): Vc(k, f) is field f at offset k - 5 from cell j,
// k = 0..11.  Each field is read once and its six gradients (eq. eqn:six) are
// formed once: the two acoustic rows from (u_n, p), the entropy row from rho
// and the p still at hand, then the tangential ones.  Against one row at a
// time, each from its two fields: half the reads and 110 of about 1000
// operations fewer.
// F32: the gradients of the FP32-bulk form, float32 stencils on float32 edge
// jumps.
template <int NV, int ORD, bool F32, class FV>
__device__ __forceinline__ void meg7_char_states_cells(FV Vc, double gamma, double* WLo,
                                                       double* WRo) {
  const double rb = 0.5 * (Vc(5, 0) + Vc(6, 0));
  const double pb = 0.5 * (Vc(5, NV - 1) + Vc(6, NV - 1));
  const double irb = rcp_nr(rb);
  const double cb = sqrt_nr(gamma * pb * irb);
  const double icb = rcp_nr(cb);
  const double ic2 = icb * icb, h2c2 = 0.5 * ic2, ca = rb * (0.5 * icb);
  const double cor = cb * irb, c2 = cb * cb;
  auto field = [&](int f, double (&v)[6], double (&g)[6]) {
    double c[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) c[k] = Vc(k, f);
    float e[11];
    if (F32) {
#pragma unroll
      for (int a = 0; a < 11; ++a) e[a] = (float)(c[a + 1] - c[a]);
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      v[q] = c[q + 3];
      if (F32)
        g[q] = (1.0f / 60.0f) * (37.0f * (e[q + 2] + e[q + 3]) - 8.0f * (e[q + 1] + e[q + 4]) +
                                 (e[q] + e[q + 5]));
      else
        g[q] = grad6(c[q], c[q + 1], c[q + 2], c[q + 4], c[q + 5], c[q + 6]);
    }
  };
  double vp[6], gp[6], v[6], g[6], mv[6], mg[6];
  double l0, r0, l1, r1, l2, r2;
  field(NV - 1, vp, gp);
  field(1, v, g);
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const double t = ca * v[q], u = ca * g[q];
    mv[q] = h2c2 * vp[q] - t;
    mg[q] = h2c2 * gp[q] - u;
    v[q] = h2c2 * vp[q] + t;
    g[q] = h2c2 * gp[q] + u;
  }
  meg7_pair<ORD>(mv, mg, l0, r0);
  meg7_pair<ORD>(v, g, l2, r2);
  hold();
  field(0, v, g);
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    v[q] -= ic2 * vp[q];
    g[q] -= ic2 * gp[q];
  }
  meg7_pair<ORD>(v, g, l1, r1);
  WLo[0] = l0 + l1 + l2;
  WRo[0] = r0 + r1 + r2;
  WLo[1] = cor * (l2 - l0);
  WRo[1] = cor * (r2 - r0);
  WLo[NV - 1] = c2 * (l0 + l2);
  WRo[NV - 1] = c2 * (r0 + r2);
#pragma unroll
  for (int t = 2; t < NV - 1; ++t) {
    hold();
    field(t, v, g);
    meg7_pair<ORD>(v, g, WLo[t], WRo[t]);
  }
}

// Conservative (rho, rho un, rho ut, E) to primitive (rho, un, ut, p),
// eq. (eqn:pressure).  A non-positive density gives a non-positive or NaN
// result, which the positivity test of the callers rejects.
__device__ __forceinline__ void cons_to_prim(const double Q[4], double gamma, double W[4]) {
  const double ir = rcp_nr(Q[0]);
  W[0] = Q[0];
  W[1] = Q[1] * ir;
  W[2] = Q[2] * ir;
  W[3] = (gamma - 1.0) * (Q[3] - 0.5 * (Q[1] * W[1] + Q[2] * W[2]));
}

// Characteristic MEG7 states of MEG7-cons (Sec. 2.3 on conservative
// variables).  Qf(q, f) / Gf(q, f) return rotated conservative field f and its
// normal gradient (spacing-scaled) at offset q-2 from cell j.  The
// eigenvectors are those of the conservative normal flux Jacobian at the
// arithmetic mean of the conservative states of cells j and j+1, with
// b1 = (gamma-1)/c^2, b2 = b1 (u^2+v^2)/2.  Rows of L:
//   ((b2 + u/c)/2, -(b1 u + 1/c)/2, -b1 v/2, b1/2), (1 - b2, b1 u, b1 v, -b1),
//   (-v, 0, 1, 0), ((b2 - u/c)/2, -(b1 u - 1/c)/2, -b1 v/2, b1/2);
// columns of R = L^{-1}: (1, u-c, v, H-uc), (1, u, v, (u^2+v^2)/2), (0, 0, 1, v),
//   (1, u+c, v, H+uc).  Every row reads all four fields, so the rows are
// limited one at a time in a rolled loop and projected back column by column.
// CG(l, cv, cg) writes the combination sum_f l[f] field f and its gradient at
// the six offsets.
template <int ORD = 7, class FQ, class FC>
__device__ __forceinline__ void meg7_char_states_cons_comb(FQ Qf, FC CG, double gamma,
                                                           double QLo[4], double QRo[4]) {
  const double q0 = 0.5 * (Qf(2, 0) + Qf(3, 0)), q1 = 0.5 * (Qf(2, 1) + Qf(3, 1));
  const double q2 = 0.5 * (Qf(2, 2) + Qf(3, 2)), q3 = 0.5 * (Qf(2, 3) + Qf(3, 3));
  const double iq0 = rcp_nr(q0);
  const double ub = q1 * iq0, vb = q2 * iq0;
  const double ke = 0.5 * (ub * ub + vb * vb);
  const double pb = (gamma - 1.0) * (q3 - q0 * ke);
  const double hb = (q3 + pb) * iq0;
  const double cb = sqrt_nr(gamma * pb * iq0);
  const double icb = rcp_nr(cb);
  const double b1 = (gamma - 1.0) * icb * icb, b2 = b1 * ke;
#pragma unroll
  for (int m = 0; m < 4; ++m) { QLo[m] = 0.0; QRo[m] = 0.0; }
#pragma unroll 1
  for (int m = 0; m < 4; ++m) {
    // the field reads do not depend on m: keep them inside the loop (an empty
    // asm with a memory clobber stops the compiler hoisting all 48 of them)
    __asm__ volatile("" ::: "memory");
    const double sg = (m == 0) ? 1.0 : -1.0;   // u/c and 1/c enter rows 0 and 3 with opposite signs
    double l0, l1, l2, l3;
    if (m == 1) {
      l0 = 1.0 - b2; l1 = b1 * ub; l2 = b1 * vb; l3 = -b1;
    } else if (m == 2) {
      l0 = -vb; l1 = 0.0; l2 = 1.0; l3 = 0.0;
    } else {
      l0 = 0.5 * (b2 + sg * ub * icb);
      l1 = -0.5 * (b1 * ub + sg * icb);
      l2 = -0.5 * b1 * vb;
      l3 = 0.5 * b1;
    }
    double cv[6], cg[6];
    const double lm[4] = {l0, l1, l2, l3};
    CG(lm, cv, cg);
    double cl, cr;
    meg7_pair<ORD>(cv, cg, cl, cr);
    double r0, r1, r2, r3;
    if (m == 1) {
      r0 = 1.0; r1 = ub; r2 = vb; r3 = ke;
    } else if (m == 2) {
      r0 = 0.0; r1 = 0.0; r2 = 1.0; r3 = vb;
    } else {
      r0 = 1.0; r1 = ub - sg * cb; r2 = vb; r3 = hb - sg * ub * cb;
    }
    QLo[0] += r0 * cl; QLo[1] += r1 * cl; QLo[2] += r2 * cl; QLo[3] += r3 * cl;
    QRo[0] += r0 * cr; QRo[1] += r1 * cr; QRo[2] += r2 * cr; QRo[3] += r3 * cr;
  }
}

// The same with staged gradients.
template <int ORD = 7, class FQ, class FG>
__device__ __forceinline__ void meg7_char_states_cons(FQ Qf, FG Gf, double gamma,
                                                      double QLo[4], double QRo[4]) {
  meg7_char_states_cons_comb<ORD>(
      Qf,
      [&](const double l[4], double cv[6], double cg[6]) {
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          cv[q] = l[0] * Qf(q, 0) + l[1] * Qf(q, 1) + l[2] * Qf(q, 2) + l[3] * Qf(q, 3);
          cg[q] = l[0] * Gf(q, 0) + l[1] * Gf(q, 1) + l[2] * Gf(q, 2) + l[3] * Gf(q, 3);
        }
      },
      gamma, QLo, QRo);
}

// The same from the cells alone: Vc(k, f) is field f at offset k - 5 from cell
// j, k = 0..11; the gradients are those of eq. (eqn:six) on the jumps of the
// combination itself.
template <int ORD = 7, class FV>
__device__ __forceinline__ void meg7_char_states_cons_cells(FV Vc, double gamma, double QLo[4],
                                                            double QRo[4]) {
  meg7_char_states_cons_comb<ORD>(
      [&](int q, int f) { return Vc(q + 3, f); },
      [&](const double l[4], double cv[6], double cg[6]) {
        double cc[12], ce[11];
#pragma unroll
        for (int k = 0; k < 12; ++k)
          cc[k] = l[0] * Vc(k, 0) + l[1] * Vc(k, 1) + l[2] * Vc(k, 2) + l[3] * Vc(k, 3);
#pragma unroll
        for (int a = 0; a < 11; ++a) ce[a] = cc[a + 1] - cc[a];
        constexpr double z = 1.0 / 60.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          cv[q] = cc[q + 3];
          cg[q] = z * (37.0 * (ce[q + 2] + ce[q + 3]) - 8.0 * (ce[q + 1] + ce[q + 4]) +
                       (ce[q] + ce[q + 5]));
        }
      },
      gamma, QLo, QRo);
}

// Normal convective flux of the state W (Sec. 1 flux vectors, rotated).
__device__ __forceinline__ void conv_flux(const double W[4], double g1inv, double F[4]) {
  const double E = W[3] * g1inv + 0.5 * W[0] * (W[1] * W[1] + W[2] * W[2]);
  const double m = W[0] * W[1];
  F[0] = m;
  F[1] = m * W[1] + W[3];
  F[2] = m * W[2];
  F[3] = W[1] * (E + W[3]);
}

// sin(x) for x in [0, pi/2]: its Taylor series to x^21 (truncation below
// 3e-16 on that interval), in Horner form on x^2.  Small in registers, unlike
// the library sine, so it can sit inside the Riemann solver.
__device__ __forceinline__ double sin_quarter(double x) {
  const double z = x * x;
  double t = 1.0 / 51090942171709440000.0;          // 1/21!
  t = fma(t, -z, 1.0 / 121645100408832000.0);        // 1/19!
  t = fma(t, -z, 1.0 / 355687428096000.0);           // 1/17!
  t = fma(t, -z, 1.0 / 1307674368000.0);             // 1/15!
  t = fma(t, -z, 1.0 / 6227020800.0);                // 1/13!
  t = fma(t, -z, 1.0 / 39916800.0);                  // 1/11!
  t = fma(t, -z, 1.0 / 362880.0);                    // 1/9!
  t = fma(t, -z, 1.0 / 5040.0);                      // 1/7!
  t = fma(t, -z, 1.0 / 120.0);                       // 1/5!
  t = fma(t, -z, 1.0 / 6.0);                         // 1/3!
  t = fma(t, -z, 1.0);
  return x * t;
}

// HLLC with Einfeldt (Roe-average) bounds in the wave-sum form
//   F = (F_L + F_R)/2 - (phi |S_L|(Q*_L - Q_L) + |S*|(Q*_R - Q*_L) + phi |S_R|(Q_R - Q*_R))/2
// which is the canonical form of eq. (eqn:Riemann).  Only the mean
// (F_L + F_R)/2 of the reconstructed fluxes enters: callers pass it as fs Fm.
// phi = 1 for HLLC; the shock-stable (low-Mach-limited) form takes
// phi = sin(pi/2 min(1, Ma/0.1)), Ma = max(|u_L|/c_L, |u_R|/c_R).
// NV = 4: W = (rho, u_n, u_t, p); NV = 5: two tangential velocities.
//
// The wave sum is gathered per jump, (phi |S_L| - |S*|) dQ_L +
// (phi |S_R| - |S*|) dQ_R + |S*| (Q_R - Q_L), with the star-state jumps
//   dQ_L = Q*_L - Q_L =  g_L (1, S_L, v_L, .),  g_L = rho_L a_L / (S_L - S*),
//   dQ_R = Q_R - Q*_R = -g_R (1, S_R, v_R, .),  g_R = rho_R a_R / (S_R - S*),
// a_L = S* - u_L, a_R = S* - u_R formed from the jumps of p and u, and the
// energy rows a_L/(S_L - S*) (E_L + p_L + m_L S*), resp. R.  The Roe sound
// speed is c~^2 = w_L c_L^2 + w_R c_R^2 + (gamma-1)/2 w_L w_R |dU|^2 (the
// Roe enthalpy less the kinetic energy of the Roe velocity, term by term:
// no cancellation).  Estimates of 1/sqrt(rho) give the specific volumes and the
// Roe weights, one of 1/(m_L - m_R) gives a_L and a_R, one of
// 1/((S_L - S*)(S_R - S*)) the other two quotients.  Nothing here is of a higher
// order than rho c^3 or c^2, so any state whose fluxes are finite goes through
// (with 1/sqrt(rho_L rho_R) and one common reciprocal of order rho^3 c^5, a step
// took 1 to 2% less -- 1024^2 182 us against 186, 128^3 774 against 782 -- and
// every flux was NaN beyond about 1e100).
// About 125 operations and 8 estimates, where the component-wise wave sum with
// two-step Newton refinements took 230 and 11.
template <int NV, bool LOW_MACH = false>
__device__ __forceinline__ void hllc_n(const double* WL, const double* WR, const double* Fm,
                                       double fs, double gamma, double g1inv, double* F) {
  const double rl = WL[0], ul = WL[1], pl = WL[NV - 1];
  const double rr = WR[0], ur = WR[1], pr = WR[NV - 1];
  const double yl = rsq_c3(rl), yr = rsq_c3(rr);
  const double al = gamma * pl * (yl * yl), ar = gamma * pr * (yr * yr);   // c^2
  const double cl = sqrt_c3(al), cr = sqrt_c3(ar);
  const double t = rr * yr * yl;                        // sqrt(rho_R / rho_L)
  const double wl = rcp_c3(1.0 + t), wr = t * wl;
  const double du = ur - ul, dp = pr - pl;
  double kl = ul * ul, kr = ur * ur, dk = du * du;
#pragma unroll
  for (int i = 2; i < NV - 1; ++i) {
    const double dv = WR[i] - WL[i];
    kl += WL[i] * WL[i];
    kr += WR[i] * WR[i];
    dk += dv * dv;
  }
  const double ut = wl * ul + wr * ur;
  const double ct = sqrt_c3(wl * al + wr * ar + (0.5 * (gamma - 1.0)) * (wl * wr) * dk);
  const double SL = fmin(ul - cl, ut - ct);
  const double SR = fmax(ur + cr, ut + ct);
  const double bL = SL - ul, bR = SR - ur;
  const double ml = rl * bL, mr = rr * bR, rD = rcp_c3(ml - mr);
  const double aL = (dp - du * mr) * rD, aR = (dp - du * ml) * rD;
  const double Ss = ul + aL;
  const double xL = bL - aL, xR = bR - aR;              // S - S*
  const double z = rcp_c3(xL * xR);
  const double qL = aL * (z * xR), qR = aR * (z * xL);  // a / (S - S*)
  double phi = 1.0;
  if (LOW_MACH) {
    // |u| < c/10 on both sides is Ma < 0.1 (at the limit phi is 1 to rounding)
    if (fabs(ul) < 0.1 * cl && fabs(ur) < 0.1 * cr)
      phi = sin_quarter((0.5 * 3.14159265358979323846) *
                        (fmax(fabs(ul) / cl, fabs(ur) / cr) / 0.1));
  }
  const double aS = fabs(Ss);
  const double vL = LOW_MACH ? phi * fabs(SL) - aS : fabs(SL) - aS;
  const double vR = LOW_MACH ? phi * fabs(SR) - aS : fabs(SR) - aS;
  const double El = pl * g1inv + 0.5 * rl * kl;
  const double Er = pr * g1inv + 0.5 * rr * kr;
  const double hL = vL * qL, hR = vR * qR;
  const double GL = hL * rl, GR = hR * rr;
  const double d0 = (GL - GR) + aS * (rr - rl);
  const double d1 = (GL * SL - GR * SR) + aS * (rr * ur - rl * ul);
  const double dE = (hL * (El + pl + ml * Ss) - hR * (Er + pr + mr * Ss)) + aS * (Er - El);
  F[0] = fs * Fm[0] - 0.5 * d0;
  F[1] = fs * Fm[1] - 0.5 * d1;
#pragma unroll
  for (int i = 2; i < NV - 1; ++i)
    F[i] = fs * Fm[i] - 0.5 * ((GL * WL[i] - GR * WR[i]) + aS * (rr * WR[i] - rl * WL[i]));
  F[NV - 1] = fs * Fm[NV - 1] - 0.5 * dE;
}
template <bool LOW_MACH = false>
__device__ __forceinline__ void hllc(const double WL[4], const double WR[4], const double Fm[4],
                                     double gamma, double g1inv, double F[4]) {
  hllc_n<4, LOW_MACH>(WL, WR, Fm, 1.0, gamma, g1inv, F);
}

// Viscous interface flux (Sec. 2.1) added to F: normal derivatives of un,
// ut, T by alpha-damping (eq. eqn:alphad, alpha_v = 4) from the shared
// gradients, tangential derivatives and velocities as two-cell means.
// g* are spacing-scaled normal gradients, d*_t true tangential derivatives.
__device__ __forceinline__ void viscous_add(double un0, double un1, double ut0, double ut1,
                                            double T0, double T1, double gun0, double gun1,
                                            double gut0, double gut1, double gT0, double gT1,
                                            double dunt0, double dunt1, double dutt0,
                                            double dutt1, double inv_dn, double mu,
                                            double kq, double F[4]) {
  // dn * dPhi/dn at j+1/2 = (g0+g1)/2 + alpha_v/2 (Phi1 - g1/2 - Phi0 - g0/2)
  const double a2 = 0.5 * kAlphaV;
  const double dun = (0.5 * (gun0 + gun1) + a2 * (un1 - 0.5 * gun1 - un0 - 0.5 * gun0)) * inv_dn;
  const double dut = (0.5 * (gut0 + gut1) + a2 * (ut1 - 0.5 * gut1 - ut0 - 0.5 * gut0)) * inv_dn;
  const double dT = (0.5 * (gT0 + gT1) + a2 * (T1 - 0.5 * gT1 - T0 - 0.5 * gT0)) * inv_dn;
  const double dunt = 0.5 * (dunt0 + dunt1), dutt = 0.5 * (dutt0 + dutt1);
  const double unf = 0.5 * (un0 + un1), utf = 0.5 * (ut0 + ut1);
  const double tnn = (2.0 / 3.0) * mu * (2.0 * dun - dutt);
  const double tnt = mu * (dut + dunt);
  const double qn = -kq * dT;  // kq = mu / (Pr (gamma - 1))
  F[1] -= tnn;
  F[2] -= tnt;
  F[3] += -(tnn * unf + tnt * utf) + qn;
}

}  // namespace gbr
