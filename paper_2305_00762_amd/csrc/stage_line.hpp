// Line-streamed form of the fused MEG7 residual + SSP-RK3 stage: every 2D
// scheme but the MP test at every interface.
//
// One workgroup owns a TX x TY tile of cells.  The tile plus a 6-cell halo is
// staged in LDS (primitives, or conservative variables for MEG7-cons), and
// that is all LDS holds: no per-line gradient, edge-jump or flux buffer.  The
// interfaces of a line are cut into segments of K consecutive ones, one per
// lane; some waves take the x lines while others take the y lines.  A lane
// walks the K + 9 cells its interfaces' stencils span once, in registers: each
// cell's flux, its edge jump to the cell before and its density detector are
// formed as it passes and added into the K interfaces' running sums (GRB
// corrections, mean flux), so a cell is read from LDS (K + 9)/K times per
// interface, where a lane per interface reads 21 values per field.  Flagged
// interfaces are compacted within the wave (ballots, a wave's own queue), so
// nothing between the tile load and the exchange of the interface fluxes needs
// a block barrier.  The fluxes then go through LDS (over the tile) to the
// cells, which form the divergence and store the stage.
//
// F32 (FP32 bulk): the GRB corrections are summed and the Riemann solver runs
// in float32 on the jumps, U^L = U_j + cL, U^R = U_{j+1} + cR, U^R - U^L =
// dU + cR - cL, every wave jump a product of small quantities; flagged
// interfaces take float32 gradients and hold their flux's deviation from the
// central one in float32.  The mean flux, MP limiter, viscous flux and
// divergence are FP64.
//
// What bounds it: VALU issue on large grids (busy 83 to 88% at 4096^2 on 30x15
// tiles, 85% on the viscous 2048^2 field, K = 4); with few rounds of tiles also
// their tail and each wave's chain (1024^2 74%, 1283x719 viscous 75%, double Mach
// 1024x256 63%, 64^2 19%).  The barrier-phased form with per-line buffers before it
// issued 1.2 times the VALU and 2.8 times the LDS instructions, whose waits held
// it at 57%.  The 48 running sums of K = 4 fit 168 registers, 3 waves per SIMD;
// K = 8 does not.
// Measured per stage (events; that form -> this): Riemann 4096^2 15x15 FP64 1087
// -> 679 us, FP32 763 -> 617, 31x15 FP64 1259 -> 642; 1024^2 15x15 FP64 87 -> 62;
// viscous shear 2048^2 15x15 FP64 341 -> 239, FP32 251 -> 218, 31x15 406 -> 224,
// 333 -> 209; MEG7-cons tube 1280x640 83 -> 64.  Unphysical smooth states go
// through the same per-wave queue as flagged interfaces (kFirstOrder): their
// first-order fallback inline held registers and split every interface in
// blocks; a step of the 1280x640 MEG7-cons tube took 212 us with it, 193
// without (it spilled 24 registers, now 2), of 1024^2 FP64 186 and 183.
#pragma once
#include <type_traits>

#include "stage_kernel.hpp"

namespace gbr {

__device__ __forceinline__ float rcpf(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsqf(float x) { return __builtin_amdgcn_rsqf(x); }

// HLLC (Einfeldt bounds) dissipation |S_L|(Q*_L-Q_L) + |S*|(Q*_R-Q*_L) +
// |S_R|(Q_R-Q*_R) from the left/right primitive states and their jump
// dW = W_R - W_L, every jump evaluated as a product of small quantities.
__device__ __forceinline__ void hllc_diss_f32(const float WL[4], const float WR[4],
                                              const float dW[4], float gamma, float g1inv,
                                              float diss[4]) {
  const float rl = WL[0], ul = WL[1], vl = WL[2], pl = WL[3];
  const float rr = WR[0], ur = WR[1], vr = WR[2], pr = WR[3];
  const float dr = dW[0], du = dW[1], dv = dW[2], dp = dW[3];
  // 1/sqrt(rho) of each side gives the specific volumes and the Roe weights (an
  // estimate each: the product of the densities leaves float32's range above
  // 1.8e19 and below 1e-19); the Roe sound speed from the jumps, as in hllc_n
  const float yl = rsqf(rl), yr = rsqf(rr);
  const float kl2 = ul * ul + vl * vl, kr2 = ur * ur + vr * vr;
  const float El = pl * g1inv + 0.5f * rl * kl2;
  const float Er = pr * g1inv + 0.5f * rr * kr2;
  const float al = gamma * pl * (yl * yl), ar = gamma * pr * (yr * yr);
  const float t = rr * yr * yl;
  const float wl = rcpf(1.0f + t), wr = t * wl;
  const float ut = wl * ul + wr * ur;
  const float at = wl * al + wr * ar +
                   (0.5f * (gamma - 1.0f)) * (wl * wr) * (du * du + dv * dv);
  const float yt = rsqf(at);   // c = a / sqrt(a)
  const float SL = fminf(fmaf(-al, rsqf(al), ul), fmaf(-at, yt, ut));
  const float SR = fmaxf(fmaf(ar, rsqf(ar), ur), fmaf(at, yt, ut));
  const float ml = rl * (SL - ul), mr = rr * (SR - ur);
  const float iden = rcpf(ml - mr);
  const float aL = (dp - du * mr) * iden;   // S* - u_L
  const float aR = (dp - du * ml) * iden;   // S* - u_R
  const float Ss = ul + aL;
  const float iL = rcpf(SL - Ss), iR = rcpf(SR - Ss);
  // Q_R - Q_L from the primitive jumps
  const float dQ[4] = {dr, rr * du + ul * dr, rr * dv + vl * dr,
                       dp * g1inv + 0.5f * (dr * kl2 + rr * (du * (ur + ul) + dv * (vr + vl)))};
  const float aSL = fabsf(SL), aSS = fabsf(Ss), aSR = fabsf(SR);
  // |S_L| dQL + |S*| (dQ - dQR - dQL) + |S_R| dQR gathered per jump as
  // (|S_L| - |S*|) dQL + (|S_R| - |S*|) dQR + |S*| dQ, with
  //   dQL = Q*_L - Q_L = g_L (1, S_L, v_L, .),  g_L = rho_L a_L / (S_L - S*),
  //   dQR = Q_R - Q*_R = -g_R (1, S_R, v_R, .), g_R = rho_R a_R / (S_R - S*),
  // and the energy rows a_L/(S_L - S*) (E_L + p_L + m_L S*), resp. R
  const float aiL = aL * iL, aiR = aR * iR;
  const float wL = aSL - aSS, wR = aSR - aSS;
  const float GL = wL * (rl * aiL), GR = wR * (rr * aiR);
  const float HL = wL * aiL * (El + pl + ml * Ss), HR = wR * aiR * (Er + pr + mr * Ss);
  diss[0] = (GL - GR) + aSS * dQ[0];
  diss[1] = (GL * SL - GR * SR) + aSS * dQ[1];
  diss[2] = (GL * vl - GR * vr) + aSS * dQ[2];
  diss[3] = (HL - HR) + aSS * dQ[3];
}

// Queue bit of an interface whose smooth reconstruction is unphysical: it takes
// first-order states and their physical fluxes.
constexpr unsigned kFirstOrder = 0x8000u;

template <int TX_, int TY_, int K_, bool VISC_, int MINW_>
struct LineCfg {
  static constexpr int TX = TX_, TY = TY_, K = K_, H = 6, MINW = MINW_;
  static constexpr bool VISC = VISC_;
  static constexpr int RX = TX + 2 * H, RY = TY + 2 * H, RS = RX * RY;
  // segments per line, lanes and waves of the x and the y sweep
  static constexpr int SGX = (TX + K) / K, SGY = (TY + K) / K;
  static constexpr int WX = (TY * SGX + 63) / 64, WY = (TX * SGY + 63) / 64;
  static constexpr int NT = 64 * (WX + WY);
  // the last segment of a line of v cells walks to cell (v + K) / K * K + 3
  static constexpr bool inside(int n) {
    for (int v = 1; v <= n; ++v)
      if ((v + K) / K * K > n + 2) return false;
    return true;
  }
  static_assert(inside(TX) && inside(TY), "segments stay inside the halo");
  static constexpr int CPT = (TX * TY + NT - 1) / NT;
  // interface fluxes over the tile: x rows, then y rows, odd row strides
  static constexpr int FX = (TX + 1) | 1, FY = (TY + 1) | 1;
  static constexpr int FY0 = TY * FX;
  static_assert(FY0 + TX * FY <= RS, "interface fluxes fit the tile");
  // Cells staged: the tile's rows with their x halo, then the y halo over the
  // tile's columns; the corners are read by the viscous flux alone.
  static constexpr int NLOAD = VISC ? RS : TY * RX + 2 * H * TX;
  __device__ static __forceinline__ void cell(int c, int& lx, int& ly) {
    if (VISC || c < TY * RX) {
      ly = c / RX;
      lx = c - ly * RX - H;
      if (VISC) ly -= H;
    } else {
      c -= TY * RX;
      ly = c / TX;
      lx = c - ly * TX;
      ly += ly < H ? -H : TY - H;
    }
  }
  // queue entries: K lane + q, and kFirstOrder
  static constexpr int QN = 64 * K * (WX + WY);
  static constexpr int LDS_BYTES = 8 * 4 * RS + 2 * QN + 16;
};

// Integer stencil weights: GRB corrections on the edge jumps
// (pos+b-4)+1/2, b = 0..8 (eq. eqn:grb, or its fourth-order subset, with
// eq. eqn:six substituted, minus Phi_j resp. Phi_{j+1}), and the mean
// reconstructed flux on the cells pos-4+b, b = 0..9.
template <int ORD>
constexpr double grb_den() { return ORD == 4 ? 1440.0 : 840.0; }
template <int ORD>
constexpr double flux_den() { return ORD == 4 ? 2880.0 : 1680.0; }
template <int ORD>
constexpr double grb_wl(int b) {
  constexpr double w7[9] = {1, -1, -23, 123, 395, -89, 15, -1, 0};
  constexpr double w4[9] = {1, 4, -60, 249, 639, -132, 20, -1, 0};
  return ORD == 4 ? w4[b] : w7[b];
}
template <int ORD>
constexpr double grb_wr(int b) {   // the mirror image with the sign flipped
  return -grb_wl<ORD>(8 - b);
}
template <int ORD>
constexpr double flux_w(int b) {
  constexpr double w7[5] = {-1, 1, 38, -250, 1052};
  constexpr double w4[5] = {-1, -4, 85, -461, 1821};
  const int a = b < 5 ? b : 9 - b;
  return ORD == 4 ? w4[a] : w7[a];
}

// One sweep's share of a lane: the K interface fluxes (line, p0 .. p0 + K - 1),
// p = 0 the interface before the line's first cell, in the rotated frame.
template <class C, int DIR, bool DETMLP, bool CONS, int ORD, bool LM, bool F32>
struct LineSweep {
  using RT = typename std::conditional<F32, float, double>::type;
  static constexpr bool X = DIR == 0;
  static constexpr int K = C::K;
  static constexpr int RS = C::RS, RX = C::RX, H = C::H;
  static constexpr int SN = X ? 1 : RX, ST = X ? RX : 1;
  static constexpr int FN = X ? 1 : 2, FT = X ? 2 : 1;

  // The sweep's interfaces over the vx x vy cells of the tile inside the grid,
  // and lane t -> line and segment (consecutive lanes of the y sweep take
  // consecutive columns).  Lanes are dealt over these cells alone, so at the
  // grid's ragged edge the work fills fewer waves and the others skip it
  // (double Mach 1024x256, 4 and 1 cells over: 98.0 -> 95.3 us a step).
  int n, lanes;   // cells of a line, lanes with work
  int div;        // segments of a line (X), lines
  float inv;
  __device__ __forceinline__ LineSweep(int vx, int vy) {
    n = X ? vx : vy;
    const int nl = X ? vy : vx, sg = (n + K) / K;
    lanes = nl * sg;
    div = X ? sg : nl;
    inv = __builtin_amdgcn_rcpf((float)div);
  }
  __device__ __forceinline__ void lane(int t, int& line, int& seg) const {
    // floor(t / div) for t < 1024, div <= 64: (t + 1/2) / div is at least
    // 1/128 off a whole number
    const int q = (int)(((float)t + 0.5f) * inv), r = t - q * div;
    line = X ? q : r;
    seg = X ? r : q;
  }
  __device__ static __forceinline__ int ridx(int line, int pos) {
    const int lx = X ? pos : line, ly = X ? line : pos;
    return (ly + H) * RX + lx + H;
  }
  // rotated reconstructed variables of cell r: primitives, or (CONS) the
  // conservative ones
  __device__ static __forceinline__ void vars(const double* U, int r, double (&V)[4]) {
    V[0] = U[r];
    V[1] = U[FN * RS + r];
    V[2] = U[FT * RS + r];
    V[3] = U[3 * RS + r];
  }
  __device__ static __forceinline__ void prims(const double (&V)[4], double gamma, double (&W)[4]) {
    if (CONS) {
      const double ir = rcp_nr(V[0]);
      W[0] = V[0];
      W[1] = V[1] * ir;
      W[2] = V[2] * ir;
      W[3] = (gamma - 1.0) * (V[3] - 0.5 * V[0] * (W[1] * W[1] + W[2] * W[2]));
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m) W[m] = V[m];
    }
  }
  __device__ static __forceinline__ double g6(const double* u, int d) {
    return grad6(u[-3 * d], u[-2 * d], u[-d], u[d], u[2 * d], u[3 * d]);
  }
  static constexpr double gw(int b) {   // eq. (eqn:six) on the edge jumps, b = 0..5
    constexpr double w[6] = {1, -8, 37, 37, -8, 1};
    return w[b];
  }

  // Viscous flux of the lane's interfaces added to F, from a second walk over
  // the K + 7 cells the normal gradients span (T = gamma p / rho formed on the
  // way) and the tangential gradients of the K + 1 cells beside them.
  __device__ static __forceinline__ void viscous(const StageParams& P, const double* U, int r0,
                                                 double (&F)[K][4]) {
    const double inv_dn = X ? P.inv_dx : P.inv_dy, inv_dt = X ? P.inv_dy : P.inv_dx;
    constexpr int NG = CONS ? 4 : 3;   // gradients: (u_n, u_t, T) or (rho, rho u_n, rho u_t, T)
    double g[K + 1][NG], un[K + 1], ut[K + 1], ir[K + 1], jT[K], pv[NG];
#pragma unroll
    for (int c = 0; c < K + 7; ++c) {
      const int r = r0 + (c - 3) * SN;
      double V[4], W[4], G[NG];
      vars(U, r, V);
      prims(V, P.gamma, W);
      const double irc = rcp_nr(V[0]);
      const double T = P.gamma * W[3] * irc;
      if (CONS) { G[0] = V[0]; G[1] = V[1]; G[2] = V[2]; }
      else { G[0] = W[1]; G[1] = W[2]; }
      G[NG - 1] = T;
      if (c >= 3 && c <= K + 3) {
        un[c - 3] = W[1];
        ut[c - 3] = W[2];
        ir[c - 3] = irc;
      }
      if (c > 0) {
#pragma unroll
        for (int m = 0; m < NG; ++m) {
          const double e = G[m] - pv[m];   // edge c - 1: cells c - 1, c
          if (m == NG - 1 && c >= 4 && c <= K + 3) jT[c - 4] = e;
#pragma unroll
          for (int k = 0; k <= K; ++k) {
            const int b = c - 1 - k;
            if (b == 0) g[k][m] = e;
            if (b > 0 && b < 6) g[k][m] += gw(b) * e;
          }
        }
      }
#pragma unroll
      for (int m = 0; m < NG; ++m) pv[m] = G[m];
      if (CONS) {   // MEG7-prim fits the budget without (and runs faster)
#pragma unroll
        for (int k = 0; k <= K; ++k)
#pragma unroll
          for (int m = 0; m < NG; ++m)
            if (c > k && c <= k + 6) pin(g[k][m]);
        hold();
      }
    }
    constexpr double z = 1.0 / 60.0;
    double dn[2], dt[2], gn[2], gt[2];   // tangential and normal derivatives at the two cells
    auto cell = [&](int k, int s) {
      const int r = r0 + k * SN;
      if (CONS) {
        // velocity gradients by the chain rule d u = (d(rho u) - u d rho) / rho
        const double tr = g6(U + r, ST) * inv_dt;
        dn[s] = (g6(U + FN * RS + r, ST) * inv_dt - un[k] * tr) * ir[k];
        dt[s] = (g6(U + FT * RS + r, ST) * inv_dt - ut[k] * tr) * ir[k];
        gn[s] = z * (g[k][1] - un[k] * g[k][0]) * ir[k];
        gt[s] = z * (g[k][2] - ut[k] * g[k][0]) * ir[k];
      } else {
        dn[s] = g6(U + FN * RS + r, ST) * inv_dt;
        dt[s] = g6(U + FT * RS + r, ST) * inv_dt;
        gn[s] = z * g[k][0];
        gt[s] = z * g[k][1];
      }
    };
    cell(0, 0);
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const int a = q & 1, b = a ^ 1;
      cell(q + 1, b);
      viscous_add(un[q], un[q + 1], ut[q], ut[q + 1], 0.0, jT[q], gn[a], gn[b], gt[a], gt[b],
                  z * g[q][NG - 1], z * g[q + 1][NG - 1], dn[a], dn[b], dt[a], dt[b], inv_dn,
                  P.mu, P.kq, F[q]);
      if (CONS) hold();
    }
  }

  // Flux of the interface right of cell r outside the smooth branch: the
  // characteristic MEG7 states (Secs. 2.3, 2.4) from the cells r - 5 .. r + 6,
  // or the two cells' states where those are unphysical or first is set.
  __device__ static __forceinline__ void flagged(const StageParams& P, const double* U, int r,
                                                 bool first, double (&F)[4]) {
    double WL[4], WR[4];
    constexpr int rot[4] = {0, FN, FT, 3};
    auto Vc = [&](int k, int f) { return U[rot[f] * RS + r + (k - 5) * SN]; };
    WL[0] = -1.0;
    if (!first) {
      if (CONS) {
        double QL[4], QR[4];
        meg7_char_states_cons_cells<ORD>(Vc, P.gamma, QL, QR);
        cons_to_prim(QL, P.gamma, WL);
        cons_to_prim(QR, P.gamma, WR);
      } else {
        meg7_char_states_cells<4, ORD, F32>(Vc, P.gamma, WL, WR);
      }
    }
    if (!(WL[0] > 0.0 && WL[3] > 0.0 && WR[0] > 0.0 && WR[3] > 0.0)) {
      double V[4];
      vars(U, r, V);
      prims(V, P.gamma, WL);
      vars(U, r + SN, V);
      prims(V, P.gamma, WR);
    }
    double FL[4], FR[4], Fm[4];
    conv_flux(WL, P.g1inv, FL);
    conv_flux(WR, P.g1inv, FR);
#pragma unroll
    for (int m = 0; m < 4; ++m) Fm[m] = FL[m] + FR[m];
    hllc_n<4, LM>(WL, WR, Fm, 0.5, P.gamma, P.g1inv, F);
    if (F32) {
      // the deviation from the central flux is held in float32
      double V0[4], V1[4];
      vars(U, r, V0);
      vars(U, r + SN, V1);
      conv_flux(V0, P.g1inv, FL);
      conv_flux(V1, P.g1inv, FR);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const double B = 0.5 * (FL[m] + FR[m]);
        F[m] = B + (double)(float)(F[m] - B);
      }
    }
  }

  // Fluxes of the lanes of one of the sweep's waves; queue: this wave's.
  // Returns whether the lane has interfaces of the tile.
  __device__ __forceinline__ bool run(const StageParams& P, const double* U,
                                      unsigned short* queue, const unsigned char* chif, int wave,
                                      int tx0, int ty0, double (&F)[K][4], int& line,
                                      int& p0) const {
    const int lid = threadIdx.x & 63, wave0 = 64 * wave, t = wave0 + lid;
    if (wave0 >= lanes) return false;
    int seg;
    lane(t, line, seg);
    const bool act = t < lanes;
    if (!act) line = seg = 0;
    p0 = seg * K;
    const int j0 = p0 - 1;                  // left cell of the first interface
    const int r0 = ridx(line, j0);

    // ---- the walk over cells j0 - 4 .. j0 + K + 4 --------------------------
    double Fm[K][4], pv[4], rw[5], re[3], nv[4];
    RT cL[K][4], cR[K][4];
    bool flag[K], first[K];
    vars(U, r0 - 4 * SN, nv);
#pragma unroll
    for (int q = 0; q < K; ++q) flag[q] = false;
#pragma unroll
    for (int c = 0; c < K + 9; ++c) {
      double V[4], W[4], f[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) V[m] = nv[m];
      if (c + 1 < K + 9) vars(U, r0 + (c - 3) * SN, nv);
      hold();
      prims(V, P.gamma, W);
      conv_flux(W, P.g1inv, f);
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const int b = c - q;
        if (b < 0 || b > 9) continue;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if (b == 0) Fm[q][m] = flux_w<ORD>(0) * f[m];
          else Fm[q][m] += flux_w<ORD>(b) * f[m];
        }
      }
      if (c > 0) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const RT e = (RT)(V[m] - pv[m]);    // edge jump c - 1
#pragma unroll
          for (int q = 0; q < K; ++q) {
            const int b = c - 1 - q;
            if (b == 0) cL[q][m] = (RT)grb_wl<ORD>(0) * e;
            if (b > 0 && b < 8) cL[q][m] += (RT)grb_wl<ORD>(b) * e;
            if (b == 1) cR[q][m] = (RT)grb_wr<ORD>(1) * e;
            if (b > 1 && b < 9) cR[q][m] += (RT)grb_wr<ORD>(b) * e;
          }
        }
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) pv[m] = V[m];
      if (!DETMLP) {
#pragma unroll
        for (int a = 0; a < 4; ++a) rw[a] = rw[a + 1];
        rw[4] = V[0];
        re[0] = re[1];
        re[1] = re[2];
        re[2] = rw[4] - rw[3];
      }
      if (c >= 4) {
        // the detector at cell j0 + o feeds the interfaces q with o in [q-2, q+3]
        const int o = c - 6;
        bool chi;
        if (DETMLP)
          chi = (chif[mlp_chi_index<C>(X ? j0 + o : line, X ? line : j0 + o)] >> DIR) & 1;
        else
          chi = detector_flag_jumps(rw[0], rw[1], rw[2], rw[3], rw[4], re[0], re[1]);
#pragma unroll
        for (int q = 0; q < K; ++q)
          if (o >= q - 2 && o <= q + 3) flag[q] = flag[q] | chi;
      }
#pragma unroll
      for (int q = 0; q < K; ++q)
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if (c >= q && c <= q + 9) pin(Fm[q][m]);
          if (c > q && c <= q + 8) pin(cL[q][m]);
          if (c > q + 1 && c <= q + 9) pin(cR[q][m]);
        }
      hold();
    }

    // ---- smooth interfaces -------------------------------------------------
    double VL[4], VR[4];
    vars(U, r0, VL);
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const bool in = act && p0 + q <= n;
      if (X) {
        const int gi = ty0 + line, gj = tx0 + j0 + q;
        if (P.sigx && in && gi < P.ny && gj < P.nx)
          P.sigx[(size_t)gi * (P.nx + 1) + gj + 1] = !flag[q];
      } else {
        const int gj = tx0 + line, gi = ty0 + j0 + q;
        if (P.sigy && in && gj < P.nx && gi < P.ny)
          P.sigy[(size_t)(gi + 1) * P.nx + gj] = !flag[q];
      }
      vars(U, r0 + (q + 1) * SN, VR);
      bool ok;
      constexpr double fs = 1.0 / flux_den<ORD>();
      if constexpr (F32) {
        float WL[4], WR[4], dW[4], diss[4];
        constexpr float s = (float)(1.0 / grb_den<ORD>());
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const float e = (float)(VR[m] - VL[m]);
          WL[m] = (float)VL[m] + s * cL[q][m];
          WR[m] = (float)VR[m] + s * cR[q][m];
          dW[m] = e + s * (cR[q][m] - cL[q][m]);
        }
        ok = WL[0] > 0.f && WL[3] > 0.f && WR[0] > 0.f && WR[3] > 0.f;
        hllc_diss_f32(WL, WR, dW, (float)P.gamma, (float)P.g1inv, diss);
#pragma unroll
        for (int m = 0; m < 4; ++m) F[q][m] = fs * Fm[q][m] - (double)(0.5f * diss[m]);
      } else {
        double WL[4], WR[4];
        constexpr double s = 1.0 / grb_den<ORD>();
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          WL[m] = VL[m] + s * cL[q][m];
          WR[m] = VR[m] + s * cR[q][m];
        }
        if (CONS) {
          const double QL[4] = {WL[0], WL[1], WL[2], WL[3]};
          const double QR[4] = {WR[0], WR[1], WR[2], WR[3]};
          cons_to_prim(QL, P.gamma, WL);
          cons_to_prim(QR, P.gamma, WR);
        }
        ok = WL[0] > 0.0 && WL[3] > 0.0 && WR[0] > 0.0 && WR[3] > 0.0;
        hllc_n<4, LM>(WL, WR, Fm[q], fs, P.gamma, P.g1inv, F[q]);
      }
      // an unphysical reconstruction joins the queue for first-order states
      first[q] = in && !flag[q] && !ok;
      flag[q] = in && (flag[q] || !ok);
#pragma unroll
      for (int m = 0; m < 4; ++m) pin(F[q][m]);
#pragma unroll
      for (int m = 0; m < 4; ++m) VL[m] = VR[m];
      hold();
    }

    // ---- interfaces outside the smooth branch, compacted within the wave ----
    int slot[K], nq = 0;
    const unsigned long long below = (1ull << lid) - 1ull;
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const unsigned long long ball = __ballot(flag[q]);
      slot[q] = nq + (int)__popcll(ball & below);
      nq += (int)__popcll(ball);
    }
    if (nq) {
#pragma unroll
      for (int q = 0; q < K; ++q)
        if (flag[q])
          queue[slot[q]] = (unsigned short)((lid * K + q) | (first[q] ? kFirstOrder : 0u));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
      for (int base = 0; base < nq; base += 64) {
        double G[4] = {0.0, 0.0, 0.0, 0.0};
        if (base + lid < nq) {
          const unsigned code = queue[base + lid];
          const int e = code & (kFirstOrder - 1);
          int ln, sg;
          lane(wave0 + e / K, ln, sg);
          flagged(P, U, ridx(ln, sg * K + e % K - 1), (code & kFirstOrder) != 0, G);
        }
        // each flux back to the lane that owns the interface
#pragma unroll
        for (int q = 0; q < K; ++q) {
          const int src = slot[q] - base;
          const bool mine = flag[q] && src >= 0 && src < 64;
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const double v = __shfl(G[m], src & 63);
            if (mine) F[q][m] = v;
          }
        }
      }
    }
    if (C::VISC) viscous(P, U, r0, F);
    return act;
  }
};

// One tile of the stage.  sU: [4][RS]; queue: C::QN entries.
template <class C, bool DETMLP, bool CONS, int ORD, bool LM, bool F32>
__device__ __forceinline__ void stage_tile_line(const StageParams& P, int tx0, int ty0, double* sU,
                                                unsigned short* queue, unsigned char* sChiF) {
  constexpr int RS = C::RS, K = C::K;
  ChiMap<C> cm;
  if (DETMLP) fetch_chimap<C>(P, cm, tx0, ty0);
  stage_load<C, CONS, false>(P, sU, tx0, ty0);
  if (DETMLP) put_chimap<C>(cm, sChiF);
  __syncthreads();
  double F[K][4];
  int line, p0;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int vx = min(C::TX, P.nx - tx0), vy = min(C::TY, P.ny - ty0);
  const LineSweep<C, 0, DETMLP, CONS, ORD, LM, F32> sx(vx, vy);
  const LineSweep<C, 1, DETMLP, CONS, ORD, LM, F32> sy(vx, vy);
  bool act;
  if (wave < C::WX)
    act = sx.run(P, sU, queue + 64 * K * wave, sChiF, wave, tx0, ty0, F, line, p0);
  else
    act = sy.run(P, sU, queue + 64 * K * wave, sChiF, wave - C::WX, tx0, ty0, F, line, p0);
  __syncthreads();   // every read of the tile is done: it becomes the flux buffer
  {
    const bool xw = wave < C::WX;
    const int N = xw ? sx.n : sy.n;
    double* f = sU + (xw ? line * C::FX : C::FY0 + line * C::FY) + p0;
#pragma unroll
    for (int q = 0; q < K; ++q)
      if (act && p0 + q <= N) {
#pragma unroll
        for (int m = 0; m < 4; ++m) f[m * RS + q] = F[q][m];
      }
  }
  __syncthreads();
  double res[C::CPT][4];
#pragma unroll
  for (int k = 0; k < C::CPT; ++k) {
    int lx, ly;
    if (!tile_cell<C>(tid, k, lx, ly)) continue;
    const double* fx = sU + ly * C::FX + lx;
    const double* fy = sU + C::FY0 + lx * C::FY + ly;
    constexpr int my[4] = {0, 2, 1, 3};   // rotated component of the y fluxes
#pragma unroll
    for (int m = 0; m < 4; ++m)
      res[k][m] = -((fx[m * RS + 1] - fx[m * RS]) * P.inv_dx) -
                  (fy[my[m] * RS + 1] - fy[my[m] * RS]) * P.inv_dy;
  }
  stage_store<C>(P, res, tx0, ty0);
}

template <class C, bool DETMLP, bool CONS, int ORD, bool LM, bool F32 = false>
__global__ __launch_bounds__(C::NT, C::MINW) void meg7_line_kernel(StageParams P) {
  __shared__ double sU[4 * C::RS];
  __shared__ unsigned short sQueue[C::QN];
  __shared__ unsigned char sChiF[DETMLP ? (C::TX + 6) * (C::TY + 6) : 1];
  int tx0, ty0;
  if (!tile_origin(P, C::TX, C::TY, tx0, ty0)) return;
  stage_tile_line<C, DETMLP, CONS, ORD, LM, F32>(P, tx0, ty0, sU, sQueue, sChiF);
}

}  // namespace gbr
