// MEG7 in three dimensions (the Euler equations, inviscid) for gfx950.
//
// The method is applied dimension by dimension, in a frame rotated to the line,
// (rho, u_n, u_t1, u_t2, p) with the tangential components taken cyclically
// (x: v, w; y: w, u; z: u, v).  A stage is two kernels of the line-streamed form
// (stage_line.hpp: a lane owns K consecutive interfaces of a line and walks the
// K + 9 cells they span once, in registers, from an LDS tile of primitives):
//   plane: tiles of a z plane (15x15, 16x16 or 20x17) with a 6-cell halo in x
//          and y, x lines and y lines on different waves at the same time;
//          writes the residual accumulator R = -dF/dx - dG/dy (40 B per cell
//          read, 40 written);
//   column: kCol3W consecutive cells of the xy plane x 15 cells along z with the
//          halo along z; adds -dH/dz and stores the residual or the SSP-RK3
//          stage (eq. rk).
// The octant Riemann field of 128^3, where 14% of the interfaces take the shock
// branch, takes 151 us in the plane kernel (158 with 15x15 tiles and two interfaces
// a lane) and 92 in the column kernel (98 with 32 lines); 163 and 105 on average
// over a run.  Neither a unit nor memory is saturated there: VALU is busy 65% and
// 61%, HBM traffic 161 and 324 MiB a launch (profiled: 177 and 119 us).  The plane
// kernel's x sweep pays for its row stride of 32 doubles on 20x17 tiles: 4.5 bank
// conflict cycles per LDS instruction, against 1.3 on the 16x16 tiles of 64^3.  One
// barrier-phased kernel per direction, with staged gradients and fluxes in LDS,
// took 126 + 141 + 159 us on that field.
#pragma once
#include "dt_kernel_common.hpp"
#include "meg7_device.hpp"
#include "stage3d_params.hpp"
#include "stage_line.hpp"

namespace gbr {

// |u|+c, |v|+c, |w|+c of one cell of the new state, each rounded as the
// time-step kernel rounds them (IEEE division and square root, one rounding
// per operation; the quotients share one refined reciprocal where div_rb gives
// the IEEE quotient), folded into (ea, eb, ec); since fl(d/x) is monotone in
// x, the minima of the per-cell limits follow from the maxima without loss.
__device__ __forceinline__ void dt3_extrema_cell(const double q[5], double gamma, double& ea,
                                                 double& eb, double& ec, bool& bad) {
#pragma clang fp contract(off)
  const double rho = q[0], rb = rcp_nr(rho);
  const bool fast = rho != 0.0 && div_rb_ok(rho) && div_rb_ok(q[1]) && div_rb_ok(q[2]) &&
                    div_rb_ok(q[3]);
  double u, v, w;
  if (fast) {
    u = div_rb(q[1], rho, rb);
    v = div_rb(q[2], rho, rb);
    w = div_rb(q[3], rho, rb);
  } else {
    u = q[1] / rho;
    v = q[2] / rho;
    w = q[3] / rho;
  }
  const double p = (gamma - 1.0) * (q[4] - rho * (u * u + v * v + w * w) / 2.0);
  const double gp = gamma * p;
  const double c = sqrt((fast && div_rb_ok(gp)) ? div_rb(gp, rho, rb) : gp / rho);
  if (!(rho > 0.0) || !(p > 0.0) || !isfinite(c) || !isfinite(u) || !isfinite(v) ||
      !isfinite(w))
    bad = true;
  ea = fmax(ea, fabs(u) + c);
  eb = fmax(eb, fabs(v) + c);
  ec = fmax(ec, fabs(w) + c);
}

// Normal convective flux of W = (rho, u_n, u_t1, u_t2, p).
__device__ __forceinline__ void conv_flux3(const double W[5], double g1inv, double F[5]) {
  const double E = W[4] * g1inv + 0.5 * W[0] * (W[1] * W[1] + W[2] * W[2] + W[3] * W[3]);
  const double m = W[0] * W[1];
  F[0] = m;
  F[1] = m * W[1] + W[4];
  F[2] = m * W[2];
  F[3] = m * W[3];
  F[4] = W[1] * (E + W[4]);
}

// A lane's walk: fluxes F of its K interfaces from the tile U (five planes of
// RS), the first one right of cell r0, cells SN apart along the line; DIR sets
// the rotation.  rof(t): r0 of lane t of the wave; queue: this wave's; valid:
// how many of the K interfaces exist.  All 64 lanes of the wave call it.
// Returns the flags, bit q set where the detector flags interface q.
template <int DIR, int K, int RS, int SN, int ORD, class RO>
__device__ __forceinline__ unsigned walk3(const double* U, double gamma, double g1inv,
                                          unsigned short* queue, int r0, int valid, RO rof,
                                          double (&F)[K][5]) {
  const int lid = threadIdx.x & 63;
  constexpr int rot[5] = {0, 1 + DIR % 3, 1 + (DIR + 1) % 3, 1 + (DIR + 2) % 3, 4};
  auto vars = [&](int r, double (&V)[5]) {
#pragma unroll
    for (int m = 0; m < 5; ++m) V[m] = U[rot[m] * RS + r];
  };
  double Fm[K][5], cL[K][5], cR[K][5], pv[5], rw[5], re[3], nv[5];
  bool flag[K], first[K];
  unsigned bits = 0;
#pragma unroll
  for (int q = 0; q < K; ++q) flag[q] = false;
  vars(r0 - 4 * SN, nv);
#pragma unroll
  for (int c = 0; c < K + 9; ++c) {
    double V[5], f[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) V[m] = nv[m];
    if (c + 1 < K + 9) vars(r0 + (c - 3) * SN, nv);
    hold();
    conv_flux3(V, g1inv, f);
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const int b = c - q;
      if (b < 0 || b > 9) continue;
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        if (b == 0) Fm[q][m] = flux_w<ORD>(0) * f[m];
        else Fm[q][m] += flux_w<ORD>(b) * f[m];
      }
    }
    if (c > 0) {
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        const double e = V[m] - pv[m];
#pragma unroll
        for (int q = 0; q < K; ++q) {
          const int b = c - 1 - q;
          if (b == 0) cL[q][m] = grb_wl<ORD>(0) * e;
          if (b > 0 && b < 8) cL[q][m] += grb_wl<ORD>(b) * e;
          if (b == 1) cR[q][m] = grb_wr<ORD>(1) * e;
          if (b > 1 && b < 9) cR[q][m] += grb_wr<ORD>(b) * e;
        }
      }
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) pv[m] = V[m];
#pragma unroll
    for (int a = 0; a < 4; ++a) rw[a] = rw[a + 1];
    rw[4] = V[0];
    re[0] = re[1];
    re[1] = re[2];
    re[2] = rw[4] - rw[3];
    if (c >= 4) {
      // the detector at cell r0 + (c - 6) SN feeds the interfaces within reach
      const int o = c - 6;
      const bool chi = detector_flag_jumps(rw[0], rw[1], rw[2], rw[3], rw[4], re[0], re[1]);
#pragma unroll
      for (int q = 0; q < K; ++q)
        if (o >= q - 2 && o <= q + 3) flag[q] = flag[q] | chi;
    }
#pragma unroll
    for (int q = 0; q < K; ++q)
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        if (c >= q && c <= q + 9) pin(Fm[q][m]);
        if (c > q && c <= q + 8) pin(cL[q][m]);
        if (c > q + 1 && c <= q + 9) pin(cR[q][m]);
      }
    hold();
  }

  // smooth interfaces
  double VL[5], VR[5];
  vars(r0, VL);
#pragma unroll
  for (int q = 0; q < K; ++q) {
    vars(r0 + (q + 1) * SN, VR);
    double WL[5], WR[5];
    constexpr double s = 1.0 / grb_den<ORD>(), fs = 1.0 / flux_den<ORD>();
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      WL[m] = VL[m] + s * cL[q][m];
      WR[m] = VR[m] + s * cR[q][m];
    }
    // an unphysical reconstruction joins the queue for first-order states
    const bool ok = WL[0] > 0.0 && WL[4] > 0.0 && WR[0] > 0.0 && WR[4] > 0.0;
    hllc_n<5>(WL, WR, Fm[q], fs, gamma, g1inv, F[q]);
#pragma unroll
    for (int m = 0; m < 5; ++m) pin(F[q][m]);
#pragma unroll
    for (int m = 0; m < 5; ++m) VL[m] = VR[m];
    if (flag[q] && q < valid) bits |= 1u << q;
    first[q] = q < valid && !flag[q] && !ok;
    flag[q] = q < valid && (flag[q] || !ok);
    hold();
  }

  // interfaces outside the smooth branch, compacted within the wave
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
      double G[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
      if (base + lid < nq) {
        const unsigned code = queue[base + lid];
        const int e = code & (kFirstOrder - 1);
        const int r = rof(e / K) + (e % K) * SN;
        double WL[5], WR[5], FL[5], FR[5];
        WL[0] = -1.0;
        if (!(code & kFirstOrder))
          meg7_char_states_cells<5, ORD, false>(
              [&](int k, int f) { return U[rot[f] * RS + r + (k - 5) * SN]; }, gamma, WL, WR);
        if (!(WL[0] > 0.0 && WL[4] > 0.0 && WR[0] > 0.0 && WR[4] > 0.0)) {
          vars(r, WL);
          vars(r + SN, WR);
        }
        conv_flux3(WL, g1inv, FL);
        conv_flux3(WR, g1inv, FR);
#pragma unroll
        for (int m = 0; m < 5; ++m) FL[m] += FR[m];
        hllc_n<5>(WL, WR, FL, 0.5, gamma, g1inv, G);
      }
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const int src = slot[q] - base;
        const bool mine = flag[q] && src >= 0 && src < 64;
#pragma unroll
        for (int m = 0; m < 5; ++m) {
          const double v = __shfl(G[m], src & 63);
          if (mine) F[q][m] = v;
        }
      }
    }
  }
  return bits;
}

// Primitives of a conserved cell to the tile.
template <int RS>
__device__ __forceinline__ bool put3(double* sU, int c, const double q[5], double gamma) {
  const double r = q[0], ir = rcp_nr(r);
  const double u = q[1] * ir, v = q[2] * ir, w = q[3] * ir;
  const double p = (gamma - 1.0) * (q[4] - 0.5 * r * (u * u + v * v + w * w));
  sU[c] = r;
  sU[RS + c] = u;
  sU[2 * RS + c] = v;
  sU[3 * RS + c] = w;
  sU[4 * RS + c] = p;
  return r > 0.0 && p > 0.0 && isfinite(q[4]) && isfinite(u) && isfinite(v) && isfinite(w);
}

// Contiguous runs of tiles per XCD, as in the 2D kernels.
__device__ __forceinline__ int tile3() {
  const int b = blockIdx.x, nb = gridDim.x;
  const int xcd = b & 7, per = nb >> 3, rem = nb & 7;
  return xcd * per + (xcd < rem ? xcd : rem) + (b >> 3);
}

// ---------------------------------------------------------------------------
// x and y lines of a z plane.
template <class C, int ORD>
__global__ __launch_bounds__(C::NT, C::MINW) void meg7_plane3_kernel(Stage3Params P) {
  constexpr int RS = C::RS, RX = C::RX, H = C::H, NT = C::NT, K = C::K, TX = C::TX, TY = C::TY;
  __shared__ double sU[5 * RS];
  __shared__ unsigned short sQueue[C::QN];
  const int tile = tile3();
  if (tile >= P.ntiles) return;
  const int tpp = P.tiles_x * P.tiles_y;
  const int z = tile / tpp, tp = tile - z * tpp;
  const int tx0 = (tp % P.tiles_x) * TX, ty0 = (tp / P.tiles_x) * TY;
  const size_t n = (size_t)P.nx * P.ny * P.nz;
  const size_t zb = (size_t)z * P.ny * P.nx;
  const int tid = threadIdx.x;

  // tile and halo: all loads issued before any is consumed
  {
    constexpr int LR = (C::NLOAD + NT - 1) / NT;
    double q[LR][5];
    int o[LR];
    cell_offsets<C, LR>(P.nx, P.ny, P.bc[0], P.bc[1], tx0, ty0, o);
#pragma unroll
    for (int k = 0; k < LR; ++k)
      if (tid + k * NT < C::NLOAD) {
#pragma unroll
        for (int m = 0; m < 5; ++m) q[k][m] = P.Qk[m * n + zb + o[k]];
      }
    bool bad = false;
#pragma unroll
    for (int k = 0; k < LR; ++k) {
      const int c = tid + k * NT;
      if (c < C::NLOAD) {
        int lx, ly;
        C::cell(c, lx, ly);
        const bool ok = put3<RS>(sU, (ly + H) * RX + lx + H, q[k], P.gamma);
        if (!ok && lx >= 0 && lx < TX && ly >= 0 && ly < TY && tx0 + lx < P.nx && ty0 + ly < P.ny)
          bad = true;
      }
    }
    if (bad) atomicOr(P.status, STATUS_BAD_STATE);
  }
  __syncthreads();

  double F[K][5];
  int line, seg;
  bool act = false;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned short* queue = sQueue + 64 * K * wave;
  auto sweep = [&](auto dir) {
    using L = LineSweep<C, decltype(dir)::value, false, false, ORD, false, false>;
    const L sw(min(TX, P.nx - tx0), min(TY, P.ny - ty0));
    const int wave0 = 64 * (wave - (L::X ? 0 : C::WX)), t = wave0 + (tid & 63);
    act = t < sw.lanes;
    if (wave0 >= sw.lanes) return;
    sw.lane(t, line, seg);
    if (!act) line = seg = 0;
    const int p0 = seg * K;
    const int valid = act ? (sw.n + 1 - p0 < K ? sw.n + 1 - p0 : K) : 0;
    const unsigned bits = walk3<decltype(dir)::value, K, RS, L::SN, ORD>(
        sU, P.gamma, P.g1inv, queue, L::ridx(line, p0 - 1), valid,
        [&](int e) {
          int ln, sg;
          sw.lane(wave0 + e, ln, sg);
          return L::ridx(ln, sg * K - 1);
        },
        F);
    if (P.sig[decltype(dir)::value]) {
      for (int q = 0; q < valid; ++q) {
        const uint8_t sigma = !((bits >> q) & 1u);
        if (L::X) {
          const int gy = ty0 + line, gi = tx0 + p0 + q;
          if (gy < P.ny && gi <= P.nx)
            P.sig[0][((size_t)z * P.ny + gy) * (P.nx + 1) + gi] = sigma;
        } else {
          const int gx = tx0 + line, gi = ty0 + p0 + q;
          if (gx < P.nx && gi <= P.ny)
            P.sig[1][((size_t)z * (P.ny + 1) + gi) * P.nx + gx] = sigma;
        }
      }
    }
  };
  if (wave < C::WX) sweep(std::integral_constant<int, 0>());
  else sweep(std::integral_constant<int, 1>());
  __syncthreads();   // every read of the tile is done: it becomes the flux buffer
  {
    const bool xw = wave < C::WX;
    const int N = xw ? min(TX, P.nx - tx0) : min(TY, P.ny - ty0);
    double* f = sU + (xw ? line * C::FX : C::FY0 + line * C::FY) + seg * K;
#pragma unroll
    for (int q = 0; q < K; ++q)
      if (act && seg * K + q <= N) {
#pragma unroll
        for (int m = 0; m < 5; ++m) f[m * RS + q] = F[q][m];
      }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < C::CPT; ++k) {
    int lx, ly;
    const bool in = tile_cell<C>(tid, k, lx, ly);
    if (!in || tx0 + lx >= P.nx || ty0 + ly >= P.ny) continue;
    const double* fx = sU + ly * C::FX + lx;
    const double* fy = sU + C::FY0 + lx * C::FY + ly;
    const size_t s = zb + (size_t)(ty0 + ly) * P.nx + tx0 + lx;
    constexpr int my[5] = {0, 3, 1, 2, 4};   // rotated component of the y fluxes
#pragma unroll
    for (int m = 0; m < 5; ++m)
      P.R[m * n + s] = -((fx[m * RS + 1] - fx[m * RS]) * P.inv_d[0]) -
                       (fy[my[m] * RS + 1] - fy[my[m] * RS]) * P.inv_d[1];
  }
}

// ---------------------------------------------------------------------------
// z lines: W consecutive cells of the xy plane (lines) x TZ cells along z.
// Lanes run across the lines, so every LDS access is W consecutive doubles.
template <int W_, int TZ_, int K_, int MINW_>
struct Col3Cfg {
  static constexpr int W = W_, TZ = TZ_, K = K_, MINW = MINW_, H = 6;
  static constexpr int RZ = TZ + 2 * H, RS = RZ * W;
  static constexpr int SG = (TZ + K) / K;
  static_assert(SG * K <= TZ + 2, "segments stay inside the halo");
  static constexpr int NT = SG * W;
  static_assert(NT % 64 == 0, "whole waves");
};

template <class C, int ORD>
__global__ __launch_bounds__(C::NT, C::MINW) void meg7_col3_kernel(Stage3Params P) {
  constexpr int RS = C::RS, W = C::W, TZ = C::TZ, H = C::H, NT = C::NT, K = C::K;
  __shared__ double sU[5 * RS];
  __shared__ unsigned short sQueue[C::NT * K];
  const int tile = tile3();
  if (tile >= P.ntiles) return;
  // z tiles of one column group run one after the other on an XCD: they share
  // their halo planes in its L2
  const int tz = tile % P.tiles_z, g0 = tile / P.tiles_z * W;
  const int z0 = tz * TZ;
  const int nl = P.nx * P.ny;
  const size_t n = (size_t)nl * P.nz;
  const int tid = threadIdx.x;
  const int l = tid % W;                     // NT is a multiple of W: a fixed line per lane
  const int gl = g0 + l < nl ? g0 + l : nl - 1;
  {
    constexpr int LR = (C::RZ * W + NT - 1) / NT;
    const bool wide = P.nz >= TZ + H;
    double q[LR][5];
#pragma unroll
    for (int k = 0; k < LR; ++k) {
      const int c = tid + k * NT, p = c / W;
      if (p < C::RZ) {
        const size_t s = (size_t)(wide ? bc_index1(z0 + p - H, P.nz, P.bc[2])
                                       : bc_index(z0 + p - H, P.nz, P.bc[2])) * nl + gl;
#pragma unroll
        for (int m = 0; m < 5; ++m) q[k][m] = P.Qk[m * n + s];
      }
    }
#pragma unroll
    for (int k = 0; k < LR; ++k) {
      const int c = tid + k * NT;
      if (c / W < C::RZ) put3<RS>(sU, c, q[k], P.gamma);
    }
  }
  __syncthreads();
  double F[K][5];
  const int p0 = tid / W * K;
  const int vz = min(TZ, P.nz - z0);   // the tile's cells inside the grid
  const int valid = vz + 1 - p0 < K ? vz + 1 - p0 : K;
  // (waves past the last interface skip the walk)
  if ((tid & ~63) / W * K <= vz) {
    const int wave0 = tid & ~63;
    const unsigned bits = walk3<2, K, RS, W, ORD>(
        sU, P.gamma, P.g1inv, sQueue + wave0 * K, (p0 - 1 + H) * W + l, valid,
        [&](int e) {
          const int t = wave0 + e;
          return (t / W * K - 1 + H) * W + t % W;
        },
        F);
    if (P.sig[2] && g0 + l < nl)
      for (int q = 0; q < valid; ++q)
        if (z0 + p0 + q <= P.nz)
          P.sig[2][(size_t)(z0 + p0 + q) * nl + g0 + l] = !((bits >> q) & 1u);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < K; ++q)
    if (q < valid) {
#pragma unroll
      for (int m = 0; m < 5; ++m) sU[m * RS + (p0 + q) * W + l] = F[q][m];
    }
  __syncthreads();

  const double dtv = P.mode != MODE_RESIDUAL ? *P.dt : 0.0;
  double ea = 0.0, eb = 0.0, ec = 0.0;   // time-step extrema (stage 3, P.dtx)
  bool ebad = false;
#pragma unroll 1
  for (int p = tid / W; p < TZ; p += NT / W) {
    if (g0 + l >= nl || z0 + p >= P.nz) continue;
    const size_t s = (size_t)(z0 + p) * nl + g0 + l;
    constexpr int mz[5] = {0, 2, 3, 1, 4};   // rotated component of the z fluxes
    double nv[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      const size_t o = m * n + s;
      const double* f = sU + mz[m] * RS + p * W + l;
      const double r = P.R[o] - (f[W] - f[0]) * P.inv_d[2];
      if (P.mode == MODE_RESIDUAL)
        nv[m] = r;
      else if (P.mode == MODE_STAGE1)
        nv[m] = P.Qn[o] + dtv * r;
      else if (P.mode == MODE_STAGE2)
        nv[m] = 0.75 * P.Qn[o] + 0.25 * P.Qk[o] + (0.25 * dtv) * r;
      else
        nv[m] = (1.0 / 3.0) * P.Qn[o] + (2.0 / 3.0) * P.Qk[o] + ((2.0 / 3.0) * dtv) * r;
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) P.out[m * n + s] = nv[m];
    if (P.dtx) dt3_extrema_cell(nv, P.gamma, ea, eb, ec, ebad);
  }
  if (P.dtx) {
    // every lane of every wave reaches this point: wave extrema into the
    // wave's slot
    if (ebad) atomicOr(P.status, 1u);
    constexpr int NW = NT / 64;
    const int nslot = P.ntiles * NW, slot = blockIdx.x * NW + (tid >> 6);
    ea = wave_extremum<true>(ea);
    eb = wave_extremum<true>(eb);
    ec = wave_extremum<true>(ec);
    if (__lane_id() == 0) {
      P.dtx[slot] = ea;
      P.dtx[nslot + slot] = eb;
      P.dtx[2 * nslot + slot] = ec;
    }
  }
}

// ---------------------------------------------------------------------------
// Time step of a state (no viscous limit).
template <bool FINISH>
__global__ __launch_bounds__(kDtThreads) void dt3_reduce_kernel(Dt3Params P) {
#pragma clang fp contract(off)
  __shared__ double red[kDtThreads / 64];
  const size_t n = (size_t)P.nx * P.ny * P.nz;
  double conv = __builtin_inf();
  bool bad = false;
  for (size_t s = (size_t)blockIdx.x * blockDim.x + threadIdx.x; s < n;
       s += (size_t)gridDim.x * blockDim.x) {
    const double rho = P.Q[s];
    const double u = P.Q[n + s] / rho, v = P.Q[2 * n + s] / rho, w = P.Q[3 * n + s] / rho;
    const double p = (P.gamma - 1.0) * (P.Q[4 * n + s] - rho * (u * u + v * v + w * w) / 2.0);
    const double c = sqrt(P.gamma * p / rho);
    if (!(rho > 0.0) || !(p > 0.0) || !isfinite(c) || !isfinite(u) || !isfinite(v) ||
        !isfinite(w))
      bad = true;
    conv = fmin(conv, fmin(P.dx / (fabs(u) + c), fmin(P.dy / (fabs(v) + c), P.dz / (fabs(w) + c))));
  }
  if (bad) atomicOr(P.status, 1u);
  if (FINISH) {
    double e[1] = {conv};
    const double id[1] = {__builtin_inf()};
    dt_commit(e, id, P.partial, P.count, [](int, double x, double y) { return fmin(x, y); },
              [&](const double* m) { dt_write(m[0], __builtin_inf(), P.cfl, P.dt, P.status); });
    return;
  }
  conv = block_min(conv, red);
  if (threadIdx.x == 0) {
    P.partial[blockIdx.x] = conv;
    P.partial[kDtBlocks + blockIdx.x] = __builtin_inf();
  }
}

}  // namespace gbr
