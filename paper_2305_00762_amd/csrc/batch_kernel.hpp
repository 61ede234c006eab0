// Many independent grids advanced by one launch per RK stage.
//
// The grids of a batch are cut into tiles of one shape; their tiles are
// numbered grid after grid (tile_start[p] is the first tile of grid p).  In
// the persistent form a fixed number of workgroups -- as many as fit on the
// chip at once -- walk that tile order in rounds of gridDim.x tiles; in the
// one-tile form the launch has one workgroup per tile and the hardware
// dispatcher is the work queue (the tile loop of the persistent form makes
// the compiler keep tile-invariant values in registers across the loop,
// which can cost occupancy; the autotuner measures both).  Within a round,
// consecutive tiles go to one XCD (workgroup b runs on XCD b mod 8), so the
// halo re-reads of neighbouring tiles meet in the same L2.  Each tile runs the
// same tile function as the single-grid kernels (inviscid or viscous form,
// chosen per grid; multiply-adds fuse as the source groups them), so a grid of
// the batch computes what a single-grid launch with the same tile shape and
// interfaces per lane computes.  The time step is per grid: a
// two-pass min-reduction with a fixed number of partials per grid.  Every
// workgroup leaves the tile loop after at most ceil(total / gridDim.x)
// rounds.
#pragma once
#include "stage_line.hpp"

namespace gbr {

// One grid of the batch (host-side description; the time-step kernels read
// it on the device).
struct BatchProb {
  double* buf[3];          // the grid's three state arrays, SoA [4][ny][nx]
  int nx, ny, bcx, bcy;
  int tiles_x;             // tile columns for the batch's tile shape
  int pad_;
  double inv_dx, inv_dy, dx, dy;
  double gamma, g1inv, mu, kq, cfl;
};

// A stage launch reads the stage parameters of grid p from tab[p]: one table
// per (array roles, stage) combination, built on the host.
struct BatchParams {
  const StageParams* __restrict__ tab;   // [nprob]
  const int* __restrict__ tile_start;    // [nprob + 1]
  int nprob, total;                      // grids, tiles
};

// The tables do not change during a launch: constant address space, so uniform
// reads are scalar loads and stay in scalar registers.
template <class T>
using ConstPtr = const __attribute__((address_space(4))) T*;

// Grid p with tile_start[p] <= t < tile_start[p + 1].
__device__ __forceinline__ int batch_find(ConstPtr<int> ts, int n, int t) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (ts[mid] <= t) lo = mid;
    else hi = mid;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Parameters of grid p, held by value: behind a pointer every wait for LDS
// traffic in the tile function made the compiler read gamma and its like again,
// as vector loads in the middle of the walk (17 per lane and tile; batch of 512
// grids: a stage launch took 5.7 ms with them, 4.7 without).  What a batch has
// no use for is null here, so its code goes.
__device__ __forceinline__ StageParams batch_params(ConstPtr<StageParams> T) {
  StageParams P{};
  P.Qk = T->Qk; P.Qn = T->Qn; P.out = T->out; P.dt = T->dt; P.status = T->status;
  P.nx = T->nx; P.ny = T->ny; P.bcx = T->bcx; P.bcy = T->bcy;
  P.tiles_x = T->tiles_x; P.ntiles = T->ntiles;
  P.inv_dx = T->inv_dx; P.inv_dy = T->inv_dy;
  P.gamma = T->gamma; P.g1inv = T->g1inv; P.mu = T->mu; P.kq = T->kq;
  P.mode = T->mode;
  return P;
}

// CI, CV: the inviscid and the viscous form of one tile shape (same lanes per
// line, so the same workgroup); F32 as in the single-grid kernel.
template <class CI, class CV, bool F32, bool LOOP>
__global__ __launch_bounds__(CI::NT, CI::MINW) void meg7_batch_kernel(BatchParams B) {
  static_assert(CI::TX == CV::TX && CI::TY == CV::TY && CI::NT == CV::NT && CI::RS == CV::RS &&
                    CI::QN == CV::QN,
                "one tile shape");
  __shared__ double sU[4 * CI::RS];
  __shared__ unsigned short sQueue[CI::QN];
  const int G = gridDim.x, b = blockIdx.x;
  const int xcd = b & 7, per = G >> 3;   // G is a multiple of 8
  for (int base = 0; base < B.total; base += G) {
    const int t = base + xcd * per + (b >> 3);
    if (t < B.total) {
      const auto ts = (ConstPtr<int>)B.tile_start;
      const int p = batch_find(ts, B.nprob, t);
      const StageParams P = batch_params((ConstPtr<StageParams>)B.tab + p);
      const int lt = t - ts[p];
      const int tx0 = (lt % P.tiles_x) * CI::TX, ty0 = (lt / P.tiles_x) * CI::TY;
      if (P.mu > 0.0)
        stage_tile_line<CV, false, false, 7, false, F32>(P, tx0, ty0, sU, sQueue, nullptr);
      else
        stage_tile_line<CI, false, false, 7, false, F32>(P, tx0, ty0, sU, sQueue, nullptr);
    }
    if (!LOOP) break;   // one tile per workgroup: gridDim.x >= total
    __syncthreads();
  }
}

}  // namespace gbr
