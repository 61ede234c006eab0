#include "stage3d.hpp"
#include "stage3d_launch.hpp"

namespace gbr {

// Interfaces per lane, measured per stage (us; octant Riemann 128^3, 96^3 and
// 40^3, Taylor-Green 64^3):
//   plane  K = 1: 264, 139, 20, 34   K = 2: 158, 88, 18, 24   K = 4: 156, 85, 26, 26
//   column K = 1: 148,  70, 12, 19   K = 2:  98, 55, 14, 14   K = 4: 124, 70, 25, 18
// Five fields' sums of K = 4 leave two waves per SIMD; K = 1 pays where the
// columns do not fill the chip and a lane's serial chain counts (40^3: 150
// workgroups).
constexpr int kFewColumns = 384;

template <int K, int ORD>
static int launch_col(const Stage3Params& P, hipStream_t s) {
  using Z = Col3Cfg<kCol3W, kCol3Z, K, 3>;
  static_assert(Z::NT <= 64 * kCol3MaxWaves, "time-step slots");
  hipLaunchKernelGGL((meg7_col3_kernel<Z, ORD>), dim3(P.ntiles), dim3(Z::NT), 0, s, P);
  return P.ntiles * (Z::NT / 64);
}

template <int ORD>
static int launch(Stage3Params& P, hipStream_t s) {
  using C = Plane3Cfg<2, 3>;
  P.tiles_x = (P.nx + C::TX - 1) / C::TX;
  P.tiles_y = (P.ny + C::TY - 1) / C::TY;
  P.ntiles = P.tiles_x * P.tiles_y * P.nz;
  hipLaunchKernelGGL((meg7_plane3_kernel<C, ORD>), dim3(P.ntiles), dim3(C::NT), 0, s, P);
  P.tiles_z = (P.nz + kCol3Z - 1) / kCol3Z;
  P.ntiles = (int)col3_tiles(P.nx, P.ny, P.nz);
  return P.ntiles < kFewColumns ? launch_col<1, ORD>(P, s) : launch_col<2, ORD>(P, s);
}

int launch_stage3(Stage3Params P, int order, hipStream_t s) {
  return order == 4 ? launch<4>(P, s) : launch<7>(P, s);
}

void launch_dt3(const Dt3Params& P, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(dt3_reduce_kernel, dim3(blocks), dim3(kDtThreads), 0, s, P);
}

}  // namespace gbr
