#include "stage3d.hpp"
#include "stage3d_launch.hpp"

namespace gbr {

// Interfaces per lane, measured per stage (us; octant Riemann 128^3 and 40^3,
// Taylor-Green 64^3):
//   plane  K = 1: 329, 27, 37   K = 2: 192, 25, 25   K = 4: 194, 36, 27
//   column K = 1: 114, 15, 15   K = 2: 115, 19, 14   K = 4: 146, 36, 18
// Five fields' sums of K = 4 leave two waves per SIMD.
template <int ORD>
static void launch(Stage3Params& P, hipStream_t s) {
  using C = Plane3Cfg<2, 3>;
  P.tiles_x = (P.nx + C::TX - 1) / C::TX;
  P.tiles_y = (P.ny + C::TY - 1) / C::TY;
  P.ntiles = P.tiles_x * P.tiles_y * P.nz;
  hipLaunchKernelGGL((meg7_plane3_kernel<C, ORD>), dim3(P.ntiles), dim3(C::NT), 0, s, P);
  using Z = Col3Cfg<kCol3W, kCol3Z, 1, 3>;
  static_assert(Z::NT == 64 * kCol3Waves, "time-step slots");
  P.tiles_z = (P.nz + kCol3Z - 1) / kCol3Z;
  P.ntiles = (int)col3_tiles(P.nx, P.ny, P.nz);
  hipLaunchKernelGGL((meg7_col3_kernel<Z, ORD>), dim3(P.ntiles), dim3(Z::NT), 0, s, P);
}

void launch_stage3(Stage3Params P, int order, hipStream_t s) {
  if (order == 4) launch<4>(P, s);
  else launch<7>(P, s);
}

void launch_dt3(const Dt3Params& P, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(dt3_reduce_kernel, dim3(blocks), dim3(kDtThreads), 0, s, P);
}

}  // namespace gbr
