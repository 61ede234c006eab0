#include "stage3d.hpp"
#include "stage3d_launch.hpp"

namespace gbr {

// Plane tiles.  Three workgroups of four waves share a CU in each form, so below
// one round of them (3 x 256 tiles of 15x15) the shortest lane wins: K = 2.
// Above it the forms' tiles take 1 : 1.25 : 1.38 of each other's time and the
// form whose tiles cost least over the grid is taken; three interfaces a lane
// need 23% less walk per interface, 16x16 divides the powers of two and
// 20x17 fills 119 and 120 of 128 lanes.  Measured per launch (us; 15x15 K = 2,
// 16x16 K = 3, 20x17 K = 3), octant Riemann fields: 128^3 168, 160, 151;
// 96^3 80, 78, 74; 80^3 55, 55, 53; 75^3 44, 51, 49; 64^3 36, 31, 38;
// 56^3 26, 30, 28; 32^3 16, 17, 18; Taylor-Green 64^3 23.0, 18.7, 20.0.
// (15x15 K = 1: 179 at 128^3, 25 at Taylor-Green 64^3.)  Taken before the Riemann
// solver's two further estimates, which add 1%.
constexpr long long kOneRound = 3 * 256;

template <class C>
static long long plane_tiles(const Stage3Params& P) {
  return (long long)((P.nx + C::TX - 1) / C::TX) * ((P.ny + C::TY - 1) / C::TY) * P.nz;
}
template <class C, int ORD>
static void launch_plane(Stage3Params& P, hipStream_t s) {
  P.tiles_x = (P.nx + C::TX - 1) / C::TX;
  P.tiles_y = (P.ny + C::TY - 1) / C::TY;
  P.ntiles = (int)plane_tiles<C>(P);
  hipLaunchKernelGGL((meg7_plane3_kernel<C, ORD>), dim3(P.ntiles), dim3(C::NT), 0, s, P);
}

template <int ORD>
static int launch(Stage3Params& P, hipStream_t s) {
  using A = LineCfg<15, 15, 2, false, 3>;
  using B = LineCfg<16, 16, 3, false, 3>;
  using C = LineCfg<20, 17, 3, false, 3>;
  const long long na = plane_tiles<A>(P), a = 100 * na, b = 125 * plane_tiles<B>(P),
                  c = 138 * plane_tiles<C>(P);
  if (na <= kOneRound || (a <= b && a <= c)) launch_plane<A, ORD>(P, s);
  else if (b <= c) launch_plane<B, ORD>(P, s);
  else launch_plane<C, ORD>(P, s);
  P.tiles_z = (P.nz + kCol3Z - 1) / kCol3Z;
  P.ntiles = (int)col3_tiles(P.nx, P.ny, P.nz);
  using Z = Col3Cfg<kCol3W, kCol3Z, 1, 4>;
  static_assert(Z::NT == 64 * kCol3Waves, "time-step slots");
  hipLaunchKernelGGL((meg7_col3_kernel<Z, ORD>), dim3(P.ntiles), dim3(Z::NT), 0, s, P);
  return P.ntiles * kCol3Waves;
}

int launch_stage3(Stage3Params P, int order, hipStream_t s) {
  return order == 4 ? launch<4>(P, s) : launch<7>(P, s);
}

void launch_dt3(const Dt3Params& P, int blocks, bool finish, hipStream_t s) {
  if (finish)
    hipLaunchKernelGGL(dt3_reduce_kernel<true>, dim3(blocks), dim3(kDtThreads), 0, s, P);
  else
    hipLaunchKernelGGL(dt3_reduce_kernel<false>, dim3(blocks), dim3(kDtThreads), 0, s, P);
}

}  // namespace gbr
