// Launch of the 3D stage kernels (stage3d.hip).
#pragma once
#include "stage3d_params.hpp"

namespace gbr {

// Column kernel: kCol3W lines x kCol3Z cells, one interface a lane, four waves a
// workgroup.  Measured per launch (us; octant Riemann 128^3, 96^3, 64^3, 40^3,
// 24^3, Taylor-Green 64^3): 92, 48, 21, 12, 8, 13; two interfaces a lane
// 95, 53, 21, 17, 14, 13; 32 lines with one 96, 49, 22, 12, 12, 15, with two
// 97, 54, 22, 15, 14, 14; 16x19 142, 77, 34, 14, 11, 19.
constexpr int kCol3W = 16, kCol3Z = 15, kCol3Waves = 4;
inline long long col3_tiles(int nx, int ny, int nz) {
  return (((long long)nx * ny + kCol3W - 1) / kCol3W) * ((nz + kCol3Z - 1) / kCol3Z);
}
// Both kernels of a residual or stage call (P.tiles_*, ntiles filled here);
// returns the waves of the column launch (a time-step slot each in stage 3).
int launch_stage3(Stage3Params P, int order, hipStream_t s);
void launch_dt3(const Dt3Params& P, int blocks, bool finish, hipStream_t s);

}  // namespace gbr
