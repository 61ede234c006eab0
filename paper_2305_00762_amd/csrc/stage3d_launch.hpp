// Launch of the 3D stage kernels (stage3d.hip).
#pragma once
#include "stage3d_params.hpp"

namespace gbr {

// Column kernel: kCol3W lines x kCol3Z cells per workgroup of at most
// kCol3MaxWaves waves.
constexpr int kCol3W = 32, kCol3Z = 15, kCol3MaxWaves = 8;
inline long long col3_tiles(int nx, int ny, int nz) {
  return (((long long)nx * ny + kCol3W - 1) / kCol3W) * ((nz + kCol3Z - 1) / kCol3Z);
}
// Both kernels of a residual or stage call (P.tiles_*, ntiles filled here);
// returns the waves of the column launch (a time-step slot each in stage 3).
int launch_stage3(Stage3Params P, int order, hipStream_t s);
void launch_dt3(const Dt3Params& P, int blocks, hipStream_t s);

}  // namespace gbr
