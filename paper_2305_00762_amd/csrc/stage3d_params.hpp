// Parameters of the 3D kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gbr {

struct Stage3Params {
  const double* __restrict__ Qk;  // state the residual is evaluated on [5][nz][ny][nx]
  const double* __restrict__ Qn;  // Q^n (stages 2, 3)
  double* R;                      // residual accumulator [5][nz][ny][nx]
  double* out;                    // residual or Q^(k+1)
  const double* __restrict__ dt;  // device scalar (stages)
  uint8_t* sig[3];                // optional interface flags per direction
  unsigned* status;
  int nx, ny, nz;
  int bc[3];                      // boundary kind per direction
  double inv_d[3];                // 1 / spacing
  double gamma, g1inv;
  int mode;                       // MODE_RESIDUAL or MODE_STAGE1..3
  int tiles_x, tiles_y;           // plane kernel
  int tiles_z;                    // column kernel
  int ntiles;                     // workgroups of the launch
  // stage 3 only (else null): per-wave time-step extrema of the output,
  // [3][column workgroups x waves]: max(|u|+c), max(|v|+c), max(|w|+c)
  double* dtx;
};

// CFL time step in 3D (inviscid), Sec. 2.5.
struct Dt3Params {
  const double* __restrict__ Q;
  double* partial;
  unsigned* count;   // arrivals, zero between launches
  double* dt;
  unsigned* status;
  int nx, ny, nz;
  double dx, dy, dz, gamma, cfl;
};

}  // namespace gbr
