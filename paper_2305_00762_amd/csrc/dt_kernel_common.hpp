// What the 2D and 3D time-step reductions share.
#pragma once
#include <hip/hip_runtime.h>

namespace gbr {

constexpr int kDtBlocks = 1024;  // pass-1 workgroups at most (partials kept in context scratch)
constexpr int kDtThreads = 256;

__device__ __forceinline__ double block_min(double v, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if (__lane_id() == 0) red[w] = v;
  __syncthreads();
  double r = red[0];
  for (int k = 1; k < (int)(blockDim.x >> 6); ++k) r = fmin(r, red[k]);
  return r;
}

}  // namespace gbr
