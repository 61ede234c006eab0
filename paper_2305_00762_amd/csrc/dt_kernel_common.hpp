// What the 2D and 3D time-step reductions share.
#pragma once
#include "meg7_device.hpp"

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

// End of a time-step reduction: the workgroup's NV extrema go to its slots of
// partial ([NV][kDtBlocks]); the workgroup that arrives last folds the slots,
// and its thread 0 passes the grid's extrema to fin.  fold(m, x, y): the
// extremum m of two values, id[m] its identity.  An extremum is exact, so the
// order of arrival does not show in the result.  Slots and count are written
// and read at device scope (the XCDs' L2s hold no common copy of plain
// accesses); atomicInc returns count to zero for the next launch, as every launch
// on one count has the same number of workgroups.
template <int NV, class Fold, class Fin>
__device__ __forceinline__ void dt_commit(double (&v)[NV], const double (&id)[NV], double* partial,
                                          unsigned* count, Fold fold, Fin fin) {
  __shared__ double red[NV][kDtThreads / 64];
  __shared__ bool last;
  auto block_fold = [&]() {
#pragma unroll
    for (int m = 0; m < NV; ++m) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v[m] = fold(m, v[m], __shfl_xor(v[m], o));
      if (__lane_id() == 0) red[m][threadIdx.x >> 6] = v[m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NV; ++m)
      for (int k = 0; k < kDtThreads / 64; ++k) v[m] = fold(m, v[m], red[m][k]);
  };
  block_fold();
  if (threadIdx.x == 0) {
    // an exchange that has returned is done at device scope
    double old[NV];
#pragma unroll
    for (int m = 0; m < NV; ++m)
      old[m] = __hip_atomic_exchange(partial + m * kDtBlocks + blockIdx.x, v[m], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int m = 0; m < NV; ++m) asm volatile("" : : "v"(old[m]) : "memory");
    last = atomicInc(count, gridDim.x - 1) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
#pragma unroll
  for (int m = 0; m < NV; ++m) v[m] = id[m];
  for (int k = threadIdx.x; k < (int)gridDim.x; k += kDtThreads)
#pragma unroll
    for (int m = 0; m < NV; ++m)
      v[m] = fold(m, v[m], __hip_atomic_load(partial + m * kDtBlocks + k, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT));
  block_fold();
  if (threadIdx.x == 0) fin(v);
}

// The step written by a finish: dt = cfl min(visc / alpha_v, conv).
__device__ __forceinline__ void dt_write(double conv, double visc, double cfl, double* dt,
                                         unsigned* status) {
#pragma clang fp contract(off)
  const double d = cfl * fmin(visc / kAlphaV, conv);
  *dt = d;
  if (!(d > 0.0) || !isfinite(d)) atomicOr(status, 2u);
}

}  // namespace gbr
