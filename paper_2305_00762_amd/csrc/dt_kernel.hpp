// CFL time step of Sec. 2.5, reduced on the device.
//
// Per cell: conv = min(dx/(|u|+c), dy/(|v|+c)) and visc = min(dx^2/nu, dy^2/nu)
// (nu = mu/rho), each evaluated with one rounding per operation and IEEE
// division / square root.  Every workgroup reduces its cells to one (conv, visc)
// pair in a fixed grid-stride pattern; on small grids the last workgroup to
// finish reduces the pairs and writes dt = cfl * min(visc / alpha_v, conv), on
// others a second launch does.  A min is exact, so the result is bit-identical
// to any other evaluation order.  A bad cell (non-finite, rho <= 0, p <= 0) is
// recorded in the status word, since fmin would otherwise drop a NaN.  The
// entry point without a context keeps its scratch clear of counters and takes
// two launches.
#pragma once
#include "batch_kernel.hpp"
#include "dt_kernel_common.hpp"
#include "stage_kernel.hpp"

namespace gbr {

// Pass-1 workgroups for n cells: 1024 from 4M cells on, where more loads in
// flight pay (-17% at 4096^2); 512 below, where the second pass's extra
// partials would cost more than they save.
inline int dt_blocks(size_t n) {
  const size_t want = (n + kDtThreads - 1) / kDtThreads;
  const size_t cap = n >= (size_t(1) << 22) ? kDtBlocks : kDtBlocks / 2;
  return (int)(want < cap ? want : cap);
}

// One launch up to this many cells, two above: the arrivals at one count wait
// their turn, and 64 workgroups of more cells each take longer than a second
// launch.  Measured (us, one launch against two): 64^2 4.1, 5.6; 128^2 4.6, 5.6;
// 181^2 4.9, 5.6; 256^2 5.7, 5.5; 512^2 10.3, 6.9.
constexpr size_t kDtOneLaunch = 40000;
constexpr int kDtArrivals = 64;
inline int dt_arrivals(size_t n) {
  const size_t want = (n + kDtThreads - 1) / kDtThreads;
  return (int)(want < (size_t)kDtArrivals ? want : kDtArrivals);
}

// Scratch of the one-launch forms: kDtTurns sets for the step of a state and as
// many for that of stage-3 extrema, each class taken in its own turn, so up to
// kDtTurns calls of a class may be under way at once (several streams).  A set is
// kDtArrivals slots of each row of partial extrema, behind those of the two-launch
// forms, and a word behind the status words.  Every launch of a set has the same
// number of workgroups, a constant of the context: whatever calls meet in a set
// (more than kDtTurns at once, or a replayed graph, which keeps the set it was
// captured with), its count is back at zero when they are done.
constexpr unsigned kDtTurns = 8;
constexpr size_t kStatusWords = 16 + 2 * kDtTurns;
constexpr size_t kDtPartials = 2 * 3 * (size_t)kDtBlocks;
static_assert(2 * kDtTurns * kDtArrivals <= (unsigned)kDtBlocks, "sets fit the partials");
struct DtSet {
  double* partial;
  unsigned* count;
};
inline DtSet dt_set(double* partial, unsigned* status, unsigned (&turn)[2], bool extrema) {
  const unsigned k = turn[extrema]++ % kDtTurns + (extrema ? kDtTurns : 0);
  return {partial + 3 * kDtBlocks + k * kDtArrivals, status + 16 + k};
}

struct DtParams {
  const double* __restrict__ Q;
  double* partial;   // [2][kDtBlocks] (context scratch holds [3][kDtBlocks])
  unsigned* count;   // arrivals, zero between launches; null: the partials only
  double* dt;
  unsigned* status;
  int nx, ny;
  double dx, dy, gamma, mu, cfl;
};

// Convective and viscous limits of cell s folded into (conv, visc).
__device__ __forceinline__ void dt_cell(const double* __restrict__ Q, size_t n, size_t s,
                                        double gamma, double mu, double dx, double dy,
                                        double& conv, double& visc, bool& bad) {
#pragma clang fp contract(off)
  const double rho = Q[s];
  const double u = Q[n + s] / rho, v = Q[2 * n + s] / rho;
  const double p = (gamma - 1.0) * (Q[3 * n + s] - rho * (u * u + v * v) / 2.0);
  const double c = sqrt(gamma * p / rho);
  if (!(rho > 0.0) || !(p > 0.0) || !isfinite(c) || !isfinite(u) || !isfinite(v)) bad = true;
  conv = fmin(conv, fmin(dx / (fabs(u) + c), dy / (fabs(v) + c)));
  if (mu > 0.0) {
    const double nu = mu / rho;
    visc = fmin(visc, fmin(dx * dx / nu, dy * dy / nu));
  }
}

// FINISH: the last workgroup writes dt.
template <bool FINISH>
__global__ __launch_bounds__(kDtThreads) void dt_reduce_kernel(DtParams P) {
#pragma clang fp contract(off)
  __shared__ double red[kDtThreads / 64];
  const size_t n = (size_t)P.nx * P.ny;
  double conv = __builtin_inf(), visc = __builtin_inf();
  bool bad = false;
  for (size_t s = (size_t)blockIdx.x * blockDim.x + threadIdx.x; s < n;
       s += (size_t)gridDim.x * blockDim.x) {
    dt_cell(P.Q, n, s, P.gamma, P.mu, P.dx, P.dy, conv, visc, bad);
  }
  if (bad) atomicOr(P.status, 1u);
  if (FINISH) {
    double v[2] = {conv, visc};
    const double id[2] = {__builtin_inf(), __builtin_inf()};
    dt_commit(v, id, P.partial, P.count, [](int, double x, double y) { return fmin(x, y); },
              [&](const double* e) { dt_write(e[0], e[1], P.cfl, P.dt, P.status); });
    return;
  }
  conv = block_min(conv, red);
  visc = block_min(visc, red);
  if (threadIdx.x == 0) {
    P.partial[blockIdx.x] = conv;
    P.partial[kDtBlocks + blockIdx.x] = visc;
  }
}

__global__ __launch_bounds__(kDtThreads) void dt_finish_kernel(const double* partial, int nblk,
                                                               double* dt, double cfl,
                                                               unsigned* status) {
  __shared__ double red[kDtThreads / 64];
  double conv = __builtin_inf(), visc = __builtin_inf();
  for (int k = threadIdx.x; k < nblk; k += blockDim.x) {
    conv = fmin(conv, partial[k]);
    visc = fmin(visc, partial[kDtBlocks + k]);
  }
  conv = block_min(conv, red);
  visc = block_min(visc, red);
  if (threadIdx.x == 0) dt_write(conv, visc, cfl, dt, status);
}

// Second pass of the time step without a context, with the status word in the same scratch as the partials.  A bad state seen by
// the first pass makes dt NaN (the caller has no context to ask), and the
// word is cleared for the next call.
__global__ __launch_bounds__(kDtThreads) void dt_finish_noalloc_kernel(const double* partial,
                                                                       int nblk, double* dt,
                                                                       double cfl,
                                                                       unsigned* status) {
#pragma clang fp contract(off)
  __shared__ double red[kDtThreads / 64];
  double conv = __builtin_inf(), visc = __builtin_inf();
  for (int k = threadIdx.x; k < nblk; k += blockDim.x) {
    conv = fmin(conv, partial[k]);
    visc = fmin(visc, partial[kDtBlocks + k]);
  }
  conv = block_min(conv, red);
  visc = block_min(visc, red);
  if (threadIdx.x == 0) {
    const double d = cfl * fmin(visc / kAlphaV, conv);
    *dt = (*status != 0u) ? __builtin_nan("") : d;
    *status = 0u;
  }
}

// dt from the extrema the stage-3 kernel left per workgroup, in one launch of up
// to 64 workgroups (1.5e5 slots of a 4096^2 grid: 9.9 us, as two launches took)
// and with the arithmetic of dt_cell -- the minimum over cells of
// fl(dx/(|u|+c)) is fl(dx/max(|u|+c)), and that of fl(fl(dx dx)/fl(mu/rho)) is
// fl(fl(dx dx)/fl(mu/min rho)), since fl(d/x) is monotone in x.
// THREE_D (inviscid): the third extremum is max(|w|+c), else min rho.
struct DtExtremaParams {
  const double* slots;   // [3][nslot]
  int nslot;
  double* partial;       // [3][kDtBlocks]
  unsigned* count;
  double* dt;
  unsigned* status;
  double cfl, dx, dy, dz, mu;
};
template <bool THREE_D>
__global__ __launch_bounds__(kDtThreads) void dt_extrema_kernel(DtExtremaParams P) {
  const double id[3] = {0.0, 0.0, THREE_D ? 0.0 : __builtin_inf()};
  double v[3] = {id[0], id[1], id[2]};
  auto fold = [](int m, double x, double y) {
    return THREE_D || m < 2 ? fmax(x, y) : fmin(x, y);
  };
  for (int k = blockIdx.x * kDtThreads + threadIdx.x; k < P.nslot; k += gridDim.x * kDtThreads)
#pragma unroll
    for (int m = 0; m < 3; ++m) v[m] = fold(m, v[m], P.slots[(size_t)m * P.nslot + k]);
  dt_commit(v, id, P.partial, P.count, fold, [&](const double* e) {
#pragma clang fp contract(off)
    double conv = fmin(P.dx / e[0], P.dy / e[1]), visc = __builtin_inf();
    if (THREE_D) conv = fmin(P.dx / e[0], fmin(P.dy / e[1], P.dz / e[2]));
    if (!THREE_D && P.mu > 0.0) {
      const double nu = P.mu / e[2];
      visc = fmin(P.dx * P.dx / nu, P.dy * P.dy / nu);
    }
    dt_write(conv, visc, P.cfl, P.dt, P.status);
  });
}

// Self-test of div_rb (the shared-reciprocal quotient of the time-step
// extrema) against IEEE division: `count` operand pairs drawn from a
// counter-based hash (splitmix64 of seed + index), magnitudes log-uniform over
// [2^-300, 2^300] with random signs, every 16th numerator zero; a zero
// quotient may differ in sign only.
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
__device__ __forceinline__ double selftest_operand(unsigned long long h) {
  // exponent in [-300, 299], 52 random mantissa bits, random sign
  const long long e = (long long)((h >> 53) % 600ull) - 300;
  const unsigned long long bits = ((unsigned long long)(e + 1023) << 52) |
                                  (h & 0x000FFFFFFFFFFFFFull) | ((h >> 52 & 1ull) << 63);
  return __longlong_as_double((long long)bits);
}
__global__ __launch_bounds__(256) void div_selftest_kernel(unsigned long long seed,
                                                           unsigned long long count,
                                                           unsigned long long* bad_count) {
  const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
  unsigned long long bad = 0;
  for (unsigned long long k = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x;
       k < count; k += stride) {
    const unsigned long long h1 = splitmix64(seed + 2 * k), h2 = splitmix64(seed + 2 * k + 1);
    const double a = (k % 16 == 15) ? 0.0 : selftest_operand(h1);
    const double b = selftest_operand(h2);
    const double q = div_rb(a, b, rcp_nr(b)), ref = a / b;
    const bool same = __double_as_longlong(q) == __double_as_longlong(ref) ||
                      (q == 0.0 && ref == 0.0);
    if (!(div_rb_ok(a) && div_rb_ok(b)) || !same) ++bad;
  }
  if (bad) atomicAdd(bad_count, bad);
}

// t += dt on the device (the clock of moving boundary segments).
__global__ void advance_time_kernel(double* t, const double* dt) {
  if (threadIdx.x == 0) *t = *t + *dt;
}

// ---------------------------------------------------------------------------
// Per-grid time step: kBatchDtBlocks partial minima per grid, then one thread
// per grid folds them (a min is exact: the result equals the single-grid one).
constexpr int kBatchDtBlocks = 32;

__global__ __launch_bounds__(kDtThreads) void batch_dt_reduce_kernel(const BatchProb* prob, int qn,
                                                                     double* partial,
                                                                     unsigned* status) {
  __shared__ double red[kDtThreads / 64];
  const int p = blockIdx.x / kBatchDtBlocks, k = blockIdx.x % kBatchDtBlocks;
  const BatchProb& g = prob[p];
  const double* Q = g.buf[qn];
  const size_t n = (size_t)g.nx * g.ny;
  double conv = __builtin_inf(), visc = __builtin_inf();
  bool bad = false;
  for (size_t s = (size_t)k * kDtThreads + threadIdx.x; s < n;
       s += (size_t)kBatchDtBlocks * kDtThreads)
    dt_cell(Q, n, s, g.gamma, g.mu, g.dx, g.dy, conv, visc, bad);
  if (bad) atomicOr(status, 1u);
  conv = block_min(conv, red);
  visc = block_min(visc, red);
  if (threadIdx.x == 0) {
    partial[(size_t)p * 2 * kBatchDtBlocks + k] = conv;
    partial[(size_t)p * 2 * kBatchDtBlocks + kBatchDtBlocks + k] = visc;
  }
}

__global__ __launch_bounds__(256) void batch_dt_finish_kernel(const BatchProb* prob, int nprob,
                                                              const double* partial, double* dt,
                                                              unsigned* status) {
#pragma clang fp contract(off)
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nprob) return;
  double conv = __builtin_inf(), visc = __builtin_inf();
  for (int k = 0; k < kBatchDtBlocks; ++k) {
    conv = fmin(conv, partial[(size_t)p * 2 * kBatchDtBlocks + k]);
    visc = fmin(visc, partial[(size_t)p * 2 * kBatchDtBlocks + kBatchDtBlocks + k]);
  }
  const double d = prob[p].cfl * fmin(visc / kAlphaV, conv);
  dt[p] = d;
  if (!(d > 0.0) || !isfinite(d)) atomicOr(status, 2u);
}

}  // namespace gbr
