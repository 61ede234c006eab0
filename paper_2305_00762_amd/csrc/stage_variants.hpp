// Tile shapes of the single-grid stage kernels and forms of the batched one:
// tables of launchers, filled from several translation units so that the
// kernels compile in parallel.
#pragma once
#include "batch_kernel.hpp"
#include "stage_line.hpp"

namespace gbr {

// A stage launcher enqueues one launch and returns its waves: a time-step slot
// each in stage 3.
using LaunchFn = int (*)(const StageParams&, hipStream_t);
constexpr int kMaxStageWaves = 8;

// Shapes trade halo work (small tiles) against LDS per workgroup and the
// number of workgroups; gbr_autotune times them on the caller's state.  A null
// entry has no build (the default shape then serves).
struct TileVariant {
  int tx, ty;             // cells per workgroup
  LaunchFn fn[2][2][2];   // [precision FP64/FP32-bulk][viscous][learned detector]
  LaunchFn cons[2];       // MEG7-cons, FP64 with the plain detector: [viscous]
  LaunchFn g4[2][2];      // fourth-order GRB, FP64 with the plain detector: [cons][viscous]
  LaunchFn ss[2][2];      // shock-stable HLLC, seventh order, FP64, plain: [cons][viscous]
  LaunchFn mpe[2][2];     // MP test at every interface, seventh order, FP64, plain: [cons][viscous]
};
enum : int { TILE_31x15 = 0, TILE_15x15, TILE_63x7, TILE_30x15, kNumVariants };
// 15x15 grids of fewer tiles run 15x7 tiles of kTinyWaves waves (stage_launch.hpp).
constexpr int kTinyTiles15 = 100, kTinyTY = 7, kTinyWaves = 4;
const TileVariant* tile_variants();

// The units' shares of the table.
void fill_fp64(TileVariant* v);
void fill_fp64_mlp(TileVariant* v);
void fill_f32(TileVariant* v);
void fill_f32_mlp(TileVariant* v);
void fill_cons(TileVariant* v);
void fill_order4(TileVariant* v);
void fill_shock_stable(TileVariant* v);
void fill_mpe(TileVariant* v);

using BatchLaunchFn = void (*)(const BatchParams&, int, hipStream_t);
struct BatchVariant {
  int tx, ty, loop;
  BatchLaunchFn fn[2];   // [FP64, FP32 bulk]
  int (*occ[2])();       // workgroups per CU
  int few_tiles;         // batches of fewer tiles launch few, one workgroup per tile
  BatchLaunchFn few[2];
};
constexpr int kNumBatchVariants = 4;
const BatchVariant* batch_variants();

}  // namespace gbr
