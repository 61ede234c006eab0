// Launchers of the line-streamed stage kernel, instantiated by the units that
// fill the table of tile shapes.
#pragma once
#include "stage_variants.hpp"

namespace gbr {

// TX x TY tiles, K interfaces per lane.
template <class C, bool MLP, bool CONS, int ORD, bool LM, bool F32>
int launch_line_cfg(const StageParams& P, hipStream_t s) {
  static_assert(C::LDS_BYTES <= 160 * 1024, "LDS per workgroup");
  static_assert(C::NT / 64 <= kMaxStageWaves, "time-step slots");
  hipLaunchKernelGGL((meg7_line_kernel<C, MLP, CONS, ORD, LM, F32>), dim3(P.ntiles), dim3(C::NT), 0,
                     s, P);
  return C::NT / 64;
}

// Interfaces per lane by the number of tiles.  K = 4 reads and forms each cell
// 3.25 times per interface where K = 1 does it 10 times, but leaves a 15x15
// tile two waves: where the tiles do not fill the chip the serial chain of a
// lane counts, and a tile's work is spread over more lanes.  Measured per
// stage, us (Riemann field, K = 1 / 4 on 15x15 tiles, K = 2 / 4 on 31x15):
//   64^2    12.2 / 22.3    18.7 / 26.5
//   256^2   15.8 / 24.9    18.2 / 25.0
//   400^2   20.6 / 26.8    29.4 / 34.2   (729 and 351 tiles)
//   512^2   29.0 / 32.3    35.8 / 33.9   (1225 and 595 tiles; shear 24.1 / 20.8, 28.8 / 20.8)
//   1024^2  80.8 / 65.7    104.3 / 68.8
constexpr int kFewTiles15 = 1024, kFewTiles31 = 448;
template <bool VISC, bool MLP, bool F32 = false, bool CONS = false, int ORD = 7, bool LM = false>
int launch_line15(const StageParams& P, hipStream_t s) {
  if (P.ntiles < kFewTiles15)
    return launch_line_cfg<LineCfg<15, 15, 1, VISC, CONS ? 3 : 4>, MLP, CONS, ORD, LM, F32>(P, s);
  return launch_line_cfg<LineCfg<15, 15, 4, VISC, 3>, MLP, CONS, ORD, LM, F32>(P, s);
}
template <bool VISC, bool MLP, bool F32 = false, bool CONS = false, int ORD = 7, bool LM = false>
int launch_line31(const StageParams& P, hipStream_t s) {
  if (P.ntiles < kFewTiles31)
    return launch_line_cfg<LineCfg<31, 15, 2, VISC, 3>, MLP, CONS, ORD, LM, F32>(P, s);
  return launch_line_cfg<LineCfg<31, 15, 4, VISC, 3>, MLP, CONS, ORD, LM, F32>(P, s);
}
template <int TX, int TY, int K, int MINW, bool VISC, bool MLP, bool F32>
int launch_line(const StageParams& P, hipStream_t s) {
  return launch_line_cfg<LineCfg<TX, TY, K, VISC, MINW>, MLP, false, 7, false, F32>(P, s);
}

// Every shape's launchers of MEG7-prim, seventh order, HLLC.
template <bool MLP, bool F32>
void fill_prim(TileVariant* v) {
  auto put = [&](int k, LaunchFn euler, LaunchFn visc) {
    v[k].fn[F32][0][MLP] = euler;
    v[k].fn[F32][1][MLP] = visc;
  };
  put(TILE_31x15, launch_line31<false, MLP, F32>, launch_line31<true, MLP, F32>);
  put(TILE_15x15, launch_line15<false, MLP, F32>, launch_line15<true, MLP, F32>);
  put(TILE_63x7, launch_line<63, 7, 4, 3, false, MLP, F32>, nullptr);
  put(TILE_30x15, launch_line<30, 15, 4, 3, false, MLP, F32>, nullptr);
  // small grids: one interface per lane, twice the workgroups of 15x15 (64^2
  // Riemann stage 9.4 us against 12.2, 256^2 13.2 against 15.8)
  put(TILE_15x7, launch_line<15, 7, 1, 4, false, MLP, F32>,
      launch_line<15, 7, 1, 4, true, MLP, F32>);
}

// The two larger shapes' launchers of another scheme: out[tile][viscous].
template <bool CONS, int ORD, bool LM>
void fill_scheme(LaunchFn (&t31)[2], LaunchFn (&t15)[2]) {
  t31[0] = launch_line31<false, false, false, CONS, ORD, LM>;
  t31[1] = launch_line31<true, false, false, CONS, ORD, LM>;
  t15[0] = launch_line15<false, false, false, CONS, ORD, LM>;
  t15[1] = launch_line15<true, false, false, CONS, ORD, LM>;
}

}  // namespace gbr
