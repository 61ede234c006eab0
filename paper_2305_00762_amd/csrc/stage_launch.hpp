// Launchers of the line-streamed stage kernel, instantiated by the units that
// fill the table of tile shapes.
#pragma once
#include "stage_variants.hpp"

namespace gbr {

// TX x TY tiles, K interfaces per lane; returns the launch's time-step slots (a
// wave each).
template <class C, bool MLP, bool CONS, int ORD, bool LM, bool F32>
int launch_line_cfg(const StageParams& P, hipStream_t s) {
  static_assert(C::LDS_BYTES <= 160 * 1024, "LDS per workgroup");
  static_assert(C::NT / 64 <= kMaxStageWaves, "time-step slots");
  hipLaunchKernelGGL((meg7_line_kernel<C, MLP, CONS, ORD, LM, F32>), dim3(P.ntiles), dim3(C::NT), 0,
                     s, P);
  return P.ntiles * (C::NT / 64);
}

// Interfaces per lane by the number of tiles.  K = 4 reads and forms each cell
// 3.25 times per interface where K = 2 does it 5.5 and K = 1 ten times, but
// leaves a 15x15 tile two waves: where the tiles do not fill the chip the serial
// chain of a lane counts, and a tile's work is spread over more lanes.  The
// viscous flux shares its walk between a lane's interfaces, so K = 1 does not
// pay there.  Measured per stage, us (K = 1, 2, 4 on 15x15 tiles; K = 2, 4 on
// 31x15):
//                 Riemann                          shear layer (viscous)
//   256^2    13.9 14.6 18.8   14.5 18.7       11.9 10.5 14.6   10.4 11.3
//   350^2    17.8 17.2 19.4   20.8 21.4       (576 tiles of 15x15)
//   400^2    18.8 20.2 20.9   23.5 26.3       16.8 13.8 15.6   19.0 15.7   (729, 351)
//   450^2    22.7 21.6 21.3   26.2 26.8       (900, 450)
//   512^2    25.9 23.9 25.4   30.6 26.8       24.7 19.1 19.7   27.5 20.1   (1225, 595)
//   600^2    31.6 28.8 30.5   38.1 33.2       (1600, 800)
//   700^2    40.6 36.1 34.8   50.6 36.4       40.7 30.7 31.1   46.2 30.3   (2209, 1081)
//   1024^2   76.0 64.2 56.6   93.9 59.5       79.8 59.3 54.1   89.9 53.3
// (taken before the Riemann solver's two further estimates, which add 1 to 2%).
// MEG7-cons needs more registers than four waves per SIMD leave, so its K = 1
// ends earlier (K = 1, 2; 15x15): 128^2 16.4 19.1, 256^2 21.8 23.7 (324 tiles),
// 400^2 35.2 28.9.
// Below 100 tiles of 15x15 (MEG7-prim) the chip is nearly empty and 15x7 tiles of
// one interface a lane, twice the workgroups, serve the shape: 24^2 to 128^2
// Riemann 10.9 us a stage (events) against 13.2, viscous 9.4 against 10.8; at
// 180^2 (144 tiles) 13.7 and 13.5, 11.2 and 10.9.
constexpr int kFewTiles15 = 800, kFewTilesCons = 400, kMidTiles15 = 1900, kFewTiles31 = 448;
template <bool VISC, bool MLP, bool F32 = false, bool CONS = false, int ORD = 7, bool LM = false>
int launch_line15(const StageParams& P, hipStream_t s) {
  if constexpr (!CONS && ORD == 7 && !LM)
    if (P.ntiles < kTinyTiles15) {
      using C = LineCfg<15, kTinyTY, 1, VISC, 4>;
      StageParams T = P;
      T.ntiles = P.tiles_x * ((P.ny + C::TY - 1) / C::TY);
      static_assert(C::NT / 64 == kTinyWaves, "time-step slots");
      return launch_line_cfg<C, MLP, CONS, ORD, LM, F32>(T, s);
    }
  if constexpr (!VISC)
    if (P.ntiles < (CONS ? kFewTilesCons : kFewTiles15))
      return launch_line_cfg<LineCfg<15, 15, 1, VISC, CONS ? 3 : 4>, MLP, CONS, ORD, LM, F32>(P, s);
  if (P.ntiles < kMidTiles15)
    return launch_line_cfg<LineCfg<15, 15, 2, VISC, 3>, MLP, CONS, ORD, LM, F32>(P, s);
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
