#include "stage_variants.hpp"

namespace gbr {
// MP test at every interface (FP64).
template <class C, bool CONS>
int launch_mpe(const StageParams& P, hipStream_t s) {
  static_assert(C::LDS_BYTES <= 160 * 1024, "LDS per workgroup");
  static_assert(C::NT / 64 <= kMaxStageWaves, "time-step slots");
  hipLaunchKernelGGL((meg7_stage_kernel<C, CONS>), dim3(P.ntiles), dim3(C::NT), 0, s, P);
  return P.ntiles * (C::NT / 64);
}

template <bool CONS>
void fill_both(TileVariant* v) {
  v[TILE_31x15].mpe[CONS][0] = launch_mpe<TileCfg<31, 15, 15, 16, 256, false>, CONS>;
  v[TILE_31x15].mpe[CONS][1] = launch_mpe<TileCfg<31, 15, 8, 16, 256, true>, CONS>;
  v[TILE_15x15].mpe[CONS][0] = launch_mpe<TileCfg<15, 15, 15, 15, 256, false>, CONS>;
  v[TILE_15x15].mpe[CONS][1] = launch_mpe<TileCfg<15, 15, 15, 15, 256, true>, CONS>;
}
void fill_mpe(TileVariant* v) {
  fill_both<false>(v);
  fill_both<true>(v);
}

const TileVariant* tile_variants() {
  static const struct Table {
    TileVariant v[kNumVariants] = {{31, 15}, {15, 15}, {63, 7}, {30, 15}};
    Table() {
      fill_fp64(v);
      fill_fp64_mlp(v);
      fill_f32(v);
      fill_f32_mlp(v);
      fill_cons(v);
      fill_order4(v);
      fill_shock_stable(v);
      fill_mpe(v);
    }
  } table;
  return table.v;
}
}  // namespace gbr
