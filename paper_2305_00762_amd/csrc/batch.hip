#include "stage_variants.hpp"

namespace gbr {
// Forms of the batched kernel: tile shape x persistent tile loop or one
// workgroup per tile.
template <int TX, int TY, int K, int MINW, bool F32, bool LOOP>
void launch_batch(const BatchParams& B, int grid, hipStream_t s) {
  using CI = LineCfg<TX, TY, K, false, MINW>;
  using CV = LineCfg<TX, TY, K, true, MINW>;
  hipLaunchKernelGGL((meg7_batch_kernel<CI, CV, F32, LOOP>), dim3(grid), dim3(CI::NT), 0, s, B);
}
template <int TX, int TY, int K, int MINW, bool F32, bool LOOP>
int batch_blocks_per_cu() {
  using CI = LineCfg<TX, TY, K, false, MINW>;
  using CV = LineCfg<TX, TY, K, true, MINW>;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, meg7_batch_kernel<CI, CV, F32, LOOP>, CI::NT,
                                                   0) != hipSuccess)
    return 0;
  return n;
}

// Fewer 15x15 tiles than this do not fill the chip with K = 4, two waves a
// tile: both forms then launch K = 2, four waves a tile, one workgroup per tile.
// Measured, us a step, FP32 bulk (K = 4 persistent, K = 4 one-tile, K = 2): Riemann
// grids, 4 of 48^2 and 96^2 (130 tiles) 77, 68, 43; one of 256^2 (324) 94, 83, 59;
// 16 of 96^2 (784) 109, 94, 79; 8 of 200^2 (1568) 137, 117, 106; 64 of 200^2 (12544)
// 646, 460, 533; viscous shear, 16 of 96^2 69, 51, 53; 8 of 200^2 123, 79, 80; 64 of
// 48^2 and 100^2 (2080) 172, 109, 112; 48 of 100^2 (2352) 160, 101, 110.
constexpr int kFewTilesBatch15 = 2200;
#define GBR_BATCH_VARIANT(TX, TY, LOOP)                                               \
  {TX, TY, LOOP,                                                                      \
   {launch_batch<TX, TY, 4, 3, false, LOOP>, launch_batch<TX, TY, 4, 3, true, LOOP>}, \
   {batch_blocks_per_cu<TX, TY, 4, 3, false, LOOP>,                                   \
    batch_blocks_per_cu<TX, TY, 4, 3, true, LOOP>},                                   \
   TX == 15 ? kFewTilesBatch15 : 0,                                                   \
   {TX == 15 ? launch_batch<15, 15, 2, 3, false, false> : nullptr,                    \
    TX == 15 ? launch_batch<15, 15, 2, 3, true, false> : nullptr}}
const BatchVariant kBatchVariants[kNumBatchVariants] = {
    GBR_BATCH_VARIANT(31, 15, true),
    GBR_BATCH_VARIANT(15, 15, true),
    GBR_BATCH_VARIANT(31, 15, false),
    GBR_BATCH_VARIANT(15, 15, false),
};
#undef GBR_BATCH_VARIANT
const BatchVariant* batch_variants() { return kBatchVariants; }
}  // namespace gbr
