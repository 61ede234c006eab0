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
#define GBR_BATCH_VARIANT(TX, TY, LOOP)                                         \
  {TX, TY, LOOP,                                                                      \
   {launch_batch<TX, TY, 4, 3, false, LOOP>, launch_batch<TX, TY, 4, 3, true, LOOP>}, \
   {batch_blocks_per_cu<TX, TY, 4, 3, false, LOOP>,                                   \
    batch_blocks_per_cu<TX, TY, 4, 3, true, LOOP>}}
const BatchVariant kBatchVariants[kNumBatchVariants] = {
    GBR_BATCH_VARIANT(31, 15, true),
    GBR_BATCH_VARIANT(15, 15, true),
    GBR_BATCH_VARIANT(31, 15, false),
    GBR_BATCH_VARIANT(15, 15, false),
};
#undef GBR_BATCH_VARIANT
const BatchVariant* batch_variants() { return kBatchVariants; }
}  // namespace gbr
