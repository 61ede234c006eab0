#include "stage_launch.hpp"

namespace gbr {
void fill_fp64(TileVariant* v) { fill_prim<false, false>(v); }
}  // namespace gbr
