#include "stage_launch.hpp"

namespace gbr {
void fill_fp64_mlp(TileVariant* v) { fill_prim<true, false>(v); }
}  // namespace gbr
