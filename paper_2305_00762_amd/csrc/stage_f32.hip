#include "stage_launch.hpp"

namespace gbr {
void fill_f32(TileVariant* v) { fill_prim<false, true>(v); }
}  // namespace gbr
