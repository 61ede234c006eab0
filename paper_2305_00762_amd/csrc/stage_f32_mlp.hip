#include "stage_launch.hpp"

namespace gbr {
void fill_f32_mlp(TileVariant* v) { fill_prim<true, true>(v); }
}  // namespace gbr
