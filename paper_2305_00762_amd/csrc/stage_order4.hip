#include "stage_launch.hpp"

namespace gbr {
void fill_order4(TileVariant* v) {
  fill_scheme<false, 4, false>(v[TILE_31x15].g4[0], v[TILE_15x15].g4[0]);
  fill_scheme<true, 4, false>(v[TILE_31x15].g4[1], v[TILE_15x15].g4[1]);
}
}  // namespace gbr
