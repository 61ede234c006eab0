#include "stage_launch.hpp"

namespace gbr {
void fill_shock_stable(TileVariant* v) {
  fill_scheme<false, 7, true>(v[TILE_31x15].ss[0], v[TILE_15x15].ss[0]);
  fill_scheme<true, 7, true>(v[TILE_31x15].ss[1], v[TILE_15x15].ss[1]);
}
}  // namespace gbr
