#include "stage_launch.hpp"

namespace gbr {
void fill_cons(TileVariant* v) {
  fill_scheme<true, 7, false>(v[TILE_31x15].cons, v[TILE_15x15].cons);
}
}  // namespace gbr
