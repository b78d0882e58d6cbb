// Resident-tile kernel instances: Gray-Scott (rd_tile_body.h).
#include "rd_tile.h"

namespace rd {
TileFn<ModelGrayScott> tile_fn_gs(int cpl, int rw) { return pick_tile<ModelGrayScott, false>(cpl, rw); }
}  // namespace rd
