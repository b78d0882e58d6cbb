// Resident-tile kernel instances: FitzHugh-Nagumo, plain passes (rd_tile_body.h).
#include "rd_tile.h"

namespace rd {
TileFn<ModelFHN> tile_fn_fhn(int cpl, int rw) { return pick_tile<ModelFHN, false>(cpl, rw); }
}  // namespace rd
