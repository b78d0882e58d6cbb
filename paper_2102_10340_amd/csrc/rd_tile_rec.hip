// Resident-tile kernel instances: FitzHugh-Nagumo, passes that record the states
// of even times (rd_tile_body.h).
#include "rd_tile.h"

namespace rd {
TileFn<ModelFHN> tile_fn_rec(int cpl, int rw) { return pick_tile<ModelFHN, true>(cpl, rw); }
}  // namespace rd
