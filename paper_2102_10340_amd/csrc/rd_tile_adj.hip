// Resident-tile reverse-pass instances (rd_tile_adj.h): blocks of 2 to 4 rows, 2
// or 4 columns per lane.
#include "rd_tile.h"

namespace rd {

namespace {

template <int CPL, bool LAMS>
TileAdjFn pick_rows(int rw)
{
    switch (rw) {
        case 2: return &tile_adjoint_kernel<CPL, 2, LAMS>;
        case 3: return &tile_adjoint_kernel<CPL, 3, LAMS>;
        case 4: return &tile_adjoint_kernel<CPL, 4, LAMS>;
        default: return nullptr;
    }
}

}  // namespace

TileAdjFn tile_adj_fn(bool lams, int cpl, int rw)
{
    if (cpl == 2) return lams ? pick_rows<2, true>(rw) : pick_rows<2, false>(rw);
    if (cpl == 4) return lams ? pick_rows<4, true>(rw) : pick_rows<4, false>(rw);
    return nullptr;
}

}  // namespace rd
