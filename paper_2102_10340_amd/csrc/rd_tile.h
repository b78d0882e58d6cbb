// rd_tile.h -- tables of the resident-tile kernel instances (rd_tile_*.hip).
#pragma once

#include "rd_launch.h"
#include "rd_tile_adj.h"
#include "rd_tile_body.h"

namespace rd {
TileFn<ModelFHN> tile_fn_fhn(int cpl, int rw);
TileFn<ModelFHN> tile_fn_rec(int cpl, int rw);
TileFn<ModelGrayScott> tile_fn_gs(int cpl, int rw);
TileFn<ModelCnn> tile_fn_cnn(int cpl, int rw);
TileAdjFn tile_adj_fn(bool lams, int cpl, int rw);
}  // namespace rd
