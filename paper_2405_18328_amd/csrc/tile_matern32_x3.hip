// Tile pass kernels: Matern-3/2, three fp16 pieces per point.
#include "tile_kernels_f16.h"

tileh_fn gp_tile_matern32_x3(int ds, int NT, bool y, int form, bool wide) { return pick_shape<GP_MATERN32_ARD, 3>(ds, NT, y, form, wide); }
