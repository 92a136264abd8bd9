// Forward-only row-tile kernel (agent_act / agent_value / a collection's values) for the 24:256:128:64:3 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FWD_PART_DEFINE(4, TileShapeNat, 32, 256, 128, 64, 32)
}
