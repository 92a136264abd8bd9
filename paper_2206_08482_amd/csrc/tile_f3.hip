// Forward-only row-tile kernel (agent_act / agent_value / a collection's values) for the 60:256:128:64:8 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FWD_PART_DEFINE(3, TileShapeNat, 64, 256, 128, 64, 32)
}
