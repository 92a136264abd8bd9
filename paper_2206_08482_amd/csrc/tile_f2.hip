// Forward-only row-tile kernel (agent_act / agent_value / a collection's values) for the 108:400:200:100:21 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FWD_PART_DEFINE(2, TileShapeNat, 128, 416, 224, 128, 32)
}
