// Forward-only row-tile kernel (agent_act / agent_value / a collection's values) for the 108:200:400:100:21 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FWD_PART_DEFINE(5, TileShapeNat, 128, 224, 416, 128, 32)
}
