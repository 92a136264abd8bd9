// Forward-only row-tile kernel in fp8 (agent_act_fp8) for the 108:200:400:100:21 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FP8_PART_DEFINE(4, 128, 256, 448, 128, 32)
}
