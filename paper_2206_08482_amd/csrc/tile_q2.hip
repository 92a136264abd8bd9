// Forward-only row-tile kernel in fp8 (agent_act_fp8) for the 108:400:200:100:21 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FP8_PART_DEFINE(2, 128, 448, 256, 128, 32)
}
