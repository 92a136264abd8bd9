// Forward-only row-tile kernel in fp8 (agent_act_fp8) for the 60:256:128:64:8 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FP8_PART_DEFINE(3, 64, 256, 128, 64, 32)
}
