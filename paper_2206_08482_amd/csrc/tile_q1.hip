// Forward-only row-tile kernel in fp8 (agent_act_fp8) for the 211:512:512:512:256:20 model (padded widths).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_FP8_PART_DEFINE(1, 256, 512, 512, 512, 256, 32)
}
