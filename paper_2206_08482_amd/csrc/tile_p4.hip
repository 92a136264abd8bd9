// Row-tile trainer kernel compiled for one model shape (padded layer widths): the paper's Table 6 models 24:256:128:64:3 and
// 23:256:128:64:9.
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_PART_DEFINE(4, 32, 256, 128, 64, 32)
}  // namespace gmi
