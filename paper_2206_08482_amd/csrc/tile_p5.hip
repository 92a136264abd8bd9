// Row-tile trainer kernel compiled for one model shape (padded layer widths): the paper's Table 6 model 108:200:400:100:21.
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_PART_DEFINE(5, 128, 224, 416, 128, 32)
}  // namespace gmi
