// Row-tile trainer kernel compiled for one model shape (padded layer widths): benchmark workloads C3 / C5 (108:400:200:100:21).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_PART_DEFINE(2, 128, 416, 224, 128, 32)
}  // namespace gmi
