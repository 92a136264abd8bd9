// Row-tile trainer kernel compiled for one model shape (padded layer widths): benchmark workload C2 (60:256:128:64:8;
// also the paper's Anymal 48:256:128:64:12 after padding).
#include "tile_kernel.h"

namespace gmi {
GMI_TILE_PART_DEFINE(3, 64, 256, 128, 64, 32)
}  // namespace gmi
