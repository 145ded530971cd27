// batch.hip -- k_batch_window, the batched runner's forecast: its instances.
#define SCH_TILE_DEFINITIONS
#include "tiles.hpp"

namespace sch {
#define SCH_DEFINE(PM, NT) SCH_BATCH_KERNELS(, PM, NT)
SCH_BATCH_TILES(SCH_DEFINE)
}  // namespace sch
