// jitter_matern.hip -- k_jitter with the Matern-type noise: its instances.
#define SCH_TILE_DEFINITIONS
#include "tiles.hpp"

namespace sch {
#define SCH_DEFINE(PM, NT, FULL) SCH_JITTER_MATERN_KERNELS(, PM, NT, FULL)
SCH_TILES(SCH_DEFINE)
}  // namespace sch
