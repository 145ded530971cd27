// jitter.hip -- k_jitter (pCN moves) with the modes form of the noise: its instances.
#define SCH_TILE_DEFINITIONS
#include "tiles.hpp"

namespace sch {
#define SCH_DEFINE(PM, NT, FULL) SCH_JITTER_KERNELS(, PM, NT, FULL)
SCH_TILES(SCH_DEFINE)
}  // namespace sch
