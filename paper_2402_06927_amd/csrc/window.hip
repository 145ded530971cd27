// window.hip -- k_window, the forecast of an ensemble: its instances.
#define SCH_TILE_DEFINITIONS
#include "tiles.hpp"

namespace sch {
#define SCH_DEFINE(PM, NT, FULL) SCH_WINDOW_KERNELS(, PM, NT, FULL)
SCH_TILES(SCH_DEFINE)
}  // namespace sch
