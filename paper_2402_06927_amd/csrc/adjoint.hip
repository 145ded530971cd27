// adjoint.hip -- k_nudge_grad, objective and gradient of nudging: its instances.
#define SCH_TILE_DEFINITIONS
#include "tiles.hpp"

namespace sch {
#define SCH_DEFINE(PM, NT, FULL) SCH_ADJOINT_KERNELS(, PM, NT, FULL)
SCH_TILES_OWN_ADJOINT(SCH_DEFINE)
#undef SCH_DEFINE
#define SCH_DEFINE(PM, NT, FULL) SCH_ADJOINT_MATERN_KERNELS(, PM, NT, FULL)
SCH_TILES(SCH_DEFINE)
}  // namespace sch
