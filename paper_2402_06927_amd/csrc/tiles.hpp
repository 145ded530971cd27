// tiles.hpp -- the kernels that hold a window, one instance per tile, are
// compiled in files of their own, side by side (window.hip, jitter.hip,
// jitter_matern.hip, adjoint.hip, batch.hip): here their declarations.
#pragma once

#include "adjoint.hpp"
#include "batch.hpp"
#include "model.hpp"
#include "tile_list.hpp"

namespace sch {

#define SCH_WINDOW_KERNELS(LINK, PM, NT, FULL)                                             \
  LINK template __global__ void k_window<PM, NT, FULL, false>(WindowArgs, HelmConst);      \
  LINK template __global__ void k_window<PM, NT, FULL, true>(WindowArgs, HelmConst);
#define SCH_JITTER_KERNELS(LINK, PM, NT, FULL) \
  LINK template __global__ void k_jitter<PM, NT, FULL, false, false>(JitterArgs, HelmConst);
#define SCH_JITTER_MATERN_KERNELS(LINK, PM, NT, FULL)                                        \
  LINK template __global__ void k_jitter<PM, NT, FULL, true, false>(JitterArgs, HelmConst);  \
  LINK template __global__ void k_jitter<PM, NT, FULL, true, true>(JitterArgs, HelmConst);
#define SCH_ADJOINT_KERNELS(LINK, PM, NT, FULL) \
  LINK template __global__ void k_nudge_grad<PM, NT, FULL, false>(NudgeArgs, HelmConst);
#define SCH_ADJOINT_MATERN_KERNELS(LINK, PM, NT, FULL) \
  LINK template __global__ void k_nudge_grad<PM, NT, FULL, true>(NudgeArgs, HelmConst);
#define SCH_BATCH_KERNELS(LINK, PM, NT) \
  LINK template __global__ void k_batch_window<PM, NT>(BatchDev, const int*, int, unsigned int*);

#ifndef SCH_TILE_DEFINITIONS
#define SCH_DECLARE(PM, NT, FULL)             \
  SCH_WINDOW_KERNELS(extern, PM, NT, FULL)    \
  SCH_JITTER_KERNELS(extern, PM, NT, FULL)    \
  SCH_JITTER_MATERN_KERNELS(extern, PM, NT, FULL) \
  SCH_ADJOINT_MATERN_KERNELS(extern, PM, NT, FULL)
SCH_TILES(SCH_DECLARE)
#undef SCH_DECLARE
#define SCH_DECLARE(PM, NT, FULL) SCH_ADJOINT_KERNELS(extern, PM, NT, FULL)
SCH_TILES_OWN_ADJOINT(SCH_DECLARE)
#undef SCH_DECLARE
#define SCH_DECLARE(PM, NT) SCH_BATCH_KERNELS(extern, PM, NT)
SCH_BATCH_TILES(SCH_DECLARE)
#undef SCH_DECLARE
#endif

}  // namespace sch
