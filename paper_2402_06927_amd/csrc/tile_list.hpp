// tile_list.hpp -- the tiles (slots per thread, threads per particle, full
// chunks only) that the model kernels are compiled for.
#pragma once

#define SCH_FULL_AND_RAGGED(X, PM, NT) X(PM, NT, true) X(PM, NT, false)
// those that doubles_adjoint() leaves to the modes-form adjoint, and the others
#define SCH_TILES_OWN_ADJOINT(X)                 \
  SCH_FULL_AND_RAGGED(X, 2, 64)                  \
  SCH_FULL_AND_RAGGED(X, 4, 64)                  \
  X(6, 64, false) SCH_FULL_AND_RAGGED(X, 8, 64)   \
  X(6, 128, false) SCH_FULL_AND_RAGGED(X, 8, 128) \
  X(6, 256, false) SCH_FULL_AND_RAGGED(X, 8, 256) \
  X(6, 512, false) SCH_FULL_AND_RAGGED(X, 8, 512) \
  X(12, 512, false) SCH_FULL_AND_RAGGED(X, 16, 512)
#define SCH_TILES_DOUBLED_ADJOINT(X)                \
  X(12, 64, false) SCH_FULL_AND_RAGGED(X, 16, 64)   \
  X(12, 128, false) SCH_FULL_AND_RAGGED(X, 16, 128) \
  X(12, 256, false) SCH_FULL_AND_RAGGED(X, 16, 256)
#define SCH_TILES(X) SCH_TILES_OWN_ADJOINT(X) SCH_TILES_DOUBLED_ADJOINT(X)

// The batched runner takes every grid as ragged, and any thread count with any
// number of nodes.
#define SCH_BATCH_ROW(X, NT) X(4, NT) X(6, NT) X(8, NT) X(12, NT) X(16, NT)
#define SCH_BATCH_TILES(X) \
  SCH_BATCH_ROW(X, 64) SCH_BATCH_ROW(X, 128) SCH_BATCH_ROW(X, 256) SCH_BATCH_ROW(X, 512)
