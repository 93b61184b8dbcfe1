// snowlb_io.h -- the initial state of a batch (launched from snowlb_io.hip).
#pragma once
#include "snowlb_internal.h"

namespace snowlb {

// Initial state of a lattice: circular tanh seed, U from U_init (ny x nx) or U0 everywhere.
struct InitArgs {
    const float* U_init;
    float U0, sx, sy, R, width, u_in;
};

// Copy 0 of every lattice of a batch, over its list of 64 x 4 tiles.
hipError_t launch_init_batch(int storage, const DomDesc* doms_dev, const TileDesc* tiles_dev, int ntiles,
                             const InitArgs* args_dev, hipStream_t s);

}  // namespace snowlb
