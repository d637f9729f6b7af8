// Batched launches of the moment form on regions (btrt_mom_tile.h): shapes and launcher.
#pragma once

#include "btrt_internal.h"

namespace btrtk {

// A member's grid.
struct BatchGrid {
    int nx, ny;
    bool perx, pery;
};

// Regions of 64 columns by `waves` times `rows` rows; cost: what a launch is expected to take, us.
struct BatchRegion {
    int rows = 0, waves = 0;
    double cost = 0;
};

// The cheapest shape for launches of `steps` (2 .. 7) steps on these members.
template <typename T>
BatchRegion batch_region(const BatchGrid* grids, int n, int steps);
// Regions of one member, `rows` rows high.
int64_t batch_regions(const BatchGrid& g, int steps, int rows);
template <typename T>
hipError_t launch_batch_region(const BatchEntry<T>* ent, const int* begin, const int* par, int ninst, int total, int flip,
                               int steps, int grid, const BatchRegion& r, hipStream_t s);

}  // namespace btrtk
