// Launchers of the batched kernels of the moment form (btrt_mom.h).

#include "btrt_mom.h"

namespace btrtk {

template <typename T>
hipError_t launch_batch_mom(const BatchEntry<T>* ent, const int* begin, const int* par, int ninst, int total, int flip,
                            int steps, int grid, int rows, hipStream_t s)
{
    if (total <= 0 || ninst <= 0) return hipSuccess;
    if (steps == 1) {
        const unsigned g = static_cast<unsigned>(grid > 0 ? std::min(grid, total) : total);
        hipLaunchKernelGGL((mom_batch1_kernel<T>), dim3(g), dim3(kBlock), 0, s, ent, begin, par, ninst, total, flip);
        return hipGetLastError();
    }
    // Several resident strips per CU: a persistent grid of `grid` blocks covers the list.
    const unsigned g = static_cast<unsigned>(grid > 0 ? std::min(grid * kWalkGroup, total) : total);
    switch (steps) {
        case 2: hipLaunchKernelGGL((mom_batchw_kernel<T, 2>), dim3(g), dim3(kWave), 0, s, ent, begin, par, ninst, total, flip, rows); break;
        case 4: hipLaunchKernelGGL((mom_batchw_kernel<T, 4>), dim3(g), dim3(kWave), 0, s, ent, begin, par, ninst, total, flip, rows); break;
        case 6: hipLaunchKernelGGL((mom_batchw_kernel<T, 6>), dim3(g), dim3(kWave), 0, s, ent, begin, par, ninst, total, flip, rows); break;
        case 7: hipLaunchKernelGGL((mom_batchw_kernel<T, 7>), dim3(g), dim3(kWave), 0, s, ent, begin, par, ninst, total, flip, rows); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int mom_strip_columns(int steps) { return steps == 1 ? kTileX : kWave - 2 * steps; }

template hipError_t launch_batch_mom<double>(const BatchEntry<double>*, const int*, const int*, int, int, int, int, int,
                                             int, hipStream_t);
template hipError_t launch_batch_mom<float>(const BatchEntry<float>*, const int*, const int*, int, int, int, int, int,
                                            int, hipStream_t);

}  // namespace btrtk
