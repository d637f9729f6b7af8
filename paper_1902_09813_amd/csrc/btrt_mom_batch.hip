// Launchers of the batched kernels of the moment form (btrt_mom.h).

#include "btrt_mom_batch.h"

#include "btrt_mom.h"

namespace btrtk {
namespace {

// ---- many instances in one launch: units are regions ------------------------------------------
// Strips of 16 rows fill 2 K rows each and a small instance has few of them, so a launch's time was one
// strip's chain. us a step, the best strips and regions (sides log-uniform, half with walls): 64
// instances of 32 .. 200 FP32 5.6 (8-row strips; 8.0 with 16) and 3.8, FP64 8.4 and 5.9; 200 of 32 .. 96 FP32
// 6.7 and 4.8; 8 of 64 .. 400 FP32 4.5 and 2.5; 256 of 32 .. 512, whose loads and stores are 69 of the 219 us
// of a seven-step launch, FP32 33.2 and 32.6, FP64 61.0 and 58.1; 12 of 64 .. 1024 FP32 11.9 and 10.6.
template <typename T, int R>
__global__ __launch_bounds__(kWave* kRegionWaves) void mom_batchr_kernel(const BatchEntry<T>* __restrict__ ent,
                                                                         const int* __restrict__ begin,
                                                                         const int* __restrict__ par, int ninst, int total,
                                                                         int flip, int steps)
{
    extern __shared__ __attribute__((aligned(16))) char region_lds[];
    T* const lds = reinterpret_cast<T*>(region_lds);
    const int g = static_cast<int>(gridDim.x);
    for (int t = xcd_tile(); t < total; t += g) {
        const int i = owner(begin, ninst, t);
        const int p = __builtin_amdgcn_readfirstlane(par[i] ^ flip);
        const SweepArgs<T> a = entry_args(ent, i, p);
        // (An index that is not a constant would put the whole of `a` into scratch memory.)
        const auto sfac = (const __attribute__((address_space(4))) T*)(ent[__builtin_amdgcn_readfirstlane(i)].a[p].sfac);
        const int local = __builtin_amdgcn_readfirstlane(t - begin[i]);
        const int tiles_x = region_count(a.nx, kWave, steps, a.perx);
        const int ty = local / tiles_x, tx = local - ty * tiles_x;
        switch (__builtin_amdgcn_readfirstlane(ent[i].variant)) {
            case 0: mom_region_any<T, false, kK1Const, R, true>(a, sfac, tx, ty, steps, lds); break;
            case 1: mom_region_any<T, false, kK1Phi, R, true>(a, sfac, tx, ty, steps, lds); break;
            case 2: mom_region_any<T, true, kK1Const, R, true>(a, sfac, tx, ty, steps, lds); break;
            default: mom_region_any<T, true, kK1Phi, R, true>(a, sfac, tx, ty, steps, lds); break;
        }
        if (t + g < total) __syncthreads();  // the next region reuses the LDS
    }
}

template <typename T, int R>
int mom_batchr_resident(int waves)
{
    struct Table {
        int n[3];
    };
    static const Table t = [] {
        Table v;
        for (int i = 0; i < 3; ++i) {
            const int w = 8 + 4 * i;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v.n[i], mom_batchr_kernel<T, R>, kWave * w,
                                                             mom_region_lds<T>(w)) != hipSuccess || v.n[i] < 1)
                v.n[i] = 1;
        }
        return v;
    }();
    return t.n[(waves - 8) / 4];
}

}  // namespace

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

template <typename T>
hipError_t launch_batch_region(const BatchEntry<T>* ent, const int* begin, const int* par, int ninst, int total, int flip,
                               int steps, int grid, const BatchRegion& r, hipStream_t s)
{
    if (total <= 0 || ninst <= 0) return hipSuccess;
    if (steps < 2 || steps > kMaxFuse || r.waves < 8 || r.waves > kRegionWaves || r.rows * r.waves - 2 * steps < 1)
        return hipErrorInvalidValue;
    const dim3 g(static_cast<unsigned>(grid > 0 ? std::min(grid, total) : total)), block(static_cast<unsigned>(kWave * r.waves));
    const unsigned lds = mom_region_lds<T>(r.waves);
    switch (r.rows) {
        case 2: hipLaunchKernelGGL((mom_batchr_kernel<T, 2>), g, block, lds, s, ent, begin, par, ninst, total, flip, steps); break;
        case 4: hipLaunchKernelGGL((mom_batchr_kernel<T, 4>), g, block, lds, s, ent, begin, par, ninst, total, flip, steps); break;
        case 6: hipLaunchKernelGGL((mom_batchr_kernel<T, 6>), g, block, lds, s, ent, begin, par, ninst, total, flip, steps); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int64_t batch_regions(const BatchGrid& g, int steps, int rows)
{
    return static_cast<int64_t>(region_count(g.nx, kWave, steps, g.perx)) * region_count(g.ny, rows, steps, g.pery);
}

template <typename T>
BatchRegion batch_region(const BatchGrid* grids, int n, int steps)
{
    BatchRegion best;
    bool walls = false;
    for (int i = 0; i < n; ++i) walls = walls || !grids[i].perx || !grids[i].pery;
    for (int rows : {2, 4, 6})
        for (int waves : {8, 12, 16}) {
            if (waves * rows - 2 * steps < 16) continue;
            int64_t regions = 0;
            for (int i = 0; i < n; ++i) regions += batch_regions(grids[i], steps, rows * waves);
            const int resident = rows == 2 ? mom_batchr_resident<T, 2>(waves)
                                           : (rows == 4 ? mom_batchr_resident<T, 4>(waves) : mom_batchr_resident<T, 6>(waves));
            if (!mom_region_try<T, kK1Const>(rows, waves, regions, resident)) continue;
            const double t = mom_region_cost<T>(regions, rows, waves, steps, resident, walls);
            if (best.rows == 0 || t < best.cost) best = BatchRegion{rows, waves, t};
        }
    return best;
}

template hipError_t launch_batch_region<double>(const BatchEntry<double>*, const int*, const int*, int, int, int, int, int,
                                                const BatchRegion&, hipStream_t);
template hipError_t launch_batch_region<float>(const BatchEntry<float>*, const int*, const int*, int, int, int, int, int,
                                               const BatchRegion&, hipStream_t);
template BatchRegion batch_region<double>(const BatchGrid*, int, int);
template BatchRegion batch_region<float>(const BatchGrid*, int, int);

int mom_strip_columns(int steps) { return steps == 1 ? kTileX : kWave - 2 * steps; }

template hipError_t launch_batch_mom<double>(const BatchEntry<double>*, const int*, const int*, int, int, int, int, int,
                                             int, hipStream_t);
template hipError_t launch_batch_mom<float>(const BatchEntry<float>*, const int*, const int*, int, int, int, int, int,
                                            int, hipStream_t);

}  // namespace btrtk
