// K steps of the moment form per launch on regions of 64 columns by R rows per wavefront (included by
// btrt_mom.h).
#pragma once

#include <cmath>

namespace btrtk {
namespace {

// Lane j receives lane j-1 (kShr1) or j+1 (kShl1), the outermost lane 0.
template <int CTRL>
__device__ __forceinline__ int lane_shift0_b32(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}

template <int CTRL>
__device__ __forceinline__ float lane_shift0(float v)
{
    return __builtin_bit_cast(float, lane_shift0_b32<CTRL>(__builtin_bit_cast(int, v)));
}

template <int CTRL>
__device__ __forceinline__ double lane_shift0(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = static_cast<unsigned>(lane_shift0_b32<CTRL>(static_cast<int>(static_cast<unsigned>(u))));
    const unsigned hi = static_cast<unsigned>(lane_shift0_b32<CTRL>(static_cast<int>(static_cast<unsigned>(u >> 32))));
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

// Regions along a direction of n nodes, `size` nodes each with `halo` nodes lost on a side: in a periodic
// direction region t starts `halo` before its output. Between walls the first region starts at the first
// node and the last one ends at the last, so a wall costs no halo and no lane lies beyond one, but for
// the far wall of a grid smaller than a region.
struct RegionSpan {
    int start, lo, hi;  // first node; output nodes lo .. hi-1
    bool wall;          // a wall at its first or last node
};

__host__ __device__ __forceinline__ int region_count(int n, int size, int halo, bool periodic)
{
    const int w = size - 2 * halo;
    return periodic ? (n + w - 1) / w : (n <= size ? 1 : 1 + (n - size + w - 1) / w);
}

__host__ __device__ __forceinline__ RegionSpan region_span(int t, int n, int size, int halo, bool periodic)
{
    const int w = size - 2 * halo;
    RegionSpan r;
    if (periodic) {
        r.start = t * w - halo;
        r.lo = t * w;
        r.hi = r.lo + w < n ? r.lo + w : n;
        r.wall = false;
    } else {
        const bool last = t * w + size >= n;
        r.start = last ? (n > size ? n - size : 0) : t * w;
        r.lo = t == 0 ? 0 : t * w + halo;
        r.hi = last ? n : (t + 1) * w + halo;
        r.wall = t == 0 || last;
    }
    return r;
}

// A workgroup of NW wavefronts owns 64 x (NW R) nodes, each lane one column of its wavefront's R rows in
// registers, and takes `steps` steps on them; the valid part narrows by one node per open side and step.
// x neighbours come by lane shifts and rows from the lane's own registers but for the first and last row
// of a wavefront, whose sums (four values a lane) go through LDS, one barrier a step. Where several regions
// share a CU issue bounds it (4096^2 FP32: a VALU instruction every 3.1 cycles and SIMD), in a single round the
// barrier's wait as well (1531 x 977 FP32: VALU busy 0.58 to 0.67). Strip walkers fill 2 K rows per strip, which at the strip heights that fill the chip
// costs up to half of what they compute (1531 x 977, four steps: 14 rows of 22), and a region of six rows
// a lane by 12 wavefronts keeps 0.68 (six steps). The four parts of each row's sums are independent, so a
// wavefront also has more to issue than a walker's chain of levels.
// sfac: the source's factor of each step (a.sfac, or where its memory is).
template <typename T, bool SRC, int KM, int R, bool EDGE, typename F>
__device__ __forceinline__ void mom_region(const SweepArgs<T>& a, F sfac, const RegionSpan& X, const RegionSpan& Y, int steps, T* lds)
{
    constexpr int SRCG = mom_srcg<SRC, KM>();
    const int lane = static_cast<int>(threadIdx.x % kWave);
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
    const int nw = static_cast<int>(blockDim.x) / kWave;
    const int cx = X.start + lane, cy = Y.start + w * R;
    const bool xwall = EDGE && !a.perx, ywall = EDGE && !a.pery;
    const int x = wrap(cx, a.nx);
    const bool oxm = xwall && cx == 0, oxp = xwall && cx == a.nx - 1;
    auto row = [&](int j) { return wrap(cy + j, a.ny); };
    MomState<T> v[R];
    T src[SRC ? R : 1];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int y = row(j), n = y * a.pitch + x;
        v[j].phi = a.phi_prev[n];
        v[j].qx = a.fin[kMomQx * a.plane + n];
        v[j].qy = a.fin[kMomQy * a.plane + n];
        v[j].g = SRCG == 1 ? a.fin[kMomG * a.plane + n] : v[j].phi;
        if constexpr (SRC) src[j] = mom_source(a, n, x, y);
    }
    auto node = [&](int j) { return mom_node(v[j].g, v[j].qx, v[j].qy); };
    auto sums = [&](int j) {
        const MomNode<T> N = node(j);
        if constexpr (EDGE) {  // lane 63 may lie beyond an x+ wall, lane 0 never beyond an x- wall
            const T mr = lane_shift0<kShl1>(N.m), rr = lane_shift0<kShl1>(N.r);
            return mom_row(N.gs, N.r, lane_shift0<kShr1>(N.p), lane_shift0<kShr1>(N.r), oxp ? T(0) : mr, oxp ? T(0) : rr);
        } else {
            return mom_row(N.gs, N.r, lane_shift<kShr1>(N.p), lane_shift<kShr1>(N.r), lane_shift<kShl1>(N.m),
                           lane_shift<kShl1>(N.r));
        }
    };
    // The walls' share of a side's links, one value for the three of them away from the corners.
    T xw[2] = {T(0), T(0)};
    if constexpr (EDGE)
#pragma unroll
        for (int i = 0; i < 2; ++i) xw[i] = fmadd(T(1) / T(18), a.wall[i] + a.wall[i], T(2) / T(9) * a.wall[i]);
    const int plane = kWave * nw;  // [A+, C+ of last rows; A-, C- of first rows][wavefront][lane], two sets in turn
    T* const mine = lds + w * kWave + lane;
    const int below = w > 0 ? kWave : 0, above = w < nw - 1 ? kWave : 0;
#pragma unroll 1
    for (int s = 0; s < steps; ++s) {
        T* const b = mine + (s & 1) * 4 * plane;
        MomRow<T> cur = sums(0);
        const MomRow<T> last = R > 1 ? sums(R - 1) : cur;
        b[0] = last.Ap;
        b[plane] = last.Cp;
        b[2 * plane] = cur.Am;
        b[3 * plane] = cur.Cm;
        __syncthreads();
        T Ap = b[-below], Cp = b[plane - below];
        const T topA = b[2 * plane + above], topC = b[3 * plane + above];
        if (ywall && w == 0) Ap = Cp = T(0);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            MomRow<T> next = cur;
            if (j + 1 < R) next = j + 1 == R - 1 ? last : sums(j + 1);
            MomPart<T> f = mom_part(cur.H, cur.J, Ap, Cp);
            T Am = j + 1 < R ? next.Am : topA, Cm = j + 1 < R ? next.Cm : topC;
            if (ywall && cy + j == a.ny - 1) Am = Cm = T(0);
            f.phi = f.phi + Am;
            f.jx = f.jx + Cm;
            f.jy = f.jy - Am;
            if constexpr (EDGE) {
                const bool oym = ywall && cy + j == 0, oyp = ywall && cy + j == a.ny - 1;
                if (oym || oyp) {  // uniform, one row of a region or two
                    T wall[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        wall[i] = a.wall[i];
                        asm volatile("" : "+v"(wall[i]));  // formed here, not held in registers through the launch
                    }
                    mom_walls(node(j), oxm, oxp, oym, oyp,
                              [&](int i, bool ox, bool oy) { return side_wall(wall, i, ox, oy); }, f);
                } else if (oxm || oxp) {  // mom_walls with one value for the three links of a side
                    const MomNode<T> N = node(j);
                    if (oxm) {
                        const T t = fmadd(T(-6), N.m, xw[0]);
                        f.phi = f.phi + t;
                        f.jx = f.jx + t;
                        f.jy = fmadd(T(2), N.r, f.jy);
                    }
                    if (oxp) {
                        const T t = fmadd(T(-6), N.p, xw[1]);
                        f.phi = f.phi + t;
                        f.jx = f.jx - t;
                        f.jy = fmadd(T(2), N.r, f.jy);
                    }
                }
            }
            Ap = cur.Ap;
            Cp = cur.Cp;
            v[j] = mom_collide<T, SRC, KM>(a, f, v[j].phi, SRC ? src[SRC ? j : 0] * sfac[s] : T(0), row(j) * a.pitch + x);
            cur = next;
        }
    }
    const bool out = cx >= X.lo && cx < X.hi;
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (out && cy + j >= Y.lo && cy + j < Y.hi) mom_put<T, SRC, KM>(a, (cy + j) * a.pitch + cx, v[j]);
}

template <typename T, bool SRC, int KM, int R, bool WALLS, typename F>
__device__ __forceinline__ void mom_region_any(const SweepArgs<T>& a, F sfac, int tx, int ty, int steps, T* lds)
{
    const RegionSpan X = region_span(tx, a.nx, kWave, steps, !WALLS || a.perx);
    const RegionSpan Y = region_span(ty, a.ny, static_cast<int>(blockDim.x) / kWave * R, steps, !WALLS || a.pery);
    // (The choice is uniform over the workgroup: every wavefront meets the same barriers.)
    if constexpr (WALLS) {
        if (X.wall || Y.wall) {
            mom_region<T, SRC, KM, R, true>(a, sfac, X, Y, steps, lds);
            return;
        }
    }
    mom_region<T, SRC, KM, R, false>(a, sfac, X, Y, steps, lds);
}

constexpr int kRegionWaves = 16;  // most wavefronts of a region: 128 registers a lane, which six rows fit

template <typename T, bool SRC, int KM, int R, bool WALLS>
__global__ __launch_bounds__(kWave* kRegionWaves) void mom_region_kernel(SweepArgs<T> a, int steps)
{
    extern __shared__ __attribute__((aligned(16))) char region_lds[];
    const int tile = xcd_tile();
    const int ty = tile / a.tiles_x;
    mom_region_any<T, SRC, KM, R, WALLS>(a, static_cast<const T*>(a.sfac), tile - ty * a.tiles_x, ty, steps, reinterpret_cast<T*>(region_lds));
}

template <typename T>
constexpr unsigned mom_region_lds(int waves) { return 2 * 4 * kWave * static_cast<unsigned>(waves * sizeof(T)); }

// Launches `steps` steps on regions of 64 columns by `waves` times R rows.
template <typename T, bool SRC, int KM, int R>
hipError_t mom_region_launch(SweepArgs<T> a, int steps, int waves, hipStream_t s)
{
    if (steps < 1 || steps > kMaxFuse || waves < 1 || waves > kRegionWaves || waves * R - 2 * steps < 1)
        return hipErrorInvalidValue;
    a.tiles_x = region_count(a.nx, kWave, steps, a.perx);
    a.tiles_y = region_count(a.ny, waves * R, steps, a.pery);
    const unsigned grid = static_cast<unsigned>(a.tiles_x) * static_cast<unsigned>(a.tiles_y);
    const dim3 block(static_cast<unsigned>(kWave * waves));
    if (a.perx && a.pery)
        hipLaunchKernelGGL((mom_region_kernel<T, SRC, KM, R, false>), dim3(grid), block, mom_region_lds<T>(waves), s, a, steps);
    else
        hipLaunchKernelGGL((mom_region_kernel<T, SRC, KM, R, true>), dim3(grid), block, mom_region_lds<T>(waves), s, a, steps);
    return hipGetLastError();
}

// Workgroups of `waves` (8, 12 or 16) wavefronts of one instantiation a CU holds.
template <typename T, bool SRC, int KM, int R, bool WALLS>
int mom_region_resident(int waves)
{
    struct Table {
        int n[3];
    };
    static const Table t = [] {
        Table v;
        for (int i = 0; i < 3; ++i) {
            const int w = 8 + 4 * i;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v.n[i], mom_region_kernel<T, SRC, KM, R, WALLS>, kWave * w,
                                                             mom_region_lds<T>(w)) != hipSuccess || v.n[i] < 1)
                v.n[i] = 1;
        }
        return v;
    }();
    return t.n[(waves - 8) / 4];
}

struct RegionShape {
    int rows = 0, waves = 0, steps = 0;
};

// What a launch of `steps` steps on `regions` regions takes, us: a model fitted on gfx950. A CU takes its
// share of the regions one after another or resident together, a whole number as far as they are few; a
// region's wavefronts spend (c steps + d) per row on the SIMD they share, more while few share it (e) or
// while no second region fills a barrier's wait (q); a launch costs t0 and every step ts.
// (Measured against it, us a step, FP32 periodic and FP64 with walls: 512^2 2 rows, 16 wavefronts, 5 steps
// 1.27 (model 1.28) and 6 steps 2.09 (2.13); 1531 x 977 6 rows, 12 wavefronts, 6 steps 3.27 (3.14) and 6
// rows, 8 wavefronts, 5 steps 6.76 (6.54); 4096^2 6, 16, 7 26.8 (26.1) and 6, 8, 7 60.0 (57.4).)
template <typename T>
double mom_region_cost(int64_t regions, int rows, int waves, int steps, int resident, bool walls)
{
    struct Fit {
        double t0, ts, c, d, e, tail, q;
    };
    const Fit m = sizeof(T) == 8 ? (walls ? Fit{0.11, 1.03, 0.039, 0.451, 0.74, 0.245, 0.167} : Fit{0.49, 0.54, 0.072, 0.336, 0.0, 0.456, 0.15})
                                 : (walls ? Fit{0.67, 0.76, 0.028, 0.293, 0.73, 0.23, 0.195} : Fit{0.92, 0.49, 0.036, 0.20, 0.03, 0.38, 1.10});
    double n = static_cast<double>(regions) / device_cus();
    n = n <= 2 * resident ? std::ceil(n) : n + m.tail;
    const double shared = std::min<double>(n, resident) * waves / 4;
    double t = n * waves / 4 * rows * (steps * m.c + m.d) * (1 + m.e / shared);
    if (resident == 1 && n > 1) t *= 1 + m.q;
    return m.t0 + t + steps * m.ts;
}

// Region shapes tried: two rows only in the largest workgroups (smaller ones were never the best), FP64 six
// rows above eight wavefronts only where all regions are resident (4096^2 with walls, 16 wavefronts, 71 us
// a step against 60), and not with an A0 field, whose six rows do not fit the registers.
template <typename T, int KM>
bool mom_region_try(int rows, int waves, int64_t regions, int resident)
{
    if (rows == 2) return waves == 16;
    if (rows == 6 && sizeof(T) == 8)
        return (KM & kK1Mask) != kK1Field && (waves == 8 || regions <= static_cast<int64_t>(device_cus()) * resident);
    return true;
}

// The cheapest shape for a grid.
template <typename T, bool SRC, int KM>
RegionShape mom_region_shape(const SweepArgs<T>& a)
{
    const bool walls = !(a.perx && a.pery);
    RegionShape best;
    double best_t = 0;
    for (int rows : {2, 4, 6})
        for (int waves : {8, 12, 16}) {
            int resident;
            if (rows == 2)
                resident = walls ? mom_region_resident<T, SRC, KM, 2, true>(waves) : mom_region_resident<T, SRC, KM, 2, false>(waves);
            else if (rows == 4)
                resident = walls ? mom_region_resident<T, SRC, KM, 4, true>(waves) : mom_region_resident<T, SRC, KM, 4, false>(waves);
            else
                resident = walls ? mom_region_resident<T, SRC, KM, 6, true>(waves) : mom_region_resident<T, SRC, KM, 6, false>(waves);
            for (int k = 2; k <= kMaxFuse && waves * rows - 2 * k >= 16; ++k) {
                const int64_t regions = static_cast<int64_t>(region_count(a.nx, kWave, k, a.perx)) *
                                        region_count(a.ny, waves * rows, k, a.pery);
                if (!mom_region_try<T, KM>(rows, waves, regions, resident)) continue;
                const double t = mom_region_cost<T>(regions, rows, waves, k, resident, walls) / k;
                if (best.steps == 0 || t < best_t) {
                    best_t = t;
                    best = RegionShape{rows, waves, k};
                }
            }
        }
    return best;
}

}  // namespace
}  // namespace btrtk
