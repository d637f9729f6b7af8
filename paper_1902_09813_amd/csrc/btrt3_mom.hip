// gfx950 kernels of the D3Q19 moment form (btrt3_mom.h).

#include "btrt3_mom.h"

#include <algorithm>

namespace btrt3k {
namespace {

constexpr int kWave = 64;
constexpr int kShr1 = 0x138;  // DPP wave_shr:1, lane j receives lane j-1
constexpr int kShl1 = 0x130;  // DPP wave_shl:1, lane j receives lane j+1

template <int CTRL>
__device__ __forceinline__ float lane_shift(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

template <int CTRL>
__device__ __forceinline__ double lane_shift(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_mov_dpp(static_cast<int>(static_cast<unsigned>(u)), CTRL, 0xf, 0xf, false));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_mov_dpp(static_cast<int>(static_cast<unsigned>(u >> 32)), CTRL, 0xf, 0xf, false));
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

__device__ __forceinline__ int xcd_tile()
{
    const int b = static_cast<int>(blockIdx.x);
    const int nb = static_cast<int>(gridDim.x);
    const int q = nb >> 3, r = nb & 7, k = b & 7, j = b >> 3;
    return k * q + (k < r ? k : r) + j;
}

__device__ __forceinline__ int wrap3(int v, int n)
{
    const int r = v % n;
    return r < 0 ? r + n : r;
}

// K steps per launch: a workgroup of NW wavefronts owns a tile of 64 x NW R columns (R rows per
// lane), K of them halo on each side, and walks z over a.zc output planes. In iteration z it takes
// plane z of the state from memory (loads issued a plane ahead); step l + 1 updates plane z - l - 1 as
// soon as step l has plane z - l. x neighbours come by lane shifts, the rows beside a lane's own
// through LDS (eight values per lane, level and plane; one barrier per level), planes from eight
// values per column and level in registers. (What bounds it: btrt3_mom.h.)
//
// The values of level l are written again only after every wavefront has read them: with K >= 2 the
// barrier of another level lies between, with K = 1 the planes alternate between two buffers.
template <int K>
constexpr int mom3_buffers() { return K == 1 ? 2 : K; }

template <typename T, int R, bool SRC, bool WALLS>
struct Mom3Level {
    T phi[R], jx[R], jy[R], jz[R];  // of the newest plane but for what the next one adds (jz: U of the plane below)
    T U[R], Ux[R], Uy[R];           // of the newest plane
    T prev[R];                      // phi of the newest plane
    T s[SRC ? R : 1];               // source of the newest plane
    Mom3Node<T> own[WALLS ? R : 1];
};

template <typename T, int R>
struct Mom3In {
    T phi[R], qx[R], qy[R], qz[R], g[R], s[R];
};

template <typename T, bool SRC, bool KPHI, bool WALLS, int K, int NW, int R>
__global__ __launch_bounds__(kWave* NW) void mom3_kernel(Sweep3<T> a)
{
    constexpr int TX = kWave - 2 * K, TY = NW * R - 2 * K;
    constexpr int NB = mom3_buffers<K>();
    __shared__ T sh[NB][2][4][NW][kWave];

    const int t = xcd_tile();
    const int per_chunk = a.tiles_x * a.tiles_y;
    const int chunk = t / per_chunk;
    const int rr = t - chunk * per_chunk;
    const int tyi = rr / a.tiles_x, txi = rr - tyi * a.tiles_x;
    const int lane = static_cast<int>(threadIdx.x % kWave);
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));  // uniform: rows are scalar

    const int ux = txi * TX - K + lane;
    const bool xin = ux >= 0 && ux < a.nx;
    const int x = !WALLS || a.per[0] ? wrap3(ux, a.nx) : (ux < 0 ? 0 : (ux >= a.nx ? a.nx - 1 : ux));
    const bool xnode = !WALLS || a.per[0] || xin;
    int col[R];                 // y * pitch + x
    bool node[R], store[R];
    bool oym[R], oyp[R];        // the row is at a y face (uniform in a wavefront, as z faces are)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int at = wv * R + r, uy = tyi * TY - K + at;
        const bool yin = uy >= 0 && uy < a.ny;
        const int y = !WALLS || a.per[1] ? wrap3(uy, a.ny) : (uy < 0 ? 0 : (uy >= a.ny ? a.ny - 1 : uy));
        node[r] = xnode && (!WALLS || a.per[1] || yin);
        store[r] = lane >= K && lane < kWave - K && at >= K && at < NW * R - K && xin && yin;
        oym[r] = WALLS && !a.per[1] && uy == 0;
        oyp[r] = WALLS && !a.per[1] && uy == a.ny - 1;
        col[r] = y * a.pitch + x;
    }
    const bool oxm = WALLS && !a.per[0] && ux == 0, oxp = WALLS && !a.per[0] && ux == a.nx - 1;
    const int z0 = chunk * a.zc, z1 = min(z0 + a.zc, a.nz);

    auto inside = [&](int z) {  // plane z inside the box: wrapped, or clamped beyond a Dirichlet face
        if (!WALLS || a.per[2]) return wrap3(z, a.nz);
        return z < 0 ? 0 : (z >= a.nz ? a.nz - 1 : z);
    };
    auto plane_ok = [&](int z) { return !WALLS || a.per[2] || (z >= 0 && z < a.nz); };
    auto load = [&](int z, Mom3In<T, R>& in) {
        const int64_t b = static_cast<int64_t>(inside(z)) * a.slab;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned n = static_cast<unsigned>(col[r]);
            in.phi[r] = (a.phi_prev + b)[n];
            in.qx[r] = (a.fin + kM3Qx * a.plane + b)[n];
            in.qy[r] = (a.fin + kM3Qy * a.plane + b)[n];
            in.qz[r] = (a.fin + kM3Qz * a.plane + b)[n];
            if constexpr (SRC) {
                in.g[r] = (a.fin + kM3G * a.plane + b)[n];
                in.s[r] = (a.src + b)[n];
            }
        }
    };

    Mom3Level<T, R, SRC, WALLS> lev[K];
#pragma unroll
    for (int l = 0; l < K; ++l)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            lev[l].phi[r] = lev[l].jx[r] = lev[l].jy[r] = lev[l].jz[r] = T(0);
            lev[l].U[r] = lev[l].Ux[r] = lev[l].Uy[r] = lev[l].prev[r] = T(0);
            if constexpr (SRC) lev[l].s[r] = T(0);
            if constexpr (WALLS) lev[l].own[r] = Mom3Node<T>{};
        }
    Mom3In<T, R> in;
    load(z0 - K, in);
    for (int z = z0 - K; z < z1 + K; ++z) {
        Mom3State<T> v[R];
        T src[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[r] = Mom3State<T>{in.phi[r], in.qx[r], in.qy[r], in.qz[r], SRC ? in.g[r] : in.phi[r]};
            src[r] = SRC ? in.s[r] : T(0);
        }
        load(z + 1 < z1 + K ? z + 1 : z, in);
#pragma unroll
        for (int l = 0; l < K; ++l) {
            const bool pz = plane_ok(z - l);
            Mom3Row<T> row[R];
            Mom3Node<T> N[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                T g = v[r].g, qx = v[r].qx, qy = v[r].qy, qz = v[r].qz;
                if constexpr (WALLS) {
                    const bool ok = pz && node[r];
                    g = ok ? g : T(0);
                    qx = ok ? qx : T(0);
                    qy = ok ? qy : T(0);
                    qz = ok ? qz : T(0);
                }
                N[r] = mom3_node(g, qx, qy, qz);
                const T p = N[r].g + N[r].b, m = N[r].g - N[r].b;
                row[r] = mom3_row(N[r], lane_shift<kShr1>(p), lane_shift<kShr1>(N[r].c), lane_shift<kShr1>(N[r].d),
                                  lane_shift<kShl1>(m), lane_shift<kShl1>(N[r].c), lane_shift<kShl1>(N[r].d));
            }
            T(&buf)[2][4][NW][kWave] = sh[K == 1 ? (z & 1) : l];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                buf[0][k][wv][lane] = row[R - 1].up[k];
                buf[1][k][wv][lane] = row[0].dn[k];
            }
            __syncthreads();
            T below[4], above[4];  // the rows beside this lane's (the tile's first and last row: not used)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                below[k] = buf[0][k][wv > 0 ? wv - 1 : 0][lane];
                above[k] = buf[1][k][wv < NW - 1 ? wv + 1 : wv][lane];
            }
            Mom3Level<T, R, SRC, WALLS>& S = lev[l];
            const int q = z - l - 1;  // the plane step l + 1 updates
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const Mom3Plane3<T> P = mom3_plane(row[r], r == 0 ? below : row[r > 0 ? r - 1 : 0].up,
                                                   r == R - 1 ? above : row[r < R - 1 ? r + 1 : r].dn);
                Mom3Sum<T> f{S.phi[r] + P.D, S.jx[r] + P.Dx, S.jy[r] + P.Dy, S.jz[r] - P.D};
                const T prev = S.prev[r];
                if constexpr (WALLS) {
                    const bool ozm = !a.per[2] && q == 0, ozp = !a.per[2] && q == a.nz - 1;
                    if (oym[r] || oyp[r] || ozm || ozp) {
                        const bool out[6] = {oxm, oxp, oym[r], oyp[r], ozm, ozp};
                        mom3_walls(S.own[r], out, a.wall, f);
                    } else if (oxm || oxp) {  // away from rows and planes at a face: the x faces alone
                        const bool out[6] = {oxm, oxp, false, false, false, false};
                        mom3_walls(S.own[r], out, a.wall, f);
                    }
                    S.own[r] = N[r];
                }
                S.phi[r] = P.M + S.U[r];
                S.jx[r] = P.Mx + S.Ux[r];
                S.jy[r] = P.My + S.Uy[r];
                S.jz[r] = S.U[r];
                S.U[r] = P.U;
                S.Ux[r] = P.Ux;
                S.Uy[r] = P.Uy;
                S.prev[r] = v[r].phi;
                T sq = T(0);
                if constexpr (SRC) {
                    sq = S.s[r];
                    S.s[r] = src[r];
                    src[r] = sq;
                }
                v[r] = mom3_collide<T, SRC, KPHI>(a, f, prev, sq);
            }
        }
        const int q = z - K;
        if (q >= z0) {
            const int64_t b = static_cast<int64_t>(q) * a.slab;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (store[r]) {
                    const unsigned n = static_cast<unsigned>(col[r]);
                    (a.phi_out + b)[n] = v[r].phi;
                    (a.fout + kM3Qx * a.plane + b)[n] = v[r].qx;
                    (a.fout + kM3Qy * a.plane + b)[n] = v[r].qy;
                    (a.fout + kM3Qz * a.plane + b)[n] = v[r].qz;
                    if constexpr (SRC) (a.fout + kM3G * a.plane + b)[n] = v[r].g;
                }
        }
    }
}

// ---- reads and set-up ---------------------------------------------------------------------------
constexpr int kBlock = 256;

// f+(0) pointwise from phi0, in FP64 and rounded once, as in init3_kernel.
template <typename T>
__global__ __launch_bounds__(kBlock) void mom3_init_kernel(Sweep3<T> a, const double* __restrict__ phi0)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (k >= static_cast<int64_t>(a.nx) * a.ny * a.nz) return;
    const int64_t row = k / a.nx;
    const int64_t n = row * a.pitch + (k - row * a.nx);
    const double p = phi0[k];
    a.phi_out[n] = static_cast<T>(p);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        a.fout[c * a.plane + n] = static_cast<T>(p * (static_cast<double>(a.a[c]) + 0.5 * static_cast<double>(a.b[c]) * p));
    if (a.src) a.fout[kM3G * a.plane + n] = static_cast<T>(p + static_cast<double>(a.src[n]));
}

template <typename T, bool SRC, bool KPHI, bool WALLS, int K, int NW, int R>
hipError_t mom3_launch(Sweep3<T> a, int zc, hipStream_t s)
{
    a.tiles_x = (a.nx + kWave - 2 * K - 1) / (kWave - 2 * K);
    a.tiles_y = (a.ny + NW * R - 2 * K - 1) / (NW * R - 2 * K);
    a.zc = zc;
    const int64_t wg = static_cast<int64_t>(a.tiles_x) * a.tiles_y * ((a.nz + zc - 1) / zc);
    if (zc < 1 || wg > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((mom3_kernel<T, SRC, KPHI, WALLS, K, NW, R>), dim3(static_cast<unsigned>(wg)), dim3(kWave * NW), 0, s, a);
    return hipGetLastError();
}

// Tiles: one step per launch 64 x 8 columns (many small workgroups), two steps 64 x 16 with two rows
// per lane (60 x 12 of them output). 256^3 FP64, us a step at the best chunk (with a reciprocal of two Newton
// steps; the third and the fixup cost 6 us more): two steps with 8
// wavefronts of two rows 205, 12 of one row 204, 16 of one row (spills) 429, 8 of one row 256; FP32: 103,
// 16 of one row 121, 16 of two rows 119, 8 of four rows 116.
constexpr int kNW = 8;
constexpr int rows_per_lane(int steps) { return steps == 2 ? 2 : 1; }

template <typename T, bool SRC, bool KPHI, bool WALLS>
hipError_t mom3_steps(const Sweep3<T>& a, int steps, int zc, hipStream_t s)
{
    if (steps == 2) return mom3_launch<T, SRC, KPHI, WALLS, 2, kNW, rows_per_lane(2)>(a, zc, s);
    return mom3_launch<T, SRC, KPHI, WALLS, 1, kNW, rows_per_lane(1)>(a, zc, s);
}

template <typename T, bool SRC, bool KPHI, bool WALLS>
int mom3_occupancy(int steps)
{
    int nb = 0;
    const hipError_t e = steps == 2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, mom3_kernel<T, SRC, KPHI, WALLS, 2, kNW, rows_per_lane(2)>, kWave * kNW, 0)
                                    : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, mom3_kernel<T, SRC, KPHI, WALLS, 1, kNW, rows_per_lane(1)>, kWave * kNW, 0);
    return e == hipSuccess && nb > 0 ? nb : 1;
}

#define BTRT3_MOM_DISPATCH(FN, ...)                                                              \
    do {                                                                                         \
        const bool walls = !(a.per[0] && a.per[1] && a.per[2]);                                  \
        if (a.src) {                                                                             \
            if (k1_per_node) return walls ? FN<T, true, true, true>(__VA_ARGS__) : FN<T, true, true, false>(__VA_ARGS__); \
            return walls ? FN<T, true, false, true>(__VA_ARGS__) : FN<T, true, false, false>(__VA_ARGS__);               \
        }                                                                                        \
        if (k1_per_node) return walls ? FN<T, false, true, true>(__VA_ARGS__) : FN<T, false, true, false>(__VA_ARGS__);  \
        return walls ? FN<T, false, false, true>(__VA_ARGS__) : FN<T, false, false, false>(__VA_ARGS__);                 \
    } while (0)

}  // namespace

template <typename T>
hipError_t launch3_mom(const Sweep3<T>& a, bool k1_per_node, int steps, int zc, hipStream_t s)
{
    if (steps != 1 && steps != 2) return hipErrorInvalidValue;
    BTRT3_MOM_DISPATCH(mom3_steps, a, steps, zc, s);
}

template <typename T>
int mom3_blocks_per_cu(const Sweep3<T>& a, bool k1_per_node, int steps)
{
    BTRT3_MOM_DISPATCH(mom3_occupancy, steps);
}

int64_t mom3_workgroups(int nx, int ny, int nz, int steps, int zc)
{
    const int tx = kWave - 2 * steps, ty = kNW * rows_per_lane(steps) - 2 * steps;
    return static_cast<int64_t>((nx + tx - 1) / tx) * ((ny + ty - 1) / ty) * ((nz + zc - 1) / zc);
}

template <typename T>
hipError_t launch3_mom_init(const Sweep3<T>& a, const double* phi0, hipStream_t s)
{
    const int64_t nn = static_cast<int64_t>(a.nx) * a.ny * a.nz;
    hipLaunchKernelGGL((mom3_init_kernel<T>), dim3(static_cast<unsigned>((nn + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a, phi0);
    return hipGetLastError();
}

#define BTRT3_MOM_INSTANTIATE(T)                                                             \
    template hipError_t launch3_mom<T>(const Sweep3<T>&, bool, int, int, hipStream_t);       \
    template int mom3_blocks_per_cu<T>(const Sweep3<T>&, bool, int);                         \
    template hipError_t launch3_mom_init<T>(const Sweep3<T>&, const double*, hipStream_t);

BTRT3_MOM_INSTANTIATE(double)
BTRT3_MOM_INSTANTIATE(float)

}  // namespace btrt3k
