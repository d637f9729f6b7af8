// Moment form of the D2Q9 sweep for k0 = 1 and K2 = k0 (all second-order rates 1): the choice of
// most problems of the paper (Zhao, Wu, Chai & Shi, arXiv:1902.09813).
//
// With these rates Eq. (6) leaves nothing of the populations but their zeroth and first moments:
// f_i+ = w_i (g + 3 c_i . q) with g = phi + s and q = j + dB - K1 (j - B + dB/2). A node's whole
// post-collision state is then (phi, qx, qy), and g where a source makes it differ from phi:
// three or four words instead of ten, aligned loads without the nine shifts of a pull, and a
// pull that needs only sums. Since w_i = a_cx a_cy with a_0 = 2/3, a_+-1 = 1/6, the sums of a pull
// split into a sum along the row and one across rows. In units of 1/36, with
//     p = (g + 3 qx)/36, m = (g - 3 qx)/36, r = 3 qy/36,
//     H = 4 g/36 + p(x-1) + m(x+1),  J = p(x-1) - m(x+1),
//     Hr = 4 r + r(x-1) + r(x+1),    Jr = r(x-1) - r(x+1),
//     A+- = H +- Hr, C+- = J +- Jr,
// the pulled moments are (rows y-1 below, y+1 above)
//     phi = 4 H(y) + A+(y-1) + A-(y+1),  jx = 4 J(y) + C+(y-1) + C-(y+1),  jy = A+(y-1) - A-(y+1).
// A Dirichlet side (half-way bounce-back, Eqs. (54)-(56)) replaces a missing node's part by
// 2 w_i phi_w - w_i (g - 3 c_i . q) of the node itself; the sums over the three links of a side
// close (mom_walls). About 50 FP64 operations per update with K1 per node, against 81 in the
// population form, and four lane shifts instead of six.
//
// What bounds it: on large grids the issue of FP64/FP32 instructions (80 VALU lane-instructions per FP64
// update at seven steps, halo and fill included, 131 in the population walker; three words of state move
// per node and launch instead of ten). Counters at 4096^2: FP64 walkers VALU busy 0.80 of the cycles at a clock
// held to 2.04 GHz (2.31 in the one-step kernel); FP32 regions an instruction every 3.1 cycles and SIMD. Short
// strips are bound by their chain instead (1024^2 with walls FP64, 10 rows kept of 18: 0.35 to 0.45 busy), small
// grids by launches (64^2 0.07). Measured per step, population form -> moment form: 4096^2 nonlinear
// FP64 92 -> 47 us, FP32 57 -> 27 us (regions); 1024^2 with walls FP64 14.6 -> 5.7 us; 64^2 FP64 4.1 -> 0.73
// us (blocks).
//
// State after n >= 1 steps: f+(n-1) as (phi(n-1), q(n-1), g(n-1)). At n = 0 the planes already
// hold f+(0) (f(0) = f^eq(phi0), so phi(0) = phi0 and q(0) = B(phi0) pointwise): the first step
// changes the step count alone, and reads at n = 0 take phi(0) from its plane.
#pragma once

#include "btrt_device.h"
#include "btrt_recip.h"

namespace btrtk {

// Planes of the moment state inside a population buffer (f[parity]); phi has its own buffer.
enum MomPlane : int { kMomQx = 0, kMomQy = 1, kMomG = 2 };

template <typename T>
struct MomNode {
    T gs, p, m, r;  // (g, g + 3 qx, g - 3 qx, 3 qy) / 36; all zero for what is not a node
};

template <typename T>
__host__ __device__ __forceinline__ MomNode<T> mom_node(T g, T qx, T qy)
{
    constexpr T c36 = T(1) / T(36), c12 = T(1) / T(12);
    MomNode<T> n;
    n.gs = c36 * g;
    n.p = fmadd(c12, qx, n.gs);
    n.m = fmadd(-c12, qx, n.gs);
    n.r = c12 * qy;
    return n;
}

// Sums along a row at one node, from its own node values and its neighbours' (left: p, r; right:
// m, r).
template <typename T>
struct MomRow {
    T H, J, Ap, Am, Cp, Cm;
};

template <typename T>
__host__ __device__ __forceinline__ MomRow<T> mom_row(T gs, T r, T pl, T rl, T mr, T rr)
{
    MomRow<T> o;
    o.H = fmadd(T(4), gs, pl + mr);
    o.J = pl - mr;
    const T hr = fmadd(T(4), r, rl + rr), jr = rl - rr;
    o.Ap = o.H + hr;
    o.Am = o.H - hr;
    o.Cp = o.J + jr;
    o.Cm = o.J - jr;
    return o;
}

// The parts of a pull that rows y-1 and y supply; row y+1 completes them.
template <typename T>
struct MomPart {
    T phi, jx, jy;
};

template <typename T>
__host__ __device__ __forceinline__ MomPart<T> mom_part(T H, T J, T Ap_below, T Cp_below)
{
    return MomPart<T>{fmadd(T(4), H, Ap_below), fmadd(T(4), J, Cp_below), Ap_below};
}

// The links that cross Dirichlet sides at node values o of the node itself; wv(i, out_x, out_y)
// is phi_w of the link of direction i. Per side: 3 links of weights (1, 4, 1)/36, the parallel
// ones closing to -6 m (x-), -6 p (x+), -6 (g/36 - r) (y-), -6 (g/36 + r) (y+) for the moment across
// the side and 2 r or p - m for the one along it; a link through a corner point belongs to both
// sides' sums and is taken off once.
template <typename T, typename Wall>
__host__ __device__ __forceinline__ void mom_walls(const MomNode<T>& o, bool oxm, bool oxp, bool oym, bool oyp, Wall wv,
                                          MomPart<T>& a)
{
    constexpr T v1 = T(2) / T(9), v5 = T(1) / T(18);
    const T gs = T(0.5) * (o.p + o.m), u2 = o.p - o.m, u = T(0.5) * u2;
    if (oxm) {
        const T a5 = wv(5, true, oym), a8 = wv(8, true, oyp);
        const T t = fmadd(T(-6), o.m, fmadd(v5, a5 + a8, v1 * wv(1, true, false)));
        a.phi = a.phi + t;
        a.jx = a.jx + t;
        a.jy = a.jy + fmadd(T(2), o.r, v5 * (a5 - a8));
    }
    if (oxp) {
        const T a6 = wv(6, true, oym), a7 = wv(7, true, oyp);
        const T t = fmadd(T(-6), o.p, fmadd(v5, a6 + a7, v1 * wv(3, true, false)));
        a.phi = a.phi + t;
        a.jx = a.jx - t;
        a.jy = a.jy + fmadd(T(2), o.r, v5 * (a6 - a7));
    }
    if (oym) {
        const T a5 = wv(5, oxm, true), a6 = wv(6, oxp, true);
        const T t = fmadd(T(-6), gs - o.r, fmadd(v5, a5 + a6, v1 * wv(2, false, true)));
        a.phi = a.phi + t;
        a.jy = a.jy + t;
        a.jx = a.jx + fmadd(v5, a5 - a6, u2);
    }
    if (oyp) {
        const T a8 = wv(8, oxm, true), a7 = wv(7, oxp, true);
        const T t = fmadd(T(-6), gs + o.r, fmadd(v5, a8 + a7, v1 * wv(4, false, true)));
        a.phi = a.phi + t;
        a.jy = a.jy - t;
        a.jx = a.jx + fmadd(v5, a8 - a7, u2);
    }
    if ((oxm || oxp) && (oym || oyp)) {
        auto corner = [&](int i, T cx, T cy) {
            const T t = fmadd(v5, wv(i, true, true), fmadd(cx, u, fmadd(cy, o.r, -gs)));
            a.phi = a.phi - t;
            a.jx = fmadd(-cx, t, a.jx);
            a.jy = fmadd(-cy, t, a.jy);
        };
        if (oxm && oym) corner(5, T(1), T(1));
        if (oxp && oym) corner(6, T(-1), T(1));
        if (oxp && oyp) corner(7, T(-1), T(-1));
        if (oxm && oyp) corner(8, T(1), T(-1));
    }
}

template <typename T>
struct MomState {
    T phi, qx, qy, g;
};

// The collision on the pulled moments: collide() of the population form with k0 = 1 and Q = 0. s is
// the part of the source that does not depend on phi.
template <typename T, bool SRC, int KM>
__host__ __device__ __forceinline__ MomState<T> mom_collide(const SweepArgs<T>& a, const MomPart<T>& f, T phi_prev, T s, int n,
                                                             NodePowers<T>* pows = nullptr)
{
    constexpr int K1M = KM & kK1Mask;
    constexpr bool GEN = (KM & kGen) != 0;
    constexpr T half = T(0.5);
    const T phi = f.phi, jx = f.jx, jy = f.jy;
    const T hbx = half * a.bx, hby = half * a.by;
    T Bx = phi * fmadd(hbx, phi, a.ax);
    T By = phi * fmadd(hby, phi, a.ay);
    T dBx, dBy;
    if (GEN && (a.fcx != T(0) || a.fcy != T(0))) {
        const T pw = abspow(phi, a.fq), pwp = pows ? pows->flux : abspow(phi_prev, a.fq);
        if (pows) pows->flux = pw;
        const T Bxp = fmadd(a.fcx, pwp, phi_prev * fmadd(hbx, phi_prev, a.ax));
        const T Byp = fmadd(a.fcy, pwp, phi_prev * fmadd(hby, phi_prev, a.ay));
        Bx = fmadd(a.fcx, pw, Bx);
        By = fmadd(a.fcy, pw, By);
        dBx = Bx - Bxp;
        dBy = By - Byp;
    } else {
        dBx = fmadd(-phi_prev, fmadd(hbx, phi_prev, a.ax), Bx);
        dBy = fmadd(-phi_prev, fmadd(hby, phi_prev, a.ay), By);
    }
    if (GEN && a.rr != T(0)) {
        const T pr = abspow(phi, a.rp), prp = pows ? pows->source : abspow(phi_prev, a.rp);
        if (pows) pows->source = pr;
        const T R = (a.rr * phi) * (T(1) - pr);
        const T Rp = (a.rr * phi_prev) * (T(1) - prp);
        s = s + fmadd(T(1.5), R, -half * Rp);
    }
    const T hx = fmadd(half, dBx, jx - Bx), hy = fmadd(half, dBy, jy - By);
    MomState<T> o;
    if constexpr (K1M != kK1Const) {
        T a11 = a.m3[0], a12 = a.m3[1], a22 = a.m3[2];
        if constexpr (K1M == kK1Field) {
            a11 = T(3) * a.afield[n];
            a12 = T(3) * a.afield[a.plane + n];
            a22 = T(3) * a.afield[2 * a.plane + n];
        }
        const T g = fmadd(a.beta, phi * phi, T(1));
        const T m11 = fmadd(a11, g, half);
        const T m12 = a12 * g;
        const T m22 = fmadd(a22, g, half);
        const T det = fmadd(m11, m22, -(m12 * m12));
        T rdet;  // as in the population form: the quotient in FP32, two Newton steps in FP64
        if constexpr (sizeof(T) == 4)
            rdet = quotient(det);
        else
            rdet = recip(det);
        const T ux = fmadd(m22, hx, -(m12 * hy));
        const T uy = fmadd(m11, hy, -(m12 * hx));
        o.qx = fmadd(-rdet, ux, jx + dBx);
        o.qy = fmadd(-rdet, uy, jy + dBy);
    } else {
        o.qx = (jx + dBx) - fmadd(a.K11, hx, a.K12 * hy);
        o.qy = (jy + dBy) - fmadd(a.K12, hx, a.K22 * hy);
    }
    o.phi = phi;
    o.g = (SRC || GEN) ? phi + s : phi;  // phi + 0 is phi where the general model has no such source
    return o;
}

// Dirichlet value of a link that crosses a side at node (x, y) in step lvl of the launch.
template <typename T, bool GEN>
__host__ __device__ __forceinline__ T mom_wall(const SweepArgs<T>& a, int x, int y, int lvl, int i, bool ox, bool oy)
{
    if constexpr (GEN)
        return table_wall(a, x, y, lvl, i, ox, oy);
    else
        return side_wall(a.wall, i, ox, oy);
}

// Whether a handle's planes include g (a source or the general model makes it differ from phi).
template <typename T>
__host__ __device__ __forceinline__ bool mom_has_g(const SweepArgs<T>& a)
{
    return a.mom_g != 0;
}

// Moments of the pull at node (x, y) from the planes (the arithmetic of every moment kernel).
template <typename T, bool GEN>
__host__ __device__ __forceinline__ MomPart<T> mom_pull(const SweepArgs<T>& a, int x, int y)
{
    const T* __restrict__ qx = a.fin + kMomQx * a.plane;
    const T* __restrict__ qy = a.fin + kMomQy * a.plane;
    const T* __restrict__ g = mom_has_g(a) ? a.fin + kMomG * a.plane : a.phi_prev;
    const bool oxm = !a.perx && x == 0, oxp = !a.perx && x == a.nx - 1;
    const bool oym = !a.pery && y == 0, oyp = !a.pery && y == a.ny - 1;
    const int xl = x == 0 ? a.nx - 1 : x - 1, xr = x == a.nx - 1 ? 0 : x + 1;
    MomRow<T> row[3];
    MomNode<T> own;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const bool off = d == 0 ? oym : (d == 2 ? oyp : false);
        int yy = y + d - 1;
        yy = yy < 0 ? a.ny - 1 : (yy >= a.ny ? 0 : yy);
        const int b = yy * a.pitch;
        MomNode<T> l{}, c{}, r{};
        if (!off) {
            c = mom_node(g[b + x], qx[b + x], qy[b + x]);
            if (!oxm) l = mom_node(g[b + xl], qx[b + xl], qy[b + xl]);
            if (!oxp) r = mom_node(g[b + xr], qx[b + xr], qy[b + xr]);
        }
        row[d] = mom_row(c.gs, c.r, l.p, l.r, r.m, r.r);
        if (d == 1) own = c;
    }
    MomPart<T> f = mom_part(row[1].H, row[1].J, row[0].Ap, row[0].Cp);
    f.phi = f.phi + row[2].Am;
    f.jx = f.jx + row[2].Cm;
    f.jy = f.jy - row[2].Am;
    if (oxm || oxp || oym || oyp)
        mom_walls(own, oxm, oxp, oym, oyp,
                  [&](int i, bool ox, bool oy) { return mom_wall<T, GEN>(a, x, y, 0, i, ox, oy); }, f);
    return f;
}

// The populations f_i(x, t) the pull stands for (reads of btrt_populations).
template <typename T, bool GEN>
__host__ __device__ __forceinline__ T mom_population(const SweepArgs<T>& a, int x, int y, int i)
{
    const T* __restrict__ qx = a.fin + kMomQx * a.plane;
    const T* __restrict__ qy = a.fin + kMomQy * a.plane;
    const T* __restrict__ g = mom_has_g(a) ? a.fin + kMomG * a.plane : a.phi_prev;
    const int cx = dir_cx(i), cy = dir_cy(i);
    const T w = i == 0 ? Lat<T>::w0 : (i < 5 ? Lat<T>::w1 : Lat<T>::w5);
    int xs = x - cx, ys = y - cy;
    bool ox = false, oy = false;
    if (xs < 0 || xs >= a.nx) { if (a.perx) xs = xs < 0 ? xs + a.nx : xs - a.nx; else ox = true; }
    if (ys < 0 || ys >= a.ny) { if (a.pery) ys = ys < 0 ? ys + a.ny : ys - a.ny; else oy = true; }
    if (!ox && !oy) {
        const int n = ys * a.pitch + xs;
        return w * fmadd(T(3), T(cx) * qx[n] + T(cy) * qy[n], g[n]);
    }
    const int n = y * a.pitch + x;
    const T back = w * fmadd(T(-3), T(cx) * qx[n] + T(cy) * qy[n], g[n]);  // f_opp+ of the node itself
    return bounce(back, T(2) * w, mom_wall<T, GEN>(a, x, y, 0, i, ox, oy));
}

namespace {

// Time-independent source term of node n = (x, y); which kind is uniform over the launch.
template <typename T>
__device__ __forceinline__ T mom_source(const SweepArgs<T>& a, int n, int x, int y)
{
    if (a.src_y) return a.src_amp * a.src[x] * a.src_y[y];
    return a.src[n];
}

template <typename T, bool SRC, int KM>
__device__ __forceinline__ void mom_put(const SweepArgs<T>& a, int n, const MomState<T>& v)
{
    a.phi_out[n] = v.phi;
    a.fout[kMomQx * a.plane + n] = v.qx;
    a.fout[kMomQy * a.plane + n] = v.qy;
    if (SRC || ((KM & kGen) != 0 && a.mom_g)) a.fout[kMomG * a.plane + n] = v.g;
}

// ---- one step per launch: one node per thread -------------------------------------------------
template <typename T, bool SRC, int KM>
__device__ __forceinline__ void mom_tile1(const SweepArgs<T>& a, int tx, int ty, int rows)
{
    const int x = tx * kTileX + static_cast<int>(threadIdx.x % kTileX);
    const int y = ty * rows + static_cast<int>(threadIdx.x / kTileX);
    if (x >= a.nx || y >= a.ny) return;
    const MomPart<T> f = mom_pull<T, (KM & kGen) != 0>(a, x, y);
    const int n = y * a.pitch + x;
    mom_put<T, SRC, KM>(a, n, mom_collide<T, SRC, KM>(a, f, a.phi_prev[n], SRC ? mom_source(a, n, x, y) * a.sfac[0] : T(0), n));
}

template <typename T, bool SRC, int KM>
__global__ __launch_bounds__(kMaxBlock1) void mom_sweep_kernel(SweepArgs<T> a)
{
    const int tile = xcd_tile();
    const int ty = tile / a.tiles_x;
    mom_tile1<T, SRC, KM>(a, tile - ty * a.tiles_x, ty, static_cast<int>(blockDim.x) / kTileX);
}

// ---- K steps per launch: strip walkers ----------------------------------------------------------
// One wavefront walks a strip of 64 C - 2K columns (C adjacent columns per lane) by `rows` rows. In
// iteration r it takes row r of the state from memory (loads issued kMomAhead rows ahead); step
// l + 1 of the launch then updates row r - l - 1 as soon as step l has row r - l: the row's sums
// complete the parts of row r - l - 1 kept from the iteration before. Six values per level, column
// and lane stay in registers between rows (the parts of one row, its phi, and A+, C+ of the newest
// row), so a seven-step FP64 walker of one column per lane needs about half the registers of the
// population walker and three wavefronts share a SIMD.
constexpr int kMomAhead = 2;

template <int K, int C>
struct MomWalk {
    static constexpr int W = kWave * C - 2 * K;  // output columns per strip
};

// What a strip has to handle at Dirichlet sides: nothing (it stays clear of them), the columns at
// x- and x+ alone, or rows at y- and y+ as well. The first two walk without a branch per row, so
// only the first and last band of a walled grid pays for the row checks.
enum MomEdge : int { kEdgeNone = 0, kEdgeX = 1, kEdgeAll = 2 };

template <typename T, int C>
struct MomIn {
    T phi[C], qx[C], qy[C], g[C], s[C];
};

template <typename T, int C, bool SRC, int EDGE>
struct MomLevel {
    T phi4[C], jx4[C];   // the newest row's parts of phi and jx but for what the next row adds
    T phi[C];            // phi of the newest row
    T Ap[2][C], Cp[C];   // A+ of the two newest rows (slots alternate, so no row is copied), C+ of the newest
    T s[SRC ? C : 1];                        // source of the newest row (time independent part)
    MomNode<T> own[EDGE != kEdgeNone ? C : 1];  // node values of the newest row
};

template <bool SRC, int KM>
constexpr int mom_srcg() { return SRC ? 1 : ((KM & kGen) != 0 ? 2 : 0); }

template <typename T, int C>
struct MomLane {
    int x[C];
    bool col[C];          // a node column of the grid
    bool store[C];        // an output column of the strip
    bool oxm[C], oxp[C];  // the columns at the x- and x+ walls
    T srcx[C];            // separable source: amp * sx(x); else 1
    unsigned srco[C];     // separable source: 0; else x (the offset of a source load in its row)
    int ys, ye;           // output rows
};

// SRCG: 0 no g plane, 1 a g plane, 2 as a.mom_g says (the general node model).
template <typename T, int C, bool SRC, int SRCG>
__device__ __forceinline__ void mom_load(const SweepArgs<T>& a, const MomLane<T, C>& L, int y, MomIn<T, C>& in)
{
    const int64_t b = static_cast<int64_t>(y) * a.pitch;
    const T* __restrict__ phi = a.phi_prev + b;
    const T* __restrict__ qx = a.fin + kMomQx * a.plane + b;
    const T* __restrict__ qy = a.fin + kMomQy * a.plane + b;
    const T* __restrict__ g = a.fin + kMomG * a.plane + b;
    const T* __restrict__ s = SRC ? (a.src_y ? a.src_y + y : a.src + b) : nullptr;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const unsigned x = static_cast<unsigned>(L.x[c]);
        in.phi[c] = phi[x];
        in.qx[c] = qx[x];
        in.qy[c] = qy[x];
        if constexpr (SRCG == 1) in.g[c] = g[x];
        if constexpr (SRCG == 2) in.g[c] = a.mom_g ? g[x] : in.phi[c];
        if constexpr (SRC) in.s[c] = s[L.srco[c]];
    }
}

__device__ __forceinline__ int step_row(int y, int ny) { return y + 1 == ny ? 0 : y + 1; }

// One iteration of the walk. y is row r inside the grid, yn the row of the loads to issue (a row of
// the grid also where the walk ends before it: an unconditional load needs no copies to merge its
// values). PH: which A+ slot row r takes. FULL: every level is past its fill rows.
template <typename T, bool SRC, int KM, int K, int C, int EDGE, int PH, bool FULL>
__device__ __forceinline__ void mom_walk_step(const SweepArgs<T>& a, const MomLane<T, C>& L, int r, int y, int yn,
                                              MomIn<T, C>& in, MomLevel<T, C, SRC, EDGE> (&lev)[K])
{
    constexpr int SRCG = mom_srcg<SRC, KM>();
    constexpr bool GEN = (KM & kGen) != 0;
    constexpr bool YWALL = EDGE == kEdgeAll;
    MomState<T> v[C];
    T src[C];  // source of the row the levels pass along
#pragma unroll
    for (int c = 0; c < C; ++c) {
        src[c] = SRC ? L.srcx[c] * in.s[c] : T(0);
        v[c] = MomState<T>{in.phi[c], in.qx[c], in.qy[c], SRCG != 0 ? in.g[c] : in.phi[c]};
    }
    mom_load<T, C, SRC, SRCG>(a, L, yn, in);
    bool row_ok = YWALL ? (a.pery || (r >= 0 && r < a.ny)) : true;  // row r - l is a row of the grid
    int yl = y;  // row r - l inside the grid
#pragma unroll
    for (int l = 0; l < K; ++l) {
        MomNode<T> N[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            T g = v[c].g, qx = v[c].qx, qy = v[c].qy;
            if constexpr (EDGE != kEdgeNone) {
                const bool node = YWALL ? (row_ok && L.col[c]) : L.col[c];
                g = node ? g : T(0);
                qx = node ? qx : T(0);
                qy = node ? qy : T(0);
            }
            N[c] = mom_node(g, qx, qy);
        }
        const T pl = lane_shift<kShr1>(N[C - 1].p), rl = lane_shift<kShr1>(N[C - 1].r);
        const T mr = lane_shift<kShl1>(N[0].m), rr = lane_shift<kShl1>(N[0].r);
        MomLevel<T, C, SRC, EDGE>& S = lev[l];
        const int q = r - l - 1;  // the row step l + 1 updates
        // Row q inside the grid: wrapped, or clamped beyond a Dirichlet side.
        const int yq = YWALL && !a.pery ? (q < 0 ? 0 : (q >= a.ny ? a.ny - 1 : q)) : (yl == 0 ? a.ny - 1 : yl - 1);
        const bool q_ok = YWALL ? (a.pery || (q >= 0 && q < a.ny)) : true;
        const bool go = FULL || q >= L.ys - (K - l - 1);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const MomRow<T> R = mom_row(N[c].gs, N[c].r, c == 0 ? pl : N[c > 0 ? c - 1 : 0].p,
                                        c == 0 ? rl : N[c > 0 ? c - 1 : 0].r, c == C - 1 ? mr : N[c < C - 1 ? c + 1 : c].m,
                                        c == C - 1 ? rr : N[c < C - 1 ? c + 1 : c].r);
            MomPart<T> f{S.phi4[c] + R.Am, S.jx4[c] + R.Cm, S.Ap[PH][c] - R.Am};
            const T prev = S.phi[c];
            if constexpr (EDGE != kEdgeNone) {
                auto wv = [&](int i, bool ox, bool oy) { return mom_wall<T, GEN>(a, L.x[c], yq, l, i, ox, oy); };
                const bool oym = YWALL && !a.pery && q == 0, oyp = YWALL && !a.pery && q == a.ny - 1;
                if (go && q_ok) {
                    if (oym || oyp)  // a row at a wall (uniform): every node has a crossing link
                        mom_walls(S.own[c], L.oxm[c], L.oxp[c], oym, oyp, wv, f);
                    else if (L.oxm[c] || L.oxp[c])
                        mom_walls(S.own[c], L.oxm[c], L.oxp[c], false, false, wv, f);
                }
                S.own[c] = N[c];
            }
            const MomPart<T> next = mom_part(R.H, R.J, S.Ap[1 - PH][c], S.Cp[c]);
            S.phi4[c] = next.phi;
            S.jx4[c] = next.jx;
            S.Ap[PH][c] = R.Ap;
            S.Cp[c] = R.Cp;
            S.phi[c] = v[c].phi;
            T sq = T(0);
            if constexpr (SRC) {
                sq = S.s[c];
                S.s[c] = src[c];
                src[c] = sq;
                sq = sq * a.sfac[l];
            }
            if (go) v[c] = mom_collide<T, SRC, KM>(a, f, prev, sq, yq * a.pitch + L.x[c]);
        }
        if (!go) return;
        yl = yq;
        row_ok = q_ok;
    }
    // Step K's row r - K.
    if (FULL || r - K >= L.ys) {
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (L.store[c]) mom_put<T, SRC, KM>(a, yl * a.pitch + L.x[c], v[c]);
    }
}

// Output rows of band sy: a.rows each, but for the first and last band of a grid with y walls, which
// take a.edge_rows (their walk costs more per row).
template <typename T>
__device__ __forceinline__ void mom_band(const SweepArgs<T>& a, int sy, int& ys, int& ye)
{
    if (a.edge_rows <= 0) {
        ys = sy * a.rows;
        ye = min(ys + a.rows, a.ny);
        return;
    }
    const int e = a.edge_rows;
    ys = sy == 0 ? 0 : (sy == a.tiles_y - 1 ? a.ny - e : e + (sy - 1) * a.rows);
    ye = sy == 0 ? e : (sy == a.tiles_y - 1 ? a.ny : min(ys + a.rows, a.ny - e));
}

template <typename T, bool SRC, int KM, int K, int C, int EDGE>
__device__ __forceinline__ void mom_strip(const SweepArgs<T>& a, int sx, int ys, int ye, int lane)
{
    constexpr int W = MomWalk<K, C>::W;
    constexpr int SRCG = mom_srcg<SRC, KM>();
    constexpr bool YWALL = EDGE == kEdgeAll;
    const int nx = a.nx, ny = a.ny;
    MomLane<T, C> L;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int at = lane * C + c, cx = sx * W - K + at;
        if (EDGE == kEdgeNone || a.perx) {
            L.x[c] = wrap(cx, nx);
            L.col[c] = true;
            L.oxm[c] = L.oxp[c] = false;
        } else {
            L.col[c] = cx >= 0 && cx < nx;
            L.x[c] = cx < 0 ? 0 : (cx >= nx ? nx - 1 : cx);
            L.oxm[c] = cx == 0;
            L.oxp[c] = cx == nx - 1;
        }
        L.store[c] = at >= K && at < kWave * C - K && cx < nx;
        L.srcx[c] = SRC && a.src_y ? a.src_amp * a.src[L.x[c]] : T(1);
        L.srco[c] = SRC && a.src_y ? 0u : static_cast<unsigned>(L.x[c]);
    }
    L.ys = ys;
    L.ye = ye;
    const int r0 = ys - K, r1 = ye + K;
    // Row q inside the grid: wrapped, or clamped beyond a Dirichlet side (its values are not used).
    auto inside = [&](int q) {
        if (!YWALL || a.pery) return wrap(q, ny);
        return q < 0 ? 0 : (q >= ny ? ny - 1 : q);
    };
    MomLevel<T, C, SRC, EDGE> lev[K];
#pragma unroll
    for (int l = 0; l < K; ++l)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            lev[l].phi4[c] = lev[l].jx4[c] = lev[l].phi[c] = lev[l].Ap[0][c] = lev[l].Ap[1][c] = lev[l].Cp[c] = T(0);
            if constexpr (SRC) lev[l].s[c] = T(0);
            if constexpr (EDGE != kEdgeNone) lev[l].own[c] = MomNode<T>{};
        }
    MomIn<T, C> in[kMomAhead];
    mom_load<T, C, SRC, SRCG>(a, L, inside(r0), in[0]);
    mom_load<T, C, SRC, SRCG>(a, L, inside(r0 + 1), in[1]);
    int r = r0;
    const int fill = ys + K;  // step K's first output row completes at iteration ys + K; 2K rows fill
    for (; r < fill; r += 2) {
        mom_walk_step<T, SRC, KM, K, C, EDGE, 0, false>(a, L, r, wrap(r, ny), inside(r + 2), in[0], lev);
        mom_walk_step<T, SRC, KM, K, C, EDGE, 1, false>(a, L, r + 1, wrap(r + 1, ny), inside(r + 3), in[1], lev);
    }
    int y = wrap(r, ny), yn = wrap(r + 2, ny);
    for (; r + 1 < r1; r += 2) {
        mom_walk_step<T, SRC, KM, K, C, EDGE, 0, true>(a, L, r, y, YWALL ? inside(r + 2) : yn, in[0], lev);
        y = step_row(y, ny);
        yn = step_row(yn, ny);
        mom_walk_step<T, SRC, KM, K, C, EDGE, 1, true>(a, L, r + 1, y, YWALL ? inside(r + 3) : yn, in[1], lev);
        y = step_row(y, ny);
        yn = step_row(yn, ny);
    }
    if (r < r1) mom_walk_step<T, SRC, KM, K, C, EDGE, 0, true>(a, L, r, y, YWALL ? inside(r + 2) : yn, in[0], lev);
}

// What strip sx of rows ys .. ye-1 has to handle: kEdgeNone where no lane's column and no row the
// walk reads is at, or beyond, a Dirichlet side.
template <int K, int C, typename T>
__device__ __forceinline__ int mom_edge(const SweepArgs<T>& a, int sx, int ys, int ye)
{
    const int cx0 = sx * MomWalk<K, C>::W - K;
    const bool x_clear = a.perx || (cx0 >= 1 && cx0 + kWave * C - 1 <= a.nx - 2);
    const bool y_clear = a.pery || (ys - K >= 1 && ye - 1 + K <= a.ny - 2);
    return !y_clear ? kEdgeAll : (x_clear ? kEdgeNone : kEdgeX);
}

// (Each wavefront's choice of a walk is uniform; the walks share no data and meet no barrier.)
template <typename T, bool SRC, int KM, int K, int C, bool WALLS>
__device__ __forceinline__ void mom_strip_any(const SweepArgs<T>& a, int sx, int ys, int ye, int lane)
{
    if constexpr (WALLS) {
        const int edge = mom_edge<K, C>(a, sx, ys, ye);
        if (edge == kEdgeAll) {
            mom_strip<T, SRC, KM, K, C, kEdgeAll>(a, sx, ys, ye, lane);
            return;
        }
        if (edge == kEdgeX) {
            mom_strip<T, SRC, KM, K, C, kEdgeX>(a, sx, ys, ye, lane);
            return;
        }
    }
    mom_strip<T, SRC, KM, K, C, kEdgeNone>(a, sx, ys, ye, lane);
}

template <typename T, bool SRC, int KM, int K, int C, bool WALLS>
__global__ __launch_bounds__(kWave* kWalkGroup) void mom_walk_kernel(SweepArgs<T> a)
{
    const int gsize = static_cast<int>(blockDim.x) / kWave;
    const int group = xcd_tile();
    const int groups_x = (a.tiles_x + gsize - 1) / gsize;
    const int sy = group / groups_x;
    const int sx = (group - sy * groups_x) * gsize + static_cast<int>(threadIdx.x / kWave);
    if (sx >= a.tiles_x) return;  // no barrier in the walk
    int ys, ye;
    mom_band(a, sy, ys, ye);
    mom_strip_any<T, SRC, KM, K, C, WALLS>(a, sx, ys, ye, static_cast<int>(threadIdx.x % kWave));
}

// ---- several steps per launch on small grids: one node per thread -------------------------------
// As block_kernel (btrt_device.h): x neighbours by lane shifts, rows through LDS (A+-, C+- of every node,
// four values instead of nine). Each step narrows the valid region by one node per side.
template <typename T, bool SRC, int KM>
__global__ __launch_bounds__(1024) void mom_block_kernel(SweepArgs<T> a, int steps, int log_ex)
{
    constexpr int SRCG = mom_srcg<SRC, KM>();
    constexpr bool GEN = (KM & kGen) != 0;
    extern __shared__ __attribute__((aligned(16))) char block_lds[];
    T* const lds = reinterpret_cast<T*>(block_lds);
    const int E = static_cast<int>(blockDim.x), EX = 1 << log_ex, EY = E >> log_ex;
    const int t = static_cast<int>(threadIdx.x), lx = t & (EX - 1), ly = t >> log_ex;
    const int tile = xcd_tile();
    const int tyi = tile / a.tiles_x, txi = tile - tyi * a.tiles_x;
    const int ux = txi * (EX - 2 * steps) - steps + lx, uy = tyi * (EY - 2 * steps) - steps + ly;
    const bool xin = ux >= 0 && ux < a.nx, yin = uy >= 0 && uy < a.ny;
    const bool node = (a.perx || xin) && (a.pery || yin);
    const int x = a.perx ? wrap(ux, a.nx) : (xin ? ux : 0), y = a.pery ? wrap(uy, a.ny) : (yin ? uy : 0);
    const bool out = xin && yin && lx >= steps && lx < EX - steps && ly >= steps && ly < EY - steps;
    const int n = y * a.pitch + x;
    const bool oxm = !a.perx && x == 0, oxp = !a.perx && x == a.nx - 1;
    const bool oym = !a.pery && y == 0, oyp = !a.pery && y == a.ny - 1;
    const bool edge = node && (oxm || oxp || oym || oyp);
    const int below = ly > 0 ? EX : 0, above = ly < EY - 1 ? EX : 0;
    MomState<T> v{T(0), T(0), T(0), T(0)};
    T src = T(0);
    if (node) {
        v.phi = a.phi_prev[n];
        v.qx = a.fin[kMomQx * a.plane + n];
        v.qy = a.fin[kMomQy * a.plane + n];
        v.g = SRCG == 1 || (SRCG == 2 && a.mom_g) ? a.fin[kMomG * a.plane + n] : v.phi;
        if constexpr (SRC) src = mom_source(a, n, x, y);
    }
    NodePowers<T> pows{T(0), T(0)};
    if constexpr (GEN) pows = node_powers(a, v.phi);
    for (int s = 0; s < steps; ++s) {
        MomNode<T> N = mom_node(v.g, v.qx, v.qy);
        if (!node) N = MomNode<T>{};
        const MomRow<T> R = mom_row(N.gs, N.r, lane_shift<kShr1>(N.p), lane_shift<kShr1>(N.r), lane_shift<kShl1>(N.m),
                                    lane_shift<kShl1>(N.r));
        T* const b = lds + (s & 1) * 4 * E + t;
        b[0 * E] = R.Ap;
        b[1 * E] = R.Cp;
        b[2 * E] = R.Am;
        b[3 * E] = R.Cm;
        __syncthreads();
        const T Ap = b[0 * E - below], Cp = b[1 * E - below], Am = b[2 * E + above], Cm = b[3 * E + above];
        MomPart<T> f = mom_part(R.H, R.J, Ap, Cp);
        f.phi = f.phi + Am;
        f.jx = f.jx + Cm;
        f.jy = f.jy - Am;
        if (edge)
            mom_walls(N, oxm, oxp, oym, oyp,
                      [&](int i, bool ox, bool oy) { return mom_wall<T, GEN>(a, x, y, s, i, ox, oy); }, f);
        v = mom_collide<T, SRC, KM>(a, f, v.phi, SRC ? src * a.sfac[s] : T(0), n, GEN ? &pows : nullptr);
    }
    if (out) mom_put<T, SRC, KM>(a, n, v);
}

// Launches `steps` steps on regions of (1 << log_ex) x (threads >> log_ex) nodes.
template <typename T, bool SRC, int KM>
hipError_t mom_block_launch(SweepArgs<T> a, int steps, int threads, int log_ex, hipStream_t s)
{
    const int tx = (1 << log_ex) - 2 * steps, ty = (threads >> log_ex) - 2 * steps;
    if (steps < 1 || steps > kMaxFuse || tx < 1 || ty < 1) return hipErrorInvalidValue;
    a.tiles_x = (a.nx + tx - 1) / tx;
    a.tiles_y = (a.ny + ty - 1) / ty;
    const unsigned grid = static_cast<unsigned>(a.tiles_x) * static_cast<unsigned>(a.tiles_y);
    hipLaunchKernelGGL((mom_block_kernel<T, SRC, KM>), dim3(grid), dim3(threads), 2 * 4 * threads * sizeof(T), s, a, steps, log_ex);
    return hipGetLastError();
}

}  // namespace
}  // namespace btrtk

#include "btrt_mom_tile.h"

namespace btrtk {
namespace {

// ---- many instances in one launch (see the population form's batched kernels) ---------------
// Arguments of member i at parity p, both uniform: read through the constant address space, into scalar
// registers as a single grid's kernel arguments are. (Plain loads in a loop that also stores come into
// vector registers.)
template <typename T>
__device__ __forceinline__ SweepArgs<T> entry_args(const BatchEntry<T>* ent, int i, int p)
{
    constexpr int kWords = sizeof(SweepArgs<T>) / sizeof(unsigned);
    static_assert(kWords * sizeof(unsigned) == sizeof(SweepArgs<T>), "whole words");
    struct Words {
        unsigned w[kWords];
    };
    using Const = const __attribute__((address_space(4))) unsigned;
    Const* src = (Const*)(&ent[__builtin_amdgcn_readfirstlane(i)].a[__builtin_amdgcn_readfirstlane(p)]);
    Words v;
#pragma unroll
    for (int k = 0; k < kWords; ++k) v.w[k] = src[k];
    return __builtin_bit_cast(SweepArgs<T>, v);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void mom_batch1_kernel(const BatchEntry<T>* __restrict__ ent,
                                                            const int* __restrict__ begin, const int* __restrict__ par,
                                                            int ninst, int total, int flip)
{
    const int g = static_cast<int>(gridDim.x);
    for (int t = xcd_tile(); t < total; t += g) {
        const int i = owner(begin, ninst, t);
        const SweepArgs<T> a = entry_args(ent, i, par[i] ^ flip);
        const int local = t - begin[i];
        const int tiles_x = (a.nx + kTileX - 1) / kTileX;
        const int ty = local / tiles_x, tx = local - ty * tiles_x;
        switch (ent[i].variant) {  // 2 * (a source) + (K1 per node)
            case 0: mom_tile1<T, false, kK1Const>(a, tx, ty, kTileY); break;
            case 1: mom_tile1<T, false, kK1Phi>(a, tx, ty, kTileY); break;
            case 2: mom_tile1<T, true, kK1Const>(a, tx, ty, kTileY); break;
            default: mom_tile1<T, true, kK1Phi>(a, tx, ty, kTileY); break;
        }
    }
}

template <typename T, int K>
__global__ __launch_bounds__(kWave) void mom_batchw_kernel(const BatchEntry<T>* __restrict__ ent,
                                                           const int* __restrict__ begin, const int* __restrict__ par,
                                                           int ninst, int total, int flip, int rows)
{
    const int g = static_cast<int>(gridDim.x);
    const int lane = static_cast<int>(threadIdx.x);
    for (int t = xcd_tile(); t < total; t += g) {
        const int i = owner(begin, ninst, t);
        SweepArgs<T> a = entry_args(ent, i, par[i] ^ flip);
        a.tiles_x = (a.nx + MomWalk<K, 1>::W - 1) / MomWalk<K, 1>::W;
        const int local = t - begin[i];
        const int sy = local / a.tiles_x, sx = local - sy * a.tiles_x;
        const int ys = sy * rows, ye = min(ys + rows, a.ny);
        switch (3 * ent[i].variant + mom_edge<K, 1>(a, sx, ys, ye)) {
            case 0: mom_strip<T, false, kK1Const, K, 1, kEdgeNone>(a, sx, ys, ye, lane); break;
            case 1: mom_strip<T, false, kK1Const, K, 1, kEdgeX>(a, sx, ys, ye, lane); break;
            case 2: mom_strip<T, false, kK1Const, K, 1, kEdgeAll>(a, sx, ys, ye, lane); break;
            case 3: mom_strip<T, false, kK1Phi, K, 1, kEdgeNone>(a, sx, ys, ye, lane); break;
            case 4: mom_strip<T, false, kK1Phi, K, 1, kEdgeX>(a, sx, ys, ye, lane); break;
            case 5: mom_strip<T, false, kK1Phi, K, 1, kEdgeAll>(a, sx, ys, ye, lane); break;
            case 6: mom_strip<T, true, kK1Const, K, 1, kEdgeNone>(a, sx, ys, ye, lane); break;
            case 7: mom_strip<T, true, kK1Const, K, 1, kEdgeX>(a, sx, ys, ye, lane); break;
            case 8: mom_strip<T, true, kK1Const, K, 1, kEdgeAll>(a, sx, ys, ye, lane); break;
            case 9: mom_strip<T, true, kK1Phi, K, 1, kEdgeNone>(a, sx, ys, ye, lane); break;
            case 10: mom_strip<T, true, kK1Phi, K, 1, kEdgeX>(a, sx, ys, ye, lane); break;
            default: mom_strip<T, true, kK1Phi, K, 1, kEdgeAll>(a, sx, ys, ye, lane); break;
        }
    }
}

// ---- launches -----------------------------------------------------------------------------------
// rows per band; edge_rows > 0: rows of the first and last band (grids with y walls of at least
// 2 edge_rows + 1 rows).
template <typename T, bool SRC, int KM, int K, int C>
hipError_t mom_walk_launch(SweepArgs<T> a, int rows, int edge_rows, int group, hipStream_t s)
{
    constexpr int W = MomWalk<K, C>::W;
    a.tiles_x = (a.nx + W - 1) / W;
    a.rows = rows;
    a.edge_rows = !a.pery && a.ny > 2 * edge_rows ? edge_rows : 0;
    a.tiles_y = a.edge_rows > 0 ? 2 + (a.ny - 2 * a.edge_rows + rows - 1) / rows : (a.ny + rows - 1) / rows;
    const int groups_x = (a.tiles_x + group - 1) / group;
    const unsigned grid = static_cast<unsigned>(groups_x) * static_cast<unsigned>(a.tiles_y);
    if (a.perx && a.pery)
        hipLaunchKernelGGL((mom_walk_kernel<T, SRC, KM, K, C, false>), dim3(grid), dim3(kWave * group), 0, s, a);
    else
        hipLaunchKernelGGL((mom_walk_kernel<T, SRC, KM, K, C, true>), dim3(grid), dim3(kWave * group), 0, s, a);
    return hipGetLastError();
}

template <typename T, bool SRC, int KM>
hipError_t mom_one_launch(SweepArgs<T> a, int rows, hipStream_t s)
{
    a.tiles_x = (a.nx + kTileX - 1) / kTileX;
    a.tiles_y = (a.ny + rows - 1) / rows;
    const unsigned grid = static_cast<unsigned>(a.tiles_x) * static_cast<unsigned>(a.tiles_y);
    hipLaunchKernelGGL((mom_sweep_kernel<T, SRC, KM>), dim3(grid), dim3(kTileX * rows), 0, s, a);
    return hipGetLastError();
}

// Columns per lane: two for FP32 from six steps on (one instance of the shifts serves two columns and
// the halo is 12 or 14 of 128 columns instead of 64: 4096^2, seven steps, 27.3 us a step against
// 32.9; FP64, whose six- and seven-step walkers would leave one wavefront per SIMD, 47.3 against
// 47.9 us at five steps, so it keeps one column).
constexpr int mom_walk_columns(int value_bytes, int steps) { return value_bytes == 4 && steps >= 6 ? 2 : 1; }
template <typename T, int K>
constexpr int mom_columns() { return mom_walk_columns(sizeof(T), K); }

// Resident wavefronts per SIMD of one walker instantiation.
template <typename T, bool SRC, int KM, int K, bool WALLS>
int mom_waves_per_simd()
{
    static const int waves = [] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, mom_walk_kernel<T, SRC, KM, K, mom_columns<T, K>(), WALLS>,
                                                         kWave, 0) != hipSuccess || nb < 4)
            nb = 4;
        return nb / 4;
    }();
    return waves;
}

// Rows per strip so that all strips of a launch are resident at once, n to a SIMD: the launch then
// takes about n (rows + 2K) rows of a walk, 2K of them fill, at 0.94 (K >= 6) or 0.72 of the rate
// where a SIMD holds a single wavefront. (FP64, measured: 4096^2, K = 7: 171 rows, two to a SIMD,
// 335 us, 64 rows 383 us; 2048^2: 86 rows, one to a SIMD, 87.8 us, 43 rows, two, 91.3 us; 1024^2,
// K = 4: 10 rows 19.0 us, 8 rows 22.2, 12 rows 20.3, 16 rows 23.5, 20 rows, one to a SIMD, 18.8.)
template <typename T, bool SRC, int KM, int K>
int mom_fit_rows(const SweepArgs<T>& a)
{
    constexpr int W = MomWalk<K, mom_columns<T, K>()>::W;
    const bool walls = !(a.perx && a.pery);
    const int64_t strips = (a.nx + W - 1) / W;
    const int64_t simds = 4LL * device_cus();
    const int most = walls ? mom_waves_per_simd<T, SRC, KM, K, true>() : mom_waves_per_simd<T, SRC, KM, K, false>();
    double best = 0;
    int rows = 0;
    for (int n = 1; n <= most; ++n) {
        int64_t bands = simds * n / strips;
        if (!a.pery && bands > 1) --bands;  // the first and last band are half as high
        bands = std::max<int64_t>(1, std::min<int64_t>(bands, a.ny));
        const int64_t r = (a.ny + bands - 1) / bands;
        const int64_t rounds = (strips * ((a.ny + r - 1) / r) + simds * n - 1) / (simds * n);
        const double cost = static_cast<double>(rounds) * n * (r + 2 * K) / (n == 1 ? (K >= 6 ? 0.94 : 0.72) : 1.0);
        if (rows == 0 || cost < best) {
            best = cost;
            rows = static_cast<int>(r);
        }
    }
    return rows;
}

// steps in use for automatic shapes below 2^20 nodes, where the reported shape is one step per launch:
// a launch costs more than the redundant rows of a short walk.
constexpr int kMomSmall = 4;

// Nodes up to which automatic shapes take the block kernel (one node per thread) instead of regions.
// (FP64 and FP32 hill, us a step: 300^2 blocks 1.15 and 0.95, regions 1.3 and 1.0; 362^2 blocks 1.54 and
// 1.27, regions of 400 x 370 1.30 and 0.99.)
constexpr int64_t kMomBlockNodes = 100000;

template <typename T, bool SRC, int KM>
int mom_fit(const SweepArgs<T>& a, int steps)
{
    switch (steps) {
        case 2: return mom_fit_rows<T, SRC, KM, 2>(a);
        case 4: return mom_fit_rows<T, SRC, KM, 4>(a);
        default: break;
    }
    if constexpr ((KM & kGen) == 0) {
        switch (steps) {
            case 3: return mom_fit_rows<T, SRC, KM, 3>(a);
            case 5: return mom_fit_rows<T, SRC, KM, 5>(a);
            case 6: return mom_fit_rows<T, SRC, KM, 6>(a);
            case 7: return mom_fit_rows<T, SRC, KM, 7>(a);
            default: break;
        }
    }
    return 0;
}

// The automatic shape. Steps per launch as for the population form (resolve_variant); strip rows
// fitted to the slots (fit_rows); the rows reported are those where they are 64 or more from six
// steps on, else the largest of 32, 16, 8 not above them.
template <typename T, bool SRC, int KM>
LaunchCfg mom_resolve(const SweepArgs<T>& a, LaunchCfg cfg)
{
    constexpr bool GEN = (KM & kGen) != 0;
    const int64_t nodes = static_cast<int64_t>(a.nx) * a.ny;
    const bool fp64 = sizeof(T) == 8, periodic = a.perx && a.pery;
    const bool automatic = cfg.steps <= 0;
    if (automatic) {
        const bool deep = !GEN && nodes >= (periodic || fp64 ? (1LL << 22) : (1LL << 24));
        const int use = deep ? (fp64 && !periodic ? kAutoDeepWalls : kAutoDeep) : (nodes >= (1LL << 20) ? kAutoFuse : kMomSmall);
        cfg.steps = nodes < (1LL << 20) ? 1 : (a.mom_16 ? kAutoFuse : use);
        if (use != cfg.steps) {
            cfg.fuse = use;
            cfg.fit_rows = mom_fit<T, SRC, KM>(a, use);
        }
        // Small grids by the block kernel (us a step, four-step walkers and blocks: FP64 64^2 1.35 and 0.73,
        // 256^2 1.60 and 1.11, 512^2 2.39 and 2.27, 700^2 2.91 and 3.50; with walls 64^2 2.40 and 0.86, 512^2
        // 3.94 and 2.27, 700^2 3.90 and 3.65; FP32 512^2 2.04 and 1.58, 700^2 2.51 and 2.34, 1000^2 3.37 and
        // 4.26); the general model as in the population form.
        if (nodes <= (fp64 && periodic ? (1LL << 18) : (1LL << 19))) {
            const BlockShape b = GEN ? block_shape(a.nx, a.ny, 1, 2.5, 2.0, 1.4, true)
                                     : block_shape(a.nx, a.ny, 1, 1.8, fp64 ? 0.19 : 0.16, fp64 ? 0.1 : 0.08, false);
            if (b.steps > 0) {
                cfg.fuse = b.steps;
                cfg.block = b.threads;
            }
        }
        // Above, the region kernel; FP64 only up to 2^20 nodes (2^21 periodic without an A0 field), above which
        // the walkers, which issue fewer instructions an update, are the faster. us a step, walkers and
        // regions: FP32 hill 500^2 1.83 and 1.14, 1024^2 3.22 and 2.42, 2600 x 2200 11.9 and 10.5; with walls
        // and a source 500^2 3.20 and 1.47, 1700 x 900 5.4 and 4.9; FP64 hill 500^2 2.04 and 1.50, 1024^2 4.5
        // and 4.0, 1700 x 900 5.9 and 5.4, 2000^2 13.6 and 14.5; walls 500^2 3.9 and 2.3, 850 x 1200 6.0 and
        // 5.4, 1700 x 900 7.5 and 8.2; A0 field 500^2 3.4 and 2.1, 1300^2 10.4 and 10.9.
        if constexpr (!GEN) {
            const int64_t most = fp64 ? (periodic && (KM & kK1Mask) != kK1Field ? (1LL << 21) : (1LL << 20) - 1) : nodes;
            if (nodes > kMomBlockNodes && nodes <= most) {
                const RegionShape r = mom_region_shape<T, SRC, KM>(a);
                if (r.steps > 0) {
                    cfg.fuse = r.steps;
                    cfg.block = kWave * r.waves;
                    cfg.wrows = r.rows;
                }
            }
        }
    }
    if (cfg.steps != 2) cfg.tile = 0;
    if (cfg.steps == 1) {
        if (cfg.rows <= 0) cfg.rows = kTileY;
        cfg.group = 0;
        return cfg;
    }
    if (cfg.tile) {
        cfg.rows = cfg.group = 0;
        return cfg;
    }
    if (cfg.rows <= 0) {
        const int k = GEN ? (cfg.steps >= 4 ? 4 : 2) : cfg.steps;  // the general model's longest launch
        if (cfg.fit_rows <= 0) cfg.fit_rows = mom_fit<T, SRC, KM>(a, k);
        cfg.rows = 8;
        if (fp64 && cfg.steps >= 6 && cfg.fit_rows >= 64) {
            cfg.rows = cfg.fit_rows;
        } else {
            for (int r : {64, 32, 16}) {
                if (r == 64 && cfg.steps < 6) continue;
                if (cfg.fit_rows >= r) {
                    cfg.rows = r;
                    break;
                }
            }
        }
        if (cfg.group <= 0) cfg.group = 1;
    }
    if (cfg.group <= 0) cfg.group = (cfg.steps < 6 && cfg.rows >= 32) ? kWalkGroup : 1;
    return cfg;
}

// One launch of cfg.steps (1 .. 7; with the general model 1, 2 or 4, or up to 7 in blocks) steps.
template <typename T, bool SRC, int KM>
hipError_t mom_variant(const SweepArgs<T>& a, const LaunchCfg& cfg, hipStream_t s)
{
    if (cfg.steps < 1 || cfg.steps > kMaxFuse) return hipErrorInvalidValue;
    if constexpr ((KM & kGen) == 0) {
        if (cfg.wrows > 0 && cfg.steps > 1) {
            const int waves = cfg.block / kWave;
            switch (cfg.wrows) {
                case 2: return mom_region_launch<T, SRC, KM, 2>(a, cfg.steps, waves, s);
                case 4: return mom_region_launch<T, SRC, KM, 4>(a, cfg.steps, waves, s);
                case 6: return mom_region_launch<T, SRC, KM, 6>(a, cfg.steps, waves, s);
                default: return hipErrorInvalidValue;
            }
        }
    }
    if (cfg.block > 0 && cfg.steps > 1)
        return mom_block_launch<T, SRC, KM>(a, cfg.steps, cfg.block, block_log_ex(cfg.block), s);
    int rows = cfg.fit_rows > 0 ? cfg.fit_rows : cfg.rows;
    if (cfg.steps == 1) {
        rows = cfg.rows;
        if (rows < 1 || rows > kMaxBlock1 / kTileX || (rows & (rows - 1))) rows = kTileY;
        return mom_one_launch<T, SRC, KM>(a, rows, s);
    }
    if (rows <= 0) rows = cfg.tile ? Tile2<T>::TY : 16;
    const int edge = cfg.fit_rows > 0 ? (rows + 1) / 2 : 0;
    const int group = cfg.group == kWalkGroup ? kWalkGroup : 1;
    switch (cfg.steps) {
        case 2: return mom_walk_launch<T, SRC, KM, 2, mom_columns<T, 2>()>(a, rows, edge, group, s);
        case 4: return mom_walk_launch<T, SRC, KM, 4, mom_columns<T, 4>()>(a, rows, edge, group, s);
        default: break;
    }
    if constexpr ((KM & kGen) == 0) {
        switch (cfg.steps) {
            case 3: return mom_walk_launch<T, SRC, KM, 3, mom_columns<T, 3>()>(a, rows, edge, group, s);
            case 5: return mom_walk_launch<T, SRC, KM, 5, mom_columns<T, 5>()>(a, rows, edge, group, s);
            case 6: return mom_walk_launch<T, SRC, KM, 6, mom_columns<T, 6>()>(a, rows, edge, group, s);
            case 7: return mom_walk_launch<T, SRC, KM, 7, mom_columns<T, 7>()>(a, rows, edge, group, s);
            default: break;
        }
    }
    return hipErrorInvalidValue;
}

// Source x K1 mode dispatch (FLAGS: kGen or 0).
#define BTRT_MOM_DISPATCH(FN, FLAGS, ...)                                                             \
    do {                                                                                              \
        const int k1 = kmode & kK1Mask;                                                               \
        if (src_kind != kSrcNone) {                                                                   \
            if (k1 == kK1Field) return FN<T, true, kK1Field | (FLAGS)>(__VA_ARGS__);                  \
            if (k1 == kK1Phi) return FN<T, true, kK1Phi | (FLAGS)>(__VA_ARGS__);                      \
            return FN<T, true, kK1Const | (FLAGS)>(__VA_ARGS__);                                      \
        }                                                                                             \
        if (k1 == kK1Field) return FN<T, false, kK1Field | (FLAGS)>(__VA_ARGS__);                     \
        if (k1 == kK1Phi) return FN<T, false, kK1Phi | (FLAGS)>(__VA_ARGS__);                         \
        return FN<T, false, kK1Const | (FLAGS)>(__VA_ARGS__);                                         \
    } while (0)

template <typename T, int FLAGS>
hipError_t mom_sweep_with(const SweepArgs<T>& a, int src_kind, int kmode, const LaunchCfg& cfg, hipStream_t s)
{
    BTRT_MOM_DISPATCH(mom_variant, FLAGS, a, cfg, s);
}

template <typename T, int FLAGS>
LaunchCfg mom_resolve_with(const SweepArgs<T>& a, int src_kind, int kmode, const LaunchCfg& cfg)
{
    BTRT_MOM_DISPATCH(mom_resolve, FLAGS, a, cfg);
}
#undef BTRT_MOM_DISPATCH

}  // namespace

// Moment-form sweeps, one translation unit per storage type and node model.
hipError_t mom_f64(const SweepArgs<double>& a, int src_kind, int kmode, const LaunchCfg& cfg, hipStream_t s);
hipError_t mom_f32(const SweepArgs<float>& a, int src_kind, int kmode, const LaunchCfg& cfg, hipStream_t s);
hipError_t mom_gen_f64(const SweepArgs<double>& a, int src_kind, int kmode, const LaunchCfg& cfg, hipStream_t s);
hipError_t mom_gen_f32(const SweepArgs<float>& a, int src_kind, int kmode, const LaunchCfg& cfg, hipStream_t s);
LaunchCfg mom_resolve_f64(const SweepArgs<double>& a, int src_kind, int kmode, const LaunchCfg& cfg);
LaunchCfg mom_resolve_f32(const SweepArgs<float>& a, int src_kind, int kmode, const LaunchCfg& cfg);
LaunchCfg mom_resolve_gen_f64(const SweepArgs<double>& a, int src_kind, int kmode, const LaunchCfg& cfg);
LaunchCfg mom_resolve_gen_f32(const SweepArgs<float>& a, int src_kind, int kmode, const LaunchCfg& cfg);

}  // namespace btrtk
