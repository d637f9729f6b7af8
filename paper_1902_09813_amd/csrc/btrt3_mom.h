// Moment form of the D3Q19 sweep for k0 = 1 and K2 = 1 (every second-order rate 1), the counterpart
// of btrt_mom.h: f_i+ = w_i (g + 3 c_i . q) with g = phi + s, so a node's state is (phi, q) and, with a
// source, g: four or five words instead of twenty.
//
// In units of 1/36, with (g, b, c, d) = (g, 3 qx, 3 qy, 3 qz)/36, p = g + b, m = g - b and _L, _R the
// values of the nodes at x-1, x+1, every node forms
//     sp = p_L + m_R, dp = p_L - m_R, sc = c_L + c_R, dc = c_L - c_R, sd = d_L + d_R, dd = d_L - d_R,
//     R+- = 2 g + sp +- (2 c + sc), Rx+- = dp +- dc       (what a node of row y+-1 pulls in this plane)
//     V+- = 2 g + sp +- (2 d + sd), Vx+- = dp +- dd       (what a node of plane z+-1 pulls from this row)
// and with t+- = g +- c of the rows y-1 (below) and y+1 (above)
//     M  = 12 g + 2 sp + R+(y-1) + R-(y+1),  Mx = 2 dp + Rx+(y-1) + Rx-(y+1),  My = R+(y-1) - R-(y+1),
//     U  = V+ + t+(y-1) + d(y-1) + t-(y+1) + d(y+1),  D = the same with -d and V-,
//     Uy = t+(y-1) - t-(y+1) + d(y-1) - d(y+1),  Dy with -d,  Ux = Vx+, Dx = Vx-,
// so that phi = M(z) + U(z-1) + D(z+1), jx = Mx + Ux + Dx, jy = My + Uy + Dy, jz = U(z-1) - D(z+1).
// A Dirichlet face (half-way bounce-back) replaces the part of a missing node; the sums over the five
// links of a face close (mom3_walls), links through an edge of the box taking the mean of two faces.
//
// What bounds it: with one step per launch the words it moves (256^3 FP64, 1.07 GB in 243 us). With two,
// FP32 the issue of its instructions (VALU busy 0.98), FP64 the waits that two wavefronts a SIMD leave open (0.53
// busy at 2.03 GHz; 242 VALU lane-instructions per update, 0.63 of a tile kept). Measured per step, population
// form -> moment form: 256^3 nonlinear FP64 687 -> 218 us, FP32 421 -> 110 us; 125^3 FP64 137 -> 33 us; 20^3 FP64 8.2 -> 5.2 us.
//
// State after n >= 1 steps: f+(n-1) as phi(n-1), q(n-1), g(n-1). At n = 0 the planes already hold f+(0)
// (pointwise from phi0): the first step changes the step count alone.
#pragma once

#include "btrt3_internal.h"
#include "btrt_recip.h"

namespace btrt3k {

enum Mom3Plane : int { kM3Qx = 0, kM3Qy = 1, kM3Qz = 2, kM3G = 3 };

template <typename T>
__host__ __device__ __forceinline__ T fma3(T a, T b, T c)
{
    if constexpr (sizeof(T) == 4)
        return fmaf(a, b, c);
    else
        return fma(a, b, c);
}

template <typename T>
struct Mom3Node {
    T g, b, c, d;  // all zero for what is not a node
};

template <typename T>
__host__ __device__ __forceinline__ Mom3Node<T> mom3_node(T g, T qx, T qy, T qz)
{
    constexpr T c36 = T(1) / T(36), c12 = T(1) / T(12);
    return Mom3Node<T>{c36 * g, c12 * qx, c12 * qy, c12 * qz};
}

// What a node passes on along its row: to rows y+1 (up) and y-1 (dn) and to the planes z+-1.
template <typename T>
struct Mom3Row {
    T M, Mx;              // 12 g + 2 sp, 2 dp
    T Vp, Vm, Vxp, Vxm;   // V+-, Vx+-
    T up[4], dn[4];       // (R+, Rx+, t+, d) and (R-, Rx-, t-, d)
};

template <typename T>
__host__ __device__ __forceinline__ Mom3Row<T> mom3_row(const Mom3Node<T>& o, T pl, T cl, T dl, T mr, T cr, T dr)
{
    Mom3Row<T> r;
    const T sp = pl + mr, dp = pl - mr, sc = cl + cr, dc = cl - cr, sd = dl + dr, dd = dl - dr;
    const T e = fma3(T(2), o.g, sp), ec = fma3(T(2), o.c, sc), ed = fma3(T(2), o.d, sd);
    r.M = fma3(T(2), sp, T(12) * o.g);
    r.Mx = T(2) * dp;
    r.Vp = e + ed;
    r.Vm = e - ed;
    r.Vxp = dp + dd;
    r.Vxm = dp - dd;
    r.up[0] = e + ec;
    r.up[1] = dp + dc;
    r.up[2] = o.g + o.c;
    r.up[3] = o.d;
    r.dn[0] = e - ec;
    r.dn[1] = dp - dc;
    r.dn[2] = o.g - o.c;
    r.dn[3] = o.d;
    return r;
}

// Sums of one plane at one node: M (for the node itself), U (for z+1) and D (for z-1).
template <typename T>
struct Mom3Plane3 {
    T M, Mx, My, U, Ux, Uy, D, Dx, Dy;
};

// below: the up values of the node at y-1, above: the dn values of the node at y+1.
template <typename T>
__host__ __device__ __forceinline__ Mom3Plane3<T> mom3_plane(const Mom3Row<T>& r, const T below[4], const T above[4])
{
    Mom3Plane3<T> p;
    p.M = r.M + (below[0] + above[0]);
    p.Mx = r.Mx + (below[1] + above[1]);
    p.My = below[0] - above[0];
    const T t = below[2] + above[2], u = below[2] - above[2], d = below[3] + above[3], e = below[3] - above[3];
    p.U = r.Vp + (t + d);
    p.D = r.Vm + (t - d);
    p.Ux = r.Vxp;
    p.Dx = r.Vxm;
    p.Uy = u + e;
    p.Dy = u - e;
    return p;
}

template <typename T>
struct Mom3Sum {
    T phi, jx, jy, jz;
};

// Links that cross Dirichlet faces at the node with values o: out[f] for faces x-, x+, y-, y+, z-, z+.
template <typename T>
__host__ __device__ __forceinline__ void mom3_walls(const Mom3Node<T>& o, const bool out[6], const T w[6], Mom3Sum<T>& s)
{
    constexpr T v1 = T(1) / T(18);  // 2 w_i of a diagonal link; an axis link has twice that
    const T q[3] = {o.b, o.c, o.d};
    T j[3] = {s.jx, s.jy, s.jz};
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        if (!out[f]) continue;
        const int ax = f / 2;
        const T sg = (f & 1) ? T(-1) : T(1);  // the crossing links come in along sg e_ax
        T v = T(4) * w[f];  // values of the five links, in halves: 2 (axis) + 4 diagonals of mean values
        T dj[3] = {T(0), T(0), T(0)};
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            const int bx = d / 2;
            if (bx == ax) continue;
            // Diagonal link along sg e_ax + (+-) e_bx: it also crosses face d when out[d].
            const T sb = (d & 1) ? T(-1) : T(1);
            const T m = out[d] ? w[f] + w[d] : T(2) * w[f];
            v = v + m;
            dj[bx] = fma3(sb, m, dj[bx]);
        }
        const T half = T(0.5) * v1;
        const T t = fma3(T(-6), fma3(-sg, q[ax], o.g), half * v);
        s.phi = s.phi + t;
        j[ax] = fma3(sg, t, j[ax]);
#pragma unroll
        for (int bx = 0; bx < 3; ++bx)
            if (bx != ax) j[bx] = j[bx] + fma3(half, dj[bx], T(2) * q[bx]);
    }
    // Links through an edge of the box belong to both faces' sums: taken off once.
#pragma unroll
    for (int f = 0; f < 6; ++f)
#pragma unroll
        for (int d = f + 1; d < 6; ++d) {
            if (d / 2 == f / 2 || !out[f] || !out[d]) continue;
            const T sf = (f & 1) ? T(-1) : T(1), sd = (d & 1) ? T(-1) : T(1);
            const T t = fma3(T(0.5) * v1, w[f] + w[d], fma3(sf, q[f / 2], fma3(sd, q[d / 2], -o.g)));
            s.phi = s.phi - t;
            j[f / 2] = fma3(-sf, t, j[f / 2]);
            j[d / 2] = fma3(-sd, t, j[d / 2]);
        }
    s.jx = j[0];
    s.jy = j[1];
    s.jz = j[2];
}

template <typename T>
struct Mom3State {
    T phi, qx, qy, qz, g;
};

// The collision on the pulled moments (collide3 with k0 = 1 and Q = 0).
template <typename T, bool SRC, bool KPHI>
__host__ __device__ __forceinline__ Mom3State<T> mom3_collide(const Sweep3<T>& a, const Mom3Sum<T>& f, T phi_prev, T s)
{
    constexpr T half = T(0.5);
    const T phi = f.phi, j[3] = {f.jx, f.jy, f.jz};
    T v[3], h[3];  // j + dB and j - B + dB/2
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const T hb = half * a.b[c];
        const T B = phi * fma3(hb, phi, a.a[c]);
        const T dB = fma3(-phi_prev, fma3(hb, phi_prev, a.a[c]), B);
        h[c] = fma3(half, dB, j[c] - B);
        v[c] = j[c] + dB;
    }
    Mom3State<T> o;
    if constexpr (KPHI) {
        // K1 h = adj(M) h / det M with M = 3 A + I/2 (Eq. (30)).
        const T g = fma3(a.beta, phi * phi, T(1));
        const T m11 = fma3(a.m3[0], g, half), m12 = a.m3[1] * g, m13 = a.m3[2] * g;
        const T m22 = fma3(a.m3[3], g, half), m23 = a.m3[4] * g, m33 = fma3(a.m3[5], g, half);
        const T c11 = fma3(m22, m33, -(m23 * m23)), c12 = fma3(m13, m23, -(m12 * m33));
        const T c13 = fma3(m12, m23, -(m13 * m22)), c22 = fma3(m11, m33, -(m13 * m13));
        const T c23 = fma3(m12, m13, -(m11 * m23)), c33 = fma3(m11, m22, -(m12 * m12));
        const T det = fma3(m11, c11, fma3(m12, c12, m13 * c13));
        const T r = btrtk::quotient(det);
        o.qx = fma3(-r, fma3(c11, h[0], fma3(c12, h[1], c13 * h[2])), v[0]);
        o.qy = fma3(-r, fma3(c12, h[0], fma3(c22, h[1], c23 * h[2])), v[1]);
        o.qz = fma3(-r, fma3(c13, h[0], fma3(c23, h[1], c33 * h[2])), v[2]);
    } else {
        o.qx = v[0] - fma3(a.K1[0], h[0], fma3(a.K1[1], h[1], a.K1[2] * h[2]));
        o.qy = v[1] - fma3(a.K1[1], h[0], fma3(a.K1[3], h[1], a.K1[4] * h[2]));
        o.qz = v[2] - fma3(a.K1[2], h[0], fma3(a.K1[4], h[1], a.K1[5] * h[2]));
    }
    o.phi = phi;
    o.g = SRC ? phi + s : phi;
    return o;
}

// Moments of the pull at node (x, y, z) from the planes: the reads' form of what the sweeps do.
template <typename T>
__host__ __device__ __forceinline__ Mom3Sum<T> mom3_pull(const Sweep3<T>& a, int x, int y, int z)
{
    const T* qx = a.fin + kM3Qx * a.plane;
    const T* qy = a.fin + kM3Qy * a.plane;
    const T* qz = a.fin + kM3Qz * a.plane;
    const T* g = a.src ? a.fin + kM3G * a.plane : a.phi_prev;
    auto at = [&](int i, int j, int k) {  // node values at wrapped coordinates; zero beyond a face
        if (i < 0 || i >= a.nx) { if (!a.per[0]) return Mom3Node<T>{}; i = i < 0 ? i + a.nx : i - a.nx; }
        if (j < 0 || j >= a.ny) { if (!a.per[1]) return Mom3Node<T>{}; j = j < 0 ? j + a.ny : j - a.ny; }
        if (k < 0 || k >= a.nz) { if (!a.per[2]) return Mom3Node<T>{}; k = k < 0 ? k + a.nz : k - a.nz; }
        const int n = k * a.slab + j * a.pitch + i;
        return mom3_node(g[n], qx[n], qy[n], qz[n]);
    };
    auto row = [&](int j, int k) {
        const Mom3Node<T> l = at(x - 1, j, k), c = at(x, j, k), r = at(x + 1, j, k);
        return mom3_row(c, l.g + l.b, l.c, l.d, r.g - r.b, r.c, r.d);
    };
    auto plane = [&](int k) {
        const Mom3Row<T> lo = row(y - 1, k), hi = row(y + 1, k);
        return mom3_plane(row(y, k), lo.up, hi.dn);
    };
    const Mom3Plane3<T> lo = plane(z - 1), mid = plane(z), hi = plane(z + 1);
    Mom3Sum<T> s{(mid.M + lo.U) + hi.D, (mid.Mx + lo.Ux) + hi.Dx, (mid.My + lo.Uy) + hi.Dy, lo.U - hi.D};
    const bool out[6] = {!a.per[0] && x == 0, !a.per[0] && x == a.nx - 1, !a.per[1] && y == 0,
                         !a.per[1] && y == a.ny - 1, !a.per[2] && z == 0, !a.per[2] && z == a.nz - 1};
    if (out[0] || out[1] || out[2] || out[3] || out[4] || out[5]) mom3_walls(at(x, y, z), out, a.wall, s);
    return s;
}

}  // namespace btrt3k
