// Device evaluation of the kernel entries of the P1 collocation.
//
// Volume entry (Section "FEM discretization", with the Corollary's mirror term):
//   G^{ij} = exp(-tau(x_i,x_j)) g(x_i, j) + R exp(-tau_bar(x_i,x_j)) g(x_bar_i, j)
//   g(x, j) = |e|/(4 pi) sum_{e ni j} sum_q w_q kappa(y_q) lambda_j(y_q) / |x - y_q|^2
// Surface entry (eq. SE1 and its mirror, Proposition 2):
//   S^{il}  = exp(-tau(x_i,x_l)) s(x_i, l) + R exp(-tau_bar(x_i,x_l)) s(x_bar_i, l)
//   s(x, l) = |t|/(4 pi) sum_{t ni l} sum_q w_q lambda_l(y_q) |(x - y_q).n| / |x - y_q|^3
// with the coplanar limit theta_F/(4 pi) on the diagonal.  tau is the exact
// line integral of the P1 kappa, tau_bar the same along the path reflected
// at the wall.  One optical depth per vertex pair; near rule (degree 5)
// when the grid Chebyshev distance is <= 2, degree 2 otherwise.
//
// FP64: tau from the kinks of kappa along the ray (march.h), or from the march
// through its tetrahedra (march_tets.h) when kink_quantum says so, g from a table by
// offset; FP32: tau from that march in FP32, g point by point.
#pragma once

#include <type_traits>
#include <utility>

#include "kernels.h"

namespace rte {

// 1/x for positive, normal x (distances, crossing counts): the hardware
// reciprocal refined by two Newton steps (FP64: the seed's relative error e
// becomes e^4, below one ulp), or the hardware reciprocal alone (FP32, one
// ulp): cheaper than the IEEE division sequence.
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }

}  // namespace rte

#include "march.h"
#include "march_tets.h"

namespace rte {

// K: optical depths from the kinks of kappa (FP64), else by the march
template <typename T, bool K>
struct EntryCtx {
    using Tab = DepthTab<T, K>;
    GridDev g;
    const T *__restrict__ kappa;   // [N] P1 vertex values of one band
    const Tab *__restrict__ tab;   // kinks of kappa, or the vertices of its tetrahedra
    double q;                      // the kinks' quantum
    StencilDev<T> st;
    const T *__restrict__ near;    // quadrature tables of the mesh: near [125][8][8], then far [24][4][8]
    StarTab star;                  // FP64: the same by offset (null: not built)
};
template <typename T, bool K>
__device__ __forceinline__ auto depth_src(const EntryCtx<T, K> &c) {
    if constexpr (K) return KinkTab{c.tab, c.kappa, c.q};
    else return KappaSrc<T>{c.tab};
}

// ---------------------------------------------------------------- compile-time Kuhn star
struct TetInfo { int slot[4]; int bits; };
struct TriInfo { int ob, oc; };

struct KuhnStar {
    TetInfo tet[kTets];
    TriInfo tri[kTris];
};

// Same enumeration as the host stencil tables: cell corner bits o (cell = j - o),
// then the axis orders in lexicographic order; keep the tetrahedra that contain j.
constexpr KuhnStar make_star() {
    KuhnStar S{};
    const int perm[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    int n = 0;
    for (int bits = 0; bits < 8; ++bits) {
        int o[3] = {bits & 1, (bits >> 1) & 1, (bits >> 2) & 1};
        for (int p = 0; p < 6; ++p) {
            int w[4][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {1, 1, 1}};
            w[1][perm[p][0]] = 1;
            w[2][perm[p][0]] = 1;
            w[2][perm[p][1]] = 1;
            bool has = false;
            for (int k = 0; k < 4; ++k)
                if (w[k][0] == o[0] && w[k][1] == o[1] && w[k][2] == o[2]) has = true;
            if (!has) continue;
            for (int k = 0; k < 4; ++k)
                S.tet[n].slot[k] = (w[k][0] - o[0] + 1) * 9 + (w[k][1] - o[1] + 1) * 3 + (w[k][2] - o[2] + 1);
            S.tet[n].bits = bits;
            ++n;
        }
    }
    const int corners[2][3][2] = {{{0, 0}, {1, 0}, {1, 1}}, {{0, 0}, {0, 1}, {1, 1}}};
    int m = 0;
    for (int ob = 0; ob < 2; ++ob)
        for (int oc = 0; oc < 2; ++oc)
            for (int t = 0; t < 2; ++t) {
                bool has = false;
                for (int k = 0; k < 3; ++k)
                    if (corners[t][k][0] == ob && corners[t][k][1] == oc) has = true;
                if (!has) continue;
                S.tri[m].ob = ob;
                S.tri[m].oc = oc;
                ++m;
            }
    return S;
}

constexpr KuhnStar kStar = make_star();
__device__ const KuhnStar kStarDev = make_star();   // for an index that is not a compile-time constant

// Corner e (bits x, y, z) of the cell j - o (o the corner bits of j in it) as a
// slot of the 3x3x3 block around j, and back.
__host__ __device__ constexpr int slot_of(int e, int o) {
    return ((e & 1) - (o & 1) + 1) * 9 + (((e >> 1) & 1) - ((o >> 1) & 1) + 1) * 3 + (((e >> 2) & 1) - ((o >> 2) & 1) + 1);
}
__host__ __device__ constexpr int corner_of(int slot, int o) {
    return (slot / 9 - 1 + (o & 1)) | ((slot / 3 % 3 - 1 + ((o >> 1) & 1)) << 1) | ((slot % 3 - 1 + ((o >> 2) & 1)) << 2);
}
// Vertex v < 15 of the star: j + bits v of {0,1}^3 (v < 8), then j - bits v - 7.
__host__ __device__ constexpr int star_slot(int v) { return v < 8 ? slot_of(v, 0) : slot_of(0, v - 7); }
// does any tetrahedron around j in the cell j - o have the cell's corner e
constexpr bool corner_used(int e, int o) {
    for (int t = 0; t < kTets; ++t)
        for (int k = 0; k < 4; ++k)
            if (kStar.tet[t].bits == o && corner_of(kStar.tet[t].slot[k], o) == e) return true;
    return false;
}

// ---------------------------------------------------------------- walls
// Wall w's axis, side and coefficient, picked by selects over the constant
// indices: an index into the grid's arrays that is not a compile-time constant
// would copy the whole kernel argument to scratch memory.
struct WallInfo {
    int axis, side;
    double R;
};
__device__ __forceinline__ WallInfo wall_info(const GridDev &g, int w) {
    WallInfo r{g.wall_axis[0], g.wall_side[0], g.R[0]};
#pragma unroll
    for (int k = 1; k < 6; ++k)
        if (w == k) r = WallInfo{g.wall_axis[k], g.wall_side[k], g.R[k]};
    return r;
}

// grid index of the wall's plane along its axis
__device__ __forceinline__ int wall_plane(const GridDev &g, const WallInfo &wi) {
    int C = 0;
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b == wi.axis && wi.side) C = g.n[b] - 1;
    return C;
}

// optical depth of the path from x (grid index P) to wall w and on to y (Q)
template <typename Src>
__device__ __forceinline__ auto tau_mirror(const GridDev &g, int w, const Src &kt, const int P[3], const int Q[3]) {
    const WallInfo wi = wall_info(g, w);
    return tau_reflected(g, kt, wi.axis, wall_plane(g, wi), P, Q);
}

// grid index of the mirror image of vertex xi in wall w
__device__ __forceinline__ void mirror_index(const GridDev &g, int w, const int xi[3], int mi[3]) {
    const WallInfo wi = wall_info(g, w);
    const int a = wi.axis;
    const int Ci = wi.side ? g.n[a] - 1 : 0;
    mi[0] = xi[0];
    mi[1] = xi[1];
    mi[2] = xi[2];
    mi[a] = 2 * Ci - xi[a];
}

// ---------------------------------------------------------------- the hole (non-convex domain)
// A path is blocked when it runs a positive length through the removed box of
// cells (kappa = +infinity there, Remark rem1) or over a part of a box face
// that the box covers.  Both ends of a segment are grid vertices (integer
// coordinates; a mirror image of one too), so the test is exact: the slab
// method with the parameters of the box planes kept as fractions n / d, d > 0,
// compared by cross multiplication.  An axis open on one side (bit 2a: below,
// 2a+1: above) has no plane there.
__device__ __forceinline__ bool frac_lt(int64_t an, int64_t ad, int64_t bn, int64_t bd) { return an * bd < bn * ad; }

__device__ __forceinline__ bool seg_meets_box(const int P[3], const int Q[3], const int lo[3], const int hi[3],
                                              unsigned open) {
    int64_t t0n = 0, t0d = 1, t1n = 1, t1d = 1;   // the segment's own [0, 1]
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int D = Q[a] - P[a];
        const bool ol = (open >> (2 * a)) & 1u, oh = (open >> (2 * a + 1)) & 1u;
        if (D == 0) {
            if (!((ol || P[a] > lo[a]) && (oh || P[a] < hi[a]))) return false;
            continue;
        }
        const int64_t ad = D > 0 ? D : -D;
        if (D > 0 ? !ol : !oh) {   // enters through the plane below (D > 0) or above
            const int64_t en = D > 0 ? lo[a] - P[a] : P[a] - hi[a];
            if (frac_lt(t0n, t0d, en, ad)) { t0n = en; t0d = ad; }
        }
        if (D > 0 ? !oh : !ol) {   // leaves through the plane above (D > 0) or below
            const int64_t ex = D > 0 ? hi[a] - P[a] : P[a] - lo[a];
            if (frac_lt(ex, ad, t1n, t1d)) { t1n = ex; t1d = ad; }
        }
    }
    return frac_lt(t0n, t0d, t1n, t1d);
}

// the straight path between grid vertices P and Q crosses the hole
__device__ __forceinline__ bool hole_blocks(const GridDev &g, const int P[3], const int Q[3]) {
    return seg_meets_box(P, Q, g.hole_lo, g.hole_hi, g.hole_open);
}

// the path from P reflected at wall w to Q crosses the hole.  Unfolded, it is
// the straight segment from P's mirror image to Q; its part beyond the wall
// is the mirror image of the first leg, so the blocking region there is the
// mirror image of the hole.  A hole that reaches the wall merges with its
// image into one box twice as long; otherwise the two boxes are tested apart.
__device__ __forceinline__ bool hole_blocks_mirror(const GridDev &g, int w, const int P[3], const int Q[3]) {
    const WallInfo wi = wall_info(g, w);
    const int a = wi.axis;
    // the wall axis' values by selects (a is not a compile-time constant)
    int Pb[3], lo[3], hi[3], C = 0, la = 0, ha = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = g.hole_lo[k];
        hi[k] = g.hole_hi[k];
        Pb[k] = P[k];
        if (k == a) {
            C = wi.side ? g.n[k] - 1 : 0;
            Pb[k] = 2 * C - P[k];
            la = g.hole_lo[k];
            ha = g.hole_hi[k];
        }
    }
    const unsigned ol = (g.hole_open >> (2 * a)) & 1u, oh = (g.hole_open >> (2 * a + 1)) & 1u;
    const unsigned others = g.hole_open & ~(3u << (2 * a));
    int blo[3], bhi[3];
    if (wi.side == 0 ? ol : oh) {
        // merged: (2C - hi, hi) at the low wall, (lo, 2C - lo) at the high one,
        // unbounded at both ends when the hole also reaches the far face
        const unsigned far = wi.side == 0 ? oh : ol;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            blo[k] = k == a ? (wi.side == 0 ? 2 * C - ha : la) : lo[k];
            bhi[k] = k == a ? (wi.side == 0 ? ha : 2 * C - la) : hi[k];
        }
        return seg_meets_box(Pb, Q, blo, bhi, others | (far ? 3u << (2 * a) : 0u));
    }
    if (seg_meets_box(Pb, Q, lo, hi, g.hole_open)) return true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        blo[k] = k == a ? 2 * C - ha : lo[k];
        bhi[k] = k == a ? 2 * C - la : hi[k];
    }
    return seg_meets_box(Pb, Q, blo, bhi, others | (oh << (2 * a)) | (ol << (2 * a + 1)));
}

// bit o of the 8 cells around vertex v (cell v - o) is set for the hole's cells
__device__ __forceinline__ int hole_cells(const GridDev &g, const int v[3]) {
    int m = 0;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        bool in = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int c = v[a] - ((o >> a) & 1);
            in = in && c >= g.hole_lo[a] && c < g.hole_hi[a];
        }
        m |= in ? (1 << o) : 0;
    }
    return m;
}

// a vertex of the closed domain: one of its cells inside the grid is no hole cell
__device__ __forceinline__ bool vertex_active(const GridDev &g, const int v[3]) {
    if (!g.has_hole) return true;
    int grid = 0;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int c = v[a] - ((o >> a) & 1);
            ok = ok && c >= 0 && c <= g.n[a] - 2;
        }
        grid |= ok ? (1 << o) : 0;
    }
    return (grid & ~hole_cells(g, v)) != 0;
}

__device__ __forceinline__ int cheb3(const int a[3], const int b[3]) {
    return max(max(abs(a[0] - b[0]), abs(a[1] - b[1])), abs(a[2] - b[2]));
}

// grid index of vertex v (fewer than 2^28 vertices: 32-bit unsigned division)
__device__ __forceinline__ void vtx_index(const GridDev &g, int64_t v, int idx[3]) {
    const unsigned u = (unsigned)v, s0 = (unsigned)g.stride[0], s1 = (unsigned)g.stride[1];
    const unsigned i0 = u / s0, r = u - i0 * s0, i1 = r / s1;
    idx[0] = (int)i0;
    idx[1] = (int)i1;
    idx[2] = (int)(r - i1 * s1);
}

// ---------------------------------------------------------------- volume quadrature
// bit o: the cell j - o around vertex j lies in the grid
__device__ __forceinline__ int cells_in_grid(const GridDev &g, const int jj[3]) {
    int m = 0;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) ok = ok && (((o >> a) & 1) ? jj[a] >= 1 : jj[a] <= g.n[a] - 2);
        m |= ok ? (1 << o) : 0;
    }
    return m;
}

// kappa at the slot of the 3x3x3 block around vertex v (inside the grid)
template <typename T, bool K>
__device__ __forceinline__ T kappa_slot(const EntryCtx<T, K> &c, int64_t v, int slot) {
    return c.kappa[v + (slot / 9 - 1) * c.g.stride[0] + (slot / 3 % 3 - 1) * c.g.stride[1] + (slot % 3 - 1)];
}

// g(x, j) point by point, for meshes without a star table (d = x - x_j, v the
// flat index of j): near offsets from the near table, far ones by the degree-2
// rule, |x - y|^2 = |h d|^2 + A.d + C per point and the 4 points of a
// tetrahedron over one common denominator.
template <bool K>
__device__ __forceinline__ double vol_points(const EntryCtx<double, K> &c, int64_t v, int cellmask, const int d0,
                                             const int d1, const int d2) {
    const GridDev &g = c.g;
    double acc = 0.0;
    if (max(max(abs(d0), abs(d1)), abs(d2)) <= kNearCheb) {
        const double *row = c.near + ((d0 + 2) * 25 + (d1 + 2) * 5 + (d2 + 2)) * 64;
#pragma nounroll
        for (int o = 0; o < 8; ++o) {
            if (!((cellmask >> o) & 1)) continue;
#pragma nounroll
            for (int e = 0; e < 8; ++e) acc += row[o * 8 + e] * kappa_slot(c, v, slot_of(e, o));
        }
        return acc * g.vol_scale;
    }
    const double x = (double)d0, y = (double)d1, z = (double)d2;
    const double D2 = g.h[0] * g.h[0] * x * x + g.h[1] * g.h[1] * y * y + g.h[2] * g.h[2] * z * z;
#pragma nounroll
    for (int t = 0; t < kTets; ++t) {
        const TetInfo &ti = kStarDev.tet[t];
        if (!((cellmask >> ti.bits) & 1)) continue;
        const double k0 = kappa_slot(c, v, ti.slot[0]), k1 = kappa_slot(c, v, ti.slot[1]);
        const double k2 = kappa_slot(c, v, ti.slot[2]), k3 = kappa_slot(c, v, ti.slot[3]);
        const double *e = c.near + kNearSize + t * 32;
        double a[4], r[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            r[q] = D2 + e[8 * q + 3] + e[8 * q + 0] * x + e[8 * q + 1] * y + e[8 * q + 2] * z;
            a[q] = e[8 * q + 4] * k0 + e[8 * q + 5] * k1 + e[8 * q + 6] * k2 + e[8 * q + 7] * k3;
        }
        const double n01 = a[0] * r[1] + a[1] * r[0], d01 = r[0] * r[1];
        const double n23 = a[2] * r[3] + a[3] * r[2], d23 = r[2] * r[3];
        acc += (n01 * d23 + n23 * d01) * recip(d01 * d23);
    }
    return acc * g.vol_scale;
}

template <int o, bool K, int... es>
__device__ __forceinline__ void cell_corners(std::integer_sequence<int, es...>, const EntryCtx<double, K> &c, int64_t v,
                                             const double *__restrict__ row, double &acc) {
    ((corner_used(es, o) ? (void)(acc = fma(row[o * 8 + es], kappa_slot(c, v, slot_of(es, o)), acc)) : (void)0), ...);
}
template <bool K, int... os>
__device__ __forceinline__ double vol_cells(std::integer_sequence<int, os...>, const EntryCtx<double, K> &c, int64_t v,
                                            int cellmask, const double *__restrict__ row) {
    double acc = 0.0;
    ((((cellmask >> os) & 1) ? cell_corners<os>(std::make_integer_sequence<int, 8>{}, c, v, row, acc) : (void)0), ...);
    return acc;
}

// The star of a source vertex: its flat index, its cells, and for a whole star
// kappa at its 15 vertices.
struct Star {
    int64_t v;
    int cellmask;
    double k[15];
};

// g(x_j + d, j): a row of the star table times kappa, 15 products and 128
// contiguous bytes per entry, where the points of the rule cost about 1100
// instructions (24 tetrahedra); a source that misses cells (on
// the boundary, at the hole) takes its cells' corner weights.  41^3: dense
// fill 12.8 -> 7.7 ms, ACA entry launches 73.5 -> 70.4 (bound by the march).
template <int, bool K>
__device__ __forceinline__ double vol_quad(const EntryCtx<double, K> &c, const Star &s, const int d[3]) {
    if (!c.star.w) return vol_points(c, s.v, s.cellmask, d[0], d[1], d[2]);
    const int64_t row = (int64_t)(d[0] - c.star.lo[0]) * c.star.st0 + (d[1] - c.star.lo[1]) * c.star.st1 +
                        (d[2] - c.star.lo[2]);
    if (s.cellmask != 255)
        return vol_cells(std::make_integer_sequence<int, 8>{}, c, s.v, s.cellmask,
                         c.star.cell + row * 64);
    const double *w = static_cast<const double *>(__builtin_assume_aligned(c.star.w + row * kStarWeights, 64));
    double acc = 0.0;   // explicit fma: the same sum wherever it is inlined
#pragma unroll
    for (int v = 0; v < 15; ++v) acc = fma(w[v], s.k[v], acc);
    return acc;
}

template <bool K>
__device__ __forceinline__ Star load_star(const EntryCtx<double, K> &c, const int jj[3], int cellmask) {
    Star s;
    s.v = (int64_t)jj[0] * c.g.stride[0] + (int64_t)jj[1] * c.g.stride[1] + jj[2];
    s.cellmask = cellmask;
    if (cellmask == 255) {
#pragma unroll
        for (int v = 0; v < 15; ++v) s.k[v] = kappa_slot(c, s.v, star_slot(v));
    }
    return s;
}

// FP32 entries, point by point (march_tets.h says why).
// Near field (grid offset d = x - x_j with |d_a| <= 2): the degree-5 rule's
// sums, tabulated per mesh by cell and corner, so g is 64 products with the
// star's kappa values (cells outside the grid skipped).
__device__ __forceinline__ float vol_near(const float *__restrict__ tab, const float kn[27], int cellmask, const int d[3]) {
    const float *row = tab + ((d[0] + 2) * 25 + (d[1] + 2) * 5 + (d[2] + 2)) * 64;
    float acc = 0.0f;
#pragma unroll
    for (int bits = 0; bits < 8; ++bits) {
        if (!((cellmask >> bits) & 1)) continue;
        const int o0 = bits & 1, o1 = (bits >> 1) & 1, o2 = (bits >> 2) & 1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int slot = ((e & 1) - o0 + 1) * 9 + (((e >> 1) & 1) - o1 + 1) * 3 + (((e >> 2) & 1) - o2 + 1);
            acc += row[bits * 8 + e] * kn[slot];
        }
    }
    return acc;
}

// Far field, one tetrahedron of the star: its 4 points' terms a_q / r_q added
// over a common denominator, so one reciprocal serves the 4 points.
template <int t>
__device__ __forceinline__ void vol_far_tet(const float *__restrict__ ft, const float kn[27], int cellmask, float D2,
                                            const float dg[3], float &acc) {
    constexpr TetInfo ti = kStar.tet[t];
    if (!((cellmask >> ti.bits) & 1)) return;
    const float k0 = kn[ti.slot[0]], k1 = kn[ti.slot[1]], k2 = kn[ti.slot[2]], k3 = kn[ti.slot[3]];
    const float *e = ft + t * 32;
    float a[4], r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        r[q] = D2 + e[8 * q + 3] + e[8 * q + 0] * dg[0] + e[8 * q + 1] * dg[1] + e[8 * q + 2] * dg[2];
        a[q] = e[8 * q + 4] * k0 + e[8 * q + 5] * k1 + e[8 * q + 6] * k2 + e[8 * q + 7] * k3;
    }
    const float n01 = a[0] * r[1] + a[1] * r[0], d01 = r[0] * r[1];
    const float n23 = a[2] * r[3] + a[3] * r[2], d23 = r[2] * r[3];
    acc += (n01 * d23 + n23 * d01) * recip(d01 * d23);
}

template <int... ts>
__device__ __forceinline__ float vol_far_all(std::integer_sequence<int, ts...>, const float *__restrict__ ft, const float kn[27],
                                         int cellmask, float D2, const float dg[3]) {
    float acc = 0.0f;
    (vol_far_tet<ts>(ft, kn, cellmask, D2, dg, acc), ...);
    return acc;
}

// The star of an FP32 source: its cells and kappa on the 3x3x3 block around it.
struct Star32 {
    int cellmask;
    float k[27];
};
__device__ __forceinline__ Star32 load_star(const EntryCtx<float, false> &c, const int jj[3], int cellmask) {
    const GridDev &g = c.g;
    Star32 r;
    r.cellmask = cellmask;
#pragma unroll
    for (int s = 0; s < 27; ++s) {
        const int dx = s / 9 - 1, dy = (s / 3) % 3 - 1, dz = s % 3 - 1;
        const int x = min(max(jj[0] + dx, 0), g.n[0] - 1);
        const int y = min(max(jj[1] + dy, 0), g.n[1] - 1);
        const int z = min(max(jj[2] + dz, 0), g.n[2] - 1);
        r.k[s] = c.kappa[x * g.stride[0] + y * g.stride[1] + z];
    }
    return r;
}
// g(x_j + d, j) without the 1/(4 pi)|e| factor.  FIRST: the axis whose square is
// rounded by itself in |h d|^2.
template <int FIRST, bool K>
__device__ __forceinline__ float vol_quad(const EntryCtx<float, K> &c, const Star32 &s, const int d[3]) {
    if (max(max(abs(d[0]), abs(d[1])), abs(d[2])) <= kNearCheb) return vol_near(c.near, s.k, s.cellmask, d);
    const GridDev &g = c.g;
    const float h2[3] = {(float)(g.h[0] * g.h[0]), (float)(g.h[1] * g.h[1]), (float)(g.h[2] * g.h[2])};
    const float dg[3] = {(float)d[0], (float)d[1], (float)d[2]};
    constexpr int A = FIRST, B = 1 - FIRST;   // rounded the same way in every kernel
    const float D2 = fma(h2[2] * dg[2], dg[2], fma(h2[B] * dg[B], dg[B], rounded_product(h2[A] * dg[A], dg[A])));
    return vol_far_all(std::make_integer_sequence<int, kTets>{}, c.near + kNearSize, s.k, s.cellmask, D2, dg);
}

// Wall modes the entry code is compiled for: no wall, exactly one wall (the
// common reflective case, kept as straight-line code), or the general mode:
// any number of walls read from the grid (a loop; its per-wall attenuations go
// through a small array in scratch memory) and the hole of a non-convex domain.
constexpr int kNoWall = 0, kOneWall = 1, kAnyWalls = 6;
inline int wall_mode(const GridDev &g) {
    return (g.has_hole || g.n_walls > 1) ? kAnyWalls : (g.n_walls == 0 ? kNoWall : kOneWall);
}

// The first term of an entry.  FP64: rounded, so that group_entry's sum is that of
// a single lane.  FP32: free to join what follows (the BF16 lo part of a dense entry
// is taken from the unrounded product).
__device__ __forceinline__ double first_term(double att, double g) { return rounded_product(att, g); }
__device__ __forceinline__ float first_term(float att, float g) { return att * g; }

// sum over the direct path and the walls of attenuation times the quadrature
// of the source star of ss seen from target tt (or from its mirror image in
// each wall); att_w[w] = R_w exp(-tau_w)
template <typename T, bool K, int NW>
__device__ __forceinline__ T vol_sum(const EntryCtx<T, K> &c, T att, const T att_w[6], const int tt[3],
                                     const int ss[3]) {
    const GridDev &g = c.g;
    int cellmask = cells_in_grid(g, ss);
    if constexpr (NW == kAnyWalls)
        if (g.has_hole) cellmask &= ~hole_cells(g, ss);   // the hole's cells are in no star
    const auto star = load_star(c, ss, cellmask);
    const int dg[3] = {tt[0] - ss[0], tt[1] - ss[1], tt[2] - ss[2]};
    T G = first_term(att, vol_quad<NW == kAnyWalls ? 0 : 1, K>(c, star, dg));
    if constexpr (NW != kNoWall) {
        const int nw = NW == kOneWall ? 1 : g.n_walls;
        for (int w = 0; w < nw; ++w) {
            int mt[3];
            mirror_index(g, w, tt, mt);
            const int dgm[3] = {mt[0] - ss[0], mt[1] - ss[1], mt[2] - ss[2]};
            G += att_w[w] * vol_quad<1, K>(c, star, dgm);
        }
    }
    if constexpr (sizeof(T) == 4) return G * (T)g.vol_scale;
    else return G;   // the scale is in the table
}

// The attenuations of a pair: exp(-tau) along the direct path, and R_w
// exp(-tau_w) per wall; a path that the hole blocks has tau = +infinity (no
// march).  Pi, Qi: the vertices' grid indices.
template <typename T, int NW, typename Src>
__device__ __forceinline__ T attenuations(const GridDev &g, const Src &kt, const int Pi[3], const int Qi[3],
                                          T att_w[6]) {
    if constexpr (NW == kAnyWalls) {
        const bool hole = g.has_hole;
        const T att = (hole && hole_blocks(g, Pi, Qi)) ? (T)0 : exp(-tau_direct(g, kt, Pi, Qi));
        for (int w = 0; w < g.n_walls; ++w)
            att_w[w] = (hole && hole_blocks_mirror(g, w, Pi, Qi))
                           ? (T)0
                           : (T)wall_info(g, w).R * exp(-tau_mirror(g, w, kt, Pi, Qi));
        return att;
    } else {
        const T att = exp(-tau_direct(g, kt, Pi, Qi));
        if constexpr (NW == kOneWall) att_w[0] = (T)g.R[0] * exp(-tau_mirror(g, 0, kt, Pi, Qi));
        return att;
    }
}

// The same for a group of P lanes of one wavefront (P a power of two, lane
// number `sub`) that share the pair.  Kinks: the families of every leg of every
// path are dealt to the lanes and added in the order of kink_sum; march: the legs
// are.  The attenuations are those of a single lane bit for bit.  buf: LDS of the
// group, group_tasks values.
template <typename T, bool K>
using GroupTask = std::conditional_t<K, Dd, T>;
template <bool K>
__host__ __device__ constexpr int group_tasks(int n_walls) {
    return (K ? 6 : 1) * (1 + 2 * n_walls);
}
__device__ __forceinline__ void group_sync() {   // orders the LDS accesses of a wavefront
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
template <int NW>
__device__ __forceinline__ double group_attenuations(const GridDev &g, const KinkTab &kt, const int Pi[3],
                                                     const int Qi[3], double att_w[6], int P, int sub, Dd *buf) {
    const int nw = NW == kAnyWalls ? g.n_walls : NW;
    for (int t = sub; t < 6 * (1 + 2 * nw); t += P) {
        const int leg = t / 6, f = t - 6 * leg;
        int V[3] = {Pi[0], Pi[1], Pi[2]}, D[3] = {Qi[0] - Pi[0], Qi[1] - Pi[1], Qi[2] - Pi[2]}, p = 1, M = 1;
        if (NW != kNoWall && leg > 0) {
            const WallInfo wi = wall_info(g, (leg - 1) >> 1);
            const Legs l = reflect_legs(wi.axis, wall_plane(g, wi), Pi, Qi);
            const bool from_q = (leg & 1) == 0;
            M = l.p + l.q;
            p = from_q ? l.q : l.p;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                V[b] = from_q ? Qi[b] : Pi[b];
                D[b] = from_q ? l.D2[b] : l.D1[b];
            }
            if (M == 0) p = M = 1;   // both on the wall: the direct depth is taken below
        }
        buf[t] = kink_one(g, kt.tab, V, D, p, M, f);
    }
    group_sync();
    const double direct = direct_depth(g, kt, Pi, Qi, add_families(buf));
    const bool hole = NW == kAnyWalls && g.has_hole;
    const double att = hole && hole_blocks(g, Pi, Qi) ? 0.0 : exp(-direct);
    if constexpr (NW != kNoWall) {
        for (int w = 0; w < nw; ++w) {
            const WallInfo wi = wall_info(g, w);
            const int C = wall_plane(g, wi);
            const Legs l = reflect_legs(wi.axis, C, Pi, Qi);
            const Dd *b = buf + 6 + 12 * w;
            const double tau = l.p + l.q == 0
                                   ? direct
                                   : reflected_depth(g, kt, wi.axis, C, Pi, Qi, l, dd_add(add_families(b), add_families(b + 6)));
            att_w[w] = hole && hole_blocks_mirror(g, w, Pi, Qi) ? 0.0 : wi.R * exp(-tau);
        }
    }
    return att;
}
template <int NW, typename T>
__device__ __forceinline__ T group_attenuations(const GridDev &g, const KappaSrc<T> &kt, const int Pi[3],
                                                const int Qi[3], T att_w[6], int P, int sub, T *buf) {
    const int nw = NW == kAnyWalls ? g.n_walls : NW;
    for (int t = sub; t < 1 + 2 * nw; t += P) {
        T A[3] = {(T)Pi[0], (T)Pi[1], (T)Pi[2]}, B[3] = {(T)Qi[0], (T)Qi[1], (T)Qi[2]};
        if (NW != kNoWall && t > 0) {   // P to the wall, the wall to Q
            const WallInfo wi = wall_info(g, (t - 1) >> 1);
            T X[3];
            wall_point<T>(wi.axis, (T)wall_plane(g, wi), A, B, X);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                A[b] = t & 1 ? A[b] : X[b];
                B[b] = t & 1 ? X[b] : B[b];
            }
        }
        buf[t] = tau_segment<T>(g, kt, A, B);
    }
    group_sync();
    const bool hole = NW == kAnyWalls && g.has_hole;
    const T att = hole && hole_blocks(g, Pi, Qi) ? (T)0 : exp(-buf[0]);
    if constexpr (NW != kNoWall)
        for (int w = 0; w < nw; ++w)
            att_w[w] = hole && hole_blocks_mirror(g, w, Pi, Qi)
                           ? (T)0
                           : (T)wall_info(g, w).R * exp(-(buf[1 + 2 * w] + buf[2 + 2 * w]));
    return att;
}

// G(i, j).  Every wall adds its own mirror-image term (one reflection per
// ray).  The optical depths come first: the star of j is loaded after the
// marches, so its values do not stay live through them.  FROM_J: the kinks are
// walked from j (the depth is the same to the bit), for launches whose lanes share
// the source: the lanes then meet the planes in step (KinkTab).
template <typename T, bool K, int NW = kAnyWalls, bool FROM_J = false>
__device__ T volume_entry(const EntryCtx<T, K> &c, int64_t i, int64_t j) {
    const GridDev &g = c.g;
    int ii[3], jj[3];
    vtx_index(g, i, ii);
    vtx_index(g, j, jj);
    if constexpr (NW == kAnyWalls)
        if (!vertex_active(g, ii)) return (T)0;   // a removed vertex (its column: an empty star)
    T att_w[6];
    constexpr bool from_j = FROM_J && K;
    const T att = attenuations<T, NW>(g, depth_src(c), from_j ? jj : ii, from_j ? ii : jj, att_w);
    return vol_sum<T, K, NW>(c, att, att_w, ii, jj);
}

// G(i, j) and G(j, i) together (lanes share j; the march goes from i): the
// optical depth along the segment (and along each reflected path, whose wall point
// is the same seen from either end) is shared; each entry takes its own source
// star and quadrature.
template <typename T, bool K, int NW = kAnyWalls>
__device__ __forceinline__ void volume_entry_pair(const EntryCtx<T, K> &c, int64_t i, int64_t j, T &gij, T &gji) {
    const GridDev &g = c.g;
    int ii[3], jj[3];
    vtx_index(g, i, ii);
    vtx_index(g, j, jj);
    T att_w[6];
    constexpr bool from_j = K;
    const T att = attenuations<T, NW>(g, depth_src(c), from_j ? jj : ii, from_j ? ii : jj, att_w);
    gij = vol_sum<T, K, NW>(c, att, att_w, ii, jj);
    gji = vol_sum<T, K, NW>(c, att, att_w, jj, ii);
    if constexpr (NW == kAnyWalls) {   // removed vertices have zero rows
        if (!vertex_active(g, ii)) gij = (T)0;
        if (!vertex_active(g, jj)) gji = (T)0;
    }
}

// ---------------------------------------------------------------- surface quadrature
// The wall kernel without its normal-distance factor: 1 / r^3 for the
// isotropic source (eq. SE1, times |d|), 1 / r^4 for the cosine-weighted one
// of Section "Example" (C2, times d^2).
template <typename T, bool C2>
__device__ __forceinline__ T wall_kernel(T r2) {
    if constexpr (C2) return recip(r2 * r2);
    else return recip(r2 * sqrt(r2));
}

template <typename T, int NQ, bool C2, int t>
__device__ __forceinline__ void tri_term(const T *__restrict__ tab, const int lb, const int lc, const int nb,
                                         const int nc, const T db, const T dc, const T da2, const T hb2,
                                         const T hc2, T &acc) {
    constexpr TriInfo ti = kStar.tri[t];
    const int sb = lb - ti.ob, sc = lc - ti.oc;
    if (sb < 0 || sb > nb - 2 || sc < 0 || sc > nc - 2) return;
    const T *e = tab + t * NQ * 4;
    T s = (T)0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const T eb = db - e[4 * q + 0], ec = dc - e[4 * q + 1];
        const T r2 = da2 + hb2 * eb * eb + hc2 * ec * ec;
        s += e[4 * q + 2] * wall_kernel<T, C2>(r2);
    }
    acc += s;
}

template <typename T, int NQ, bool C2, int... ts>
__device__ __forceinline__ T tri_all(std::integer_sequence<int, ts...>, const T *__restrict__ tab, int lb, int lc,
                                     int nb, int nc, T db, T dc, T da2, T hb2, T hc2) {
    T acc = (T)0;
    (tri_term<T, NQ, C2, ts>(tab, lb, lc, nb, nc, db, dc, da2, hb2, hc2, acc), ...);
    return acc;
}

// s(x, l) including 1/(4 pi) and the element areas; x given by its grid
// coordinates (possibly outside the box for a mirror image) and index.
template <typename T, bool K>
__device__ T surf_quad(const EntryCtx<T, K> &c, const int xi[3], const int ll[3], bool near) {
    const GridDev &g = c.g;
    T acc = (T)0;
#pragma nounroll
    for (int f = 0; f < 6; ++f) {
        if (!((g.emit_faces >> f) & 1u)) continue;
        // the face's axis a and its other axes b < cc, by selects (an index into the grid's
        // arrays that is not a compile-time constant copies the kernel argument to scratch)
        const bool a0 = f < 2, a2 = f >= 4;
        const int na = a0 ? g.n[0] : (a2 ? g.n[2] : g.n[1]), nb = a0 ? g.n[1] : g.n[0], nc = a2 ? g.n[1] : g.n[2];
        const int la = a0 ? ll[0] : (a2 ? ll[2] : ll[1]), lb = a0 ? ll[1] : ll[0], lc = a2 ? ll[1] : ll[2];
        const int xa = a0 ? xi[0] : (a2 ? xi[2] : xi[1]), xb = a0 ? xi[1] : xi[0], xc = a2 ? xi[1] : xi[2];
        const int pf = (f & 1) ? na - 1 : 0;
        if (la != pf) continue;
        if (xa == pf) {
            // coplanar limit: theta_F(x)/(4 pi) on the diagonal (isotropic), half
            // that for the cosine-weighted source
            if (xb == lb && xc == lc) {
                T frac = (T)1;
                if (xb < 0 || xb > nb - 1) frac = (T)0;
                else if (xb == 0 || xb == nb - 1) frac *= (T)0.5;
                if (xc < 0 || xc > nc - 1) frac = (T)0;
                else if (xc == 0 || xc == nc - 1) frac *= (T)0.5;
                acc += (g.emission ? (T)0.25 : (T)0.5) * frac;
            }
            continue;
        }
        const double ha = a0 ? g.h[0] : (a2 ? g.h[2] : g.h[1]), hb = a0 ? g.h[1] : g.h[0], hc = a2 ? g.h[1] : g.h[2];
        const T da = (T)(xa - pf) * (T)ha;
        const T da2 = da * da;
        const T hb2 = (T)(hb * hb), hc2 = (T)(hc * hc);
        const T db = (T)(xb - lb), dc = (T)(xc - lc);
        constexpr auto seq = std::make_integer_sequence<int, kTris>{};
        T s;
        if (g.emission) {
            s = near ? tri_all<T, 7, true>(seq, c.st.tri_near, lb, lc, nb, nc, db, dc, da2, hb2, hc2)
                     : tri_all<T, 3, true>(seq, c.st.tri_far, lb, lc, nb, nc, db, dc, da2, hb2, hc2);
            s *= da2;
        } else {
            s = near ? tri_all<T, 7, false>(seq, c.st.tri_near, lb, lc, nb, nc, db, dc, da2, hb2, hc2)
                     : tri_all<T, 3, false>(seq, c.st.tri_far, lb, lc, nb, nc, db, dc, da2, hb2, hc2);
            s *= fabs(da);
        }
        acc += s * (T)(a0 ? g.area_scale[0] : (a2 ? g.area_scale[2] : g.area_scale[1]));
    }
    return acc;
}

// The general mode's surface quadrature: the emitting rectangles are the
// emitting box faces (f < 6) and the hole's emitting faces (f >= 6); a square
// emits when it lies in its rectangle and the cell it bounds on the domain
// side is no hole cell (bit ob + 2 oc of sqmask: the square l - (ob, oc)).  A
// rectangle seen from behind adds nothing; on the diagonal in the rectangle's
// plane the planar angle of the emitting squares, pi/2 each, over 4 pi.  For
// the box faces of a mesh without a hole this is surf_quad, term for term.
template <typename T, int NQ, bool C2, int t>
__device__ __forceinline__ void tri_term_m(const T *__restrict__ tab, int sqmask, const T db, const T dc, const T da2,
                                           const T hb2, const T hc2, T &acc) {
    constexpr TriInfo ti = kStar.tri[t];
    if (!((sqmask >> (ti.ob + 2 * ti.oc)) & 1)) return;
    const T *e = tab + t * NQ * 4;
    T s = (T)0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const T eb = db - e[4 * q + 0], ec = dc - e[4 * q + 1];
        const T r2 = da2 + hb2 * eb * eb + hc2 * ec * ec;
        s += e[4 * q + 2] * wall_kernel<T, C2>(r2);
    }
    acc += s;
}

template <typename T, int NQ, bool C2, int... ts>
__device__ __forceinline__ T tri_all_m(std::integer_sequence<int, ts...>, const T *__restrict__ tab, int sqmask, T db,
                                       T dc, T da2, T hb2, T hc2) {
    T acc = (T)0;
    (tri_term_m<T, NQ, C2, ts>(tab, sqmask, db, dc, da2, hb2, hc2, acc), ...);
    return acc;
}

template <typename T, bool K>
__device__ T surf_quad_rects(const EntryCtx<T, K> &c, const int xi[3], const int ll[3], bool near) {
    const GridDev &g = c.g;
    T acc = (T)0;
    for (int f = 0; f < 12; ++f) {
        const bool box = f < 6;
        const int fb = box ? f : f - 6;
        if (!(((box ? g.emit_faces : g.hole_emit) >> fb) & 1u)) continue;
        const int a = fb / 2, hi_side = fb & 1;
        const int b = (a == 0) ? 1 : 0;
        const int cc = (a == 2) ? 1 : 2;
        // the rectangle's plane, inward normal sign and square ranges [lo, hi), by selects
        int pf = 0, rlo[2] = {0, 0}, rhi[2] = {0, 0};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int lo_k = box ? 0 : g.hole_lo[k], hi_k = box ? g.n[k] - 1 : g.hole_hi[k];
            if (k == a) pf = hi_side ? hi_k : lo_k;
            if (k == b) { rlo[0] = lo_k; rhi[0] = hi_k; }
            if (k == cc) { rlo[1] = lo_k; rhi[1] = hi_k; }
        }
        const int sign = box ? (hi_side ? -1 : 1) : (hi_side ? 1 : -1);
        if (ll[a] != pf) continue;
        int sqmask = 0;
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const int sb = ll[b] - (o & 1), sc = ll[cc] - (o >> 1);
            if (sb < rlo[0] || sb >= rhi[0] || sc < rlo[1] || sc >= rhi[1]) continue;
            bool covered = false;
            if (box && g.has_hole) {
                int cell[3];
                cell[0] = a == 0 ? (sign > 0 ? pf : pf - 1) : (b == 0 ? sb : sc);
                cell[1] = a == 1 ? (sign > 0 ? pf : pf - 1) : (b == 1 ? sb : sc);
                cell[2] = a == 2 ? (sign > 0 ? pf : pf - 1) : sc;
                covered = cell[0] >= g.hole_lo[0] && cell[0] < g.hole_hi[0] && cell[1] >= g.hole_lo[1] &&
                          cell[1] < g.hole_hi[1] && cell[2] >= g.hole_lo[2] && cell[2] < g.hole_hi[2];
            }
            sqmask |= covered ? 0 : (1 << o);
        }
        if (xi[a] == pf) {
            // coplanar limit: theta(x)/(4 pi) on the diagonal, pi/2 per emitting square
            // (isotropic), half that for the cosine-weighted source
            if (xi[0] == ll[0] && xi[1] == ll[1] && xi[2] == ll[2])
                acc += (g.emission ? (T)0.0625 : (T)0.125) * (T)__builtin_popcount(sqmask);
            continue;
        }
        const int d = (xi[a] - pf) * sign;
        if (d <= 0) continue;
        T ha = (T)0, hb2 = (T)0, hc2 = (T)0, as = (T)0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k == a) { ha = (T)g.h[k]; as = (T)g.area_scale[k]; }
            if (k == b) hb2 = (T)(g.h[k] * g.h[k]);
            if (k == cc) hc2 = (T)(g.h[k] * g.h[k]);
        }
        const T da = (T)d * ha;
        const T da2 = da * da;
        const T db = (T)(xi[b] - ll[b]), dc = (T)(xi[cc] - ll[cc]);
        constexpr auto seq = std::make_integer_sequence<int, kTris>{};
        T s;
        if (g.emission) {
            s = near ? tri_all_m<T, 7, true>(seq, c.st.tri_near, sqmask, db, dc, da2, hb2, hc2)
                     : tri_all_m<T, 3, true>(seq, c.st.tri_far, sqmask, db, dc, da2, hb2, hc2);
            s *= da2;
        } else {
            s = near ? tri_all_m<T, 7, false>(seq, c.st.tri_near, sqmask, db, dc, da2, hb2, hc2)
                     : tri_all_m<T, 3, false>(seq, c.st.tri_far, sqmask, db, dc, da2, hb2, hc2);
            s *= da;
        }
        acc += s * as;
    }
    return acc;
}

// S(i, l) from the attenuations of the pair
template <typename T, bool K, int NW>
__device__ __forceinline__ T surf_sum(const EntryCtx<T, K> &c, T att, const T att_w[6], const int ii[3], const int ll[3]) {
    const GridDev &g = c.g;
    if constexpr (NW == kAnyWalls) {
        T S = att == (T)0 ? (T)0 : first_term(att, surf_quad_rects(c, ii, ll, cheb3(ii, ll) <= kNearCheb));
        for (int w = 0; w < g.n_walls; ++w) {
            if (att_w[w] == (T)0) continue;
            int mi[3];
            mirror_index(g, w, ii, mi);
            S += att_w[w] * surf_quad_rects(c, mi, ll, cheb3(mi, ll) <= kNearCheb);
        }
        return S;
    } else {
        T S = first_term(att, surf_quad(c, ii, ll, cheb3(ii, ll) <= kNearCheb));
        if constexpr (NW == kOneWall) {
            int mi[3];
            mirror_index(g, 0, ii, mi);
            S += att_w[0] * surf_quad(c, mi, ll, cheb3(mi, ll) <= kNearCheb);
        }
        return S;
    }
}

template <typename T, bool K, int NW = kAnyWalls, bool FROM_J = false>
__device__ T surface_entry(const EntryCtx<T, K> &c, int64_t i, int64_t l) {
    const GridDev &g = c.g;
    int ii[3], ll[3];
    vtx_index(g, i, ii);
    vtx_index(g, l, ll);
    if constexpr (NW == kAnyWalls)
        if (!vertex_active(g, ii)) return (T)0;   // a removed vertex
    T att_w[6];
    constexpr bool from_j = FROM_J && K;
    const T att = attenuations<T, NW>(g, depth_src(c), from_j ? ll : ii, from_j ? ii : ll, att_w);
    return surf_sum<T, K, NW>(c, att, att_w, ii, ll);
}

template <int KIND, int NW = kAnyWalls, bool FROM_J = false, typename T, bool K>
__device__ __forceinline__ T entry(const EntryCtx<T, K> &c, int64_t i, int64_t j) {
    if constexpr (KIND == RTE_VOLUME) return volume_entry<T, K, NW, FROM_J>(c, i, j);
    else return surface_entry<T, K, NW, FROM_J>(c, i, j);
}

// The entry of a pair shared by a group of P lanes (group_attenuations); every
// lane returns it.
template <int KIND, int NW, bool FROM_J, typename T, bool K>
__device__ __forceinline__ T group_entry(const EntryCtx<T, K> &c, int64_t i, int64_t j, int P, int sub,
                                         GroupTask<T, K> *buf) {
    const GridDev &g = c.g;
    int ii[3], jj[3];
    vtx_index(g, i, ii);
    vtx_index(g, j, jj);
    if constexpr (NW == kAnyWalls)
        if (!vertex_active(g, ii)) return (T)0;   // a removed vertex
    T att_w[6];
    constexpr bool from_j = FROM_J && K;
    const T att = group_attenuations<NW>(g, depth_src(c), from_j ? jj : ii, from_j ? ii : jj, att_w, P, sub, buf);
    if constexpr (KIND == RTE_VOLUME) return vol_sum<T, K, NW>(c, att, att_w, ii, jj);
    else return surf_sum<T, K, NW>(c, att, att_w, ii, jj);
}

}  // namespace rte
