// Optical depth by a merged march through the Kuhn tetrahedra: FP32 entries, and FP64
// entries of a band that the kinks of kappa (march.h) do not resolve (kink_quantum).
//
// The march follows the six plane families that bound the Kuhn tetrahedra
// (x_a = const and x_a - x_b = const in grid units): the next crossing of every
// family is kept, the smallest one ends the current piece, and kappa is linear
// on each piece, so the piece contributes its length times kappa at its midpoint.
// No term is larger than the depth, so the error follows the kappa that the ray
// meets, whatever the largest kappa of the band.
//
// FP32 does not take the kinks and the quadrature by offset (vol_quad), which would
// be faster there too (steps of 33x17x17 with one wall in 4 bands 518 -> 237 ms, where
// this takes 327; of 29^3 in 2 bands 277 -> 223, where this takes 259).  It keeps its
// rounding: a block whose ACA ends near its break-even rank is stored dense or low-rank
// on the last bits of its entries.  With entries moved by 1e-7 about 20 of 50,000 blocks
// change sides, which products in FP32 or with both BF16 parts do not show (1e-6) and
// products with the BF16 hi parts alone do: up to 1e-3 of an element, as much as a change
// of the storage type.
#pragma once

namespace rte {

// Minimum of two finite values without the quieting of signalling NaNs that
// fmin() adds on this target (two extra instructions per call in the march).
__device__ __forceinline__ double fmin_finite(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float fmin_finite(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}


// The four vertex values of the Kuhn tetrahedron of a point in the cell with
// flat base index b, at local coordinates (u0, u1, u2) in [0, 1]^3 (grid
// units), and the coordinates sorted decreasingly: kappa there is the P1
// (Freudenthal) interpolant kb + u0 (k1 - kb) + u1 (k2 - k1) + u2 (k3 - k2).  FP64
// takes it by the vertices' weights, none negative: a ray in a face opposite a vertex
// of huge kappa weighs that by an exact 0, where differences of kappa would round at
// its size (8e-10 of the depth beside 1e8).
template <typename T>
struct TetSample {
    T kb, k1, k2, k3, u0, u1, u2;
    __device__ __forceinline__ T value() const {
        if constexpr (sizeof(T) == 8) return ((T)1 - u0) * kb + (u0 - u1) * k1 + (u1 - u2) * k2 + u2 * k3;
        else return kb + u0 * (k1 - kb) + u1 * (k2 - k1) + u2 * (k3 - k2);
    }
};

// The Kuhn tetrahedron of the point is given by the decreasing order of its
// local coordinates: from the base corner it adds the axis of the largest
// coordinate, then that of the middle one.  Ties pick the lowest axis as the
// largest and the highest axis as the smallest, so the two never coincide
// (the value is continuous across the faces the ties lie on).
//
// The vertices are b, b + s_L, b + s0 + s1 + 1 - s_S and b + s0 + s1 + 1 (s_a
// the axis strides, L and S the largest and smallest axes).  They are read from
//   FP32: a table of every (cell base, tetrahedron) pair, the tetrahedron numbered
//   t = 2 L + (S > L ? S - 1 : S): one 16-byte load per piece instead of four
//   gathers over the grid (the ACA entry launches of the 41^3 operator 98.6 ->
//   78.0 ms);
//   FP64: a table of the eight corner values of every cell base, in the order
//   k(b), k(b + s0 + s1 + 1), then b + s0, b + s1, b + 1, b + s0 + s1, b + s1 + 1,
//   b + s0 + 1: three loads from one 64-byte row per piece (the first two values
//   together), as fast as 32-byte rows per tetrahedron.
// A base outside the grid (only the unused sample after a segment's last piece, or a
// piece of rounding length) reads the nearest row.
template <typename T>
struct KappaSrc {
    const T *__restrict__ tab;   // FP32 [N][6][4], FP64 [N][8]
};

template <typename T>
__device__ __forceinline__ TetSample<T> tet_sample(const GridDev &g, const KappaSrc<T> &src, int b, T u0, T u1, T u2) {
    const bool c01 = u0 >= u1, c02 = u0 >= u2, c12 = u1 >= u2;
    const T hi = fmax(fmax(u0, u1), u2), lo = fmin(fmin(u0, u1), u2);
    const T mid = fmax(fmin(u0, u1), fmin(fmax(u0, u1), u2));
    const int nv = g.n[0] * g.n[1] * g.n[2];
    const int bc = min(max(b, 0), nv - 1);
    if constexpr (sizeof(T) == 4) {
        const int L = (c01 && c02) ? 0 : (c12 ? 1 : 2);
        const int S = (c02 && c12) ? 2 : (c01 ? 1 : 0);
        const int t = 2 * L + (S > L ? S - 1 : S);
        const float4 q = *reinterpret_cast<const float4 *>(src.tab + ((int64_t)bc * 6 + t) * 4);
        return {q.x, q.y, q.z, q.w, hi, mid, lo};
    } else {
        // row slots: b + s_L at 2 + L; b + s0 + s1 + 1 - s_S at 6, 7, 5 for S = 0, 1, 2
        const int i1 = (c01 && c02) ? 2 : (c12 ? 3 : 4);
        const int i2 = (c02 && c12) ? 5 : (c01 ? 7 : 6);
        const double *r = src.tab + (int64_t)bc * 8;
        const double2 q = *reinterpret_cast<const double2 *>(r);
        return {q.x, r[i1], r[i2], q.y, hi, mid, lo};
    }
}

// The state of the march along one segment: start() sets it up for P -> Q
// and samples the tetrahedron of its first piece; piece() moves the families
// crossed at the end of the current piece on, samples the next piece's
// tetrahedron into nxt (its loads run while this piece is added) and adds the
// current one, true once that piece ends the segment; tau() is the optical
// depth.
template <typename T>
struct March {
    T D[3], tn[6], dt[6], w[3], ws[3];
    T len, tp, t, acc;
    int b, db[3];

    __device__ __forceinline__ T next_end() const {
        return fmin_finite(fmin_finite(fmin_finite(tn[0], tn[1]), fmin_finite(tn[2], tn[3])),
                           fmin_finite(fmin_finite(tn[4], tn[5]), (T)1));
    }

    // false when the segment has zero length (tau = 0, nothing sampled)
    __device__ __forceinline__ bool start(const GridDev &g, const KappaSrc<T> &kt, const T P[3], const T Q[3],
                                          TetSample<T> &first) {
#pragma unroll
        for (int a = 0; a < 3; ++a) D[a] = Q[a] - P[a];
        const T wx = D[0] * (T)g.h[0], wy = D[1] * (T)g.h[1], wz = D[2] * (T)g.h[2];
        // rounded the same way in every kernel
        len = sqrt(fma(wz, wz, fma(wx, wx, rounded_product(wy, wy))));
        if (len == (T)0) return false;
        const T F0[6] = {P[0], P[1], P[2], P[0] - P[1], P[1] - P[2], P[0] - P[2]};
        const T dF[6] = {D[0], D[1], D[2], D[0] - D[1], D[1] - D[2], D[0] - D[2]};
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            if (dF[f] != (T)0) {
                const T next = dF[f] > (T)0 ? floor(F0[f]) + (T)1 : ceil(F0[f]) - (T)1;
                dt[f] = (T)1 / fabs(dF[f]);
                tn[f] = (next - F0[f]) / dF[f];
            } else {
                dt[f] = (T)0;
                tn[f] = (T)2;   // never before the end of the segment
            }
        }
        // cell of the first piece: along a, the one the segment enters from P
        // (the top cell when the segment lies in the top plane of a)
        b = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int sa = D[a] > (T)0 ? 1 : (D[a] < (T)0 ? -1 : 0);
            int ca = D[a] < (T)0 ? (int)ceil(P[a]) - 1 : (int)floor(P[a]);
            ca = min(max(ca, 0), g.n[a] - 2);
            b += ca * g.stride[a];
            db[a] = sa * g.stride[a];
            w[a] = P[a] - (T)ca;
            ws[a] = (T)sa;
        }
        tp = (T)0;
        t = next_end();
        acc = (T)0;
        const T tm0 = (T)0.5 * t;
        first = tet_sample<T>(g, kt, b, w[0] + tm0 * D[0], w[1] + tm0 * D[1], w[2] + tm0 * D[2]);
        return true;
    }

    __device__ __forceinline__ bool piece(const GridDev &g, const KappaSrc<T> &kt, const TetSample<T> &cur,
                                          TetSample<T> &nxt) {
        const bool last = t >= (T)1;
#pragma unroll
        for (int f = 0; f < 3; ++f)
            if (tn[f] <= t) {
                tn[f] += dt[f];
                b += db[f];
                w[f] -= ws[f];
            }
#pragma unroll
        for (int f = 3; f < 6; ++f)
            if (tn[f] <= t) tn[f] += dt[f];
        const T tq = next_end();
        const T tm = (T)0.5 * (t + tq);
        nxt = tet_sample<T>(g, kt, b, w[0] + tm * D[0], w[1] + tm * D[1], w[2] + tm * D[2]);
        acc += (t - tp) * cur.value();
        tp = t;
        t = tq;
        return last;
    }

    // FP64: not below 0, where a grazed block of huge kappa could take the rounding of a sample
    __device__ __forceinline__ T tau() const {
        if constexpr (sizeof(T) == 8) return fmax(len * acc, 0.0);
        else return len * acc;
    }
};

// every piece advances at least one family: a segment has at most
// sum_f |dF_f| + 7 <= 3 (|D0|+|D1|+|D2|) + 7 pieces
__device__ __forceinline__ int march_cap(const GridDev &g) { return 3 * (g.n[0] + g.n[1] + g.n[2]) + 16; }

// tau along the segment P -> Q given in grid coordinates, both in the closed
// box.  The P1 kappa is linear between consecutive crossings of the six plane
// families, so each piece contributes its length times kappa at its midpoint
// (exact).  The next crossing time of family f advances by the constant
// 1/|dF_f| per crossing; a crossing of family a (a < 3) moves the cell by one
// along axis a, which updates its flat index and P's coordinates relative to
// the cell corner.  Only the last crossing of a family can be taken a few
// rounding units early (the segment ends on a vertex, that is on a plane of
// every family); the piece that follows is of rounding length, and tet_sample
// keeps its loads in bounds.  The loop is software
// pipelined: the kappa values of the next piece are loaded while the current
// one is added (a piece of zero length, where two families cross together,
// adds zero; after the last piece one more sample is loaded and unused).
template <typename T>
__device__ T tau_segment(const GridDev &g, const KappaSrc<T> &kt, const T P[3], const T Q[3]) {
    March<T> m;
    // two named samples in turn, so that no copy closes the loop
    TetSample<T> sa, sb;
    if (!m.start(g, kt, P, Q, sa)) return (T)0;
    const int cap = march_cap(g);
    for (int it = 0; it < cap; it += 2) {
        if (m.piece(g, kt, sa, sb)) break;
        if (m.piece(g, kt, sb, sa)) break;
    }
    return m.tau();
}

// optical depth between the vertices P and Q
template <typename T>
__device__ __forceinline__ T tau_direct(const GridDev &g, const KappaSrc<T> &kt, const int P[3], const int Q[3]) {
    const T p[3] = {(T)P[0], (T)P[1], (T)P[2]}, q[3] = {(T)Q[0], (T)Q[1], (T)Q[2]};
    return tau_segment<T>(g, kt, p, q);
}

// Where the path from P to the plane x_a = C and on to Q meets it: on the segment
// from the mirror image of P to Q.
template <typename T>
__device__ __forceinline__ void wall_point(int a, T C, const T P[3], const T Q[3], T X[3]) {
    T Pb[3] = {P[0], P[1], P[2]};
    Pb[a] = (T)2 * C - P[a];
    const T den = Q[a] - Pb[a];
    if (den == (T)0) {
        X[0] = Q[0]; X[1] = Q[1]; X[2] = Q[2];
    } else {
        const T t = (C - Pb[a]) / den;
#pragma unroll
        for (int b = 0; b < 3; ++b) X[b] = Pb[b] + t * (Q[b] - Pb[b]);
        X[a] = C;
    }
}

// optical depth of the path from P to the plane x_a = C and on to Q
template <typename T>
__device__ __forceinline__ T tau_reflected(const GridDev &g, const KappaSrc<T> &kt, int a, int C, const int P[3],
                                           const int Q[3]) {
    const T p[3] = {(T)P[0], (T)P[1], (T)P[2]}, q[3] = {(T)Q[0], (T)Q[1], (T)Q[2]};
    T X[3];
    wall_point<T>(a, (T)C, p, q, X);
    return tau_segment<T>(g, kt, p, X) + tau_segment<T>(g, kt, X, q);
}

}  // namespace rte
