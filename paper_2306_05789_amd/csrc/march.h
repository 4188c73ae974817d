// Optical depth between grid vertices from the kinks of the P1 kappa along the ray, to
// one rounding of the exact value (FP64 entries; those in FP32, and bands that the kinks
// do not resolve, take the march of march_tets.h).
//
// Along a ray x(s) = V + s D, s in [0, 1], kappa is continuous and piecewise
// linear, with a kink where the ray crosses a face of a Kuhn tetrahedron.  By
// the Peano kernel of the trapezoid rule
//   int_0^w kappa ds = w (kappa(0) + kappa(w)) / 2 - 1/2 sum_k [kappa']_k s_k (w - s_k),
// so every crossing adds a term of its own, whatever the order of the others:
// no merge of the six plane families, no sample of the tetrahedra in between.
//
// The faces lie in six plane families: x_a = const (a = 0, 1, 2) and
// x_a - x_b = const ((a, b) = (0,1), (1,2), (2,0)).  The jump of the slope
// across a face, per unit of the family's coordinate, is a second difference of
// kappa (kappa at the two vertices opposite the face minus the two face
// vertices they are symmetric about), the same in either direction:
//   x_a:       J(v) = k(v + a + d) - k(v + d) - k(v) + k(v - a), d = e_b + e_c, v the low corner of
//              the face's square (both of its triangles have the same jump);
//   x_a - x_b: J(v) = k(v + a) + k(v + b) - k(v) - k(v + a + b), v the face's lowest vertex if the third
//              axis comes last, that vertex plus e_c if it comes first.
// They are tabulated per family and vertex (k_kink_table).  With N = |d(family coordinate)/ds| the
// crossings from a vertex are at s_k = k / N, so a family adds
//   -1/2 (1/N) sum_k J(v_k) k (w N - k),
// and v_k is found by two integer Bresenham updates per crossing: exact, so a
// ray through edges and vertices is treated as the same ray moved by an
// infinitesimal positive offset (the same one in every family), which crosses
// faces only; a moved ray may leave the box by its upper planes,
// where the table holds the continuation of kappa by its nearest value (the
// integral is continuous in the ray, so any continuation gives the same depth).
//
// Nothing is rounded on the way: the table holds the jumps in units of a quantum q, a
// power of two of which every kappa of the band is at most 2^61 (kink_quantum), as
// 64-bit integers, the weights k (w N - k) are integers too (times M when the segment
// is cut at w = p / M), and a family's sum is kept in 96 bits.  What a crossing's term
// loses otherwise comes back times the number of crossings, because the families'
// sums cancel: with jumps and sums in FP64 the error was eps times the largest
// kappa near the ray times N (2e-14 on an ordinary field of 41^3, 1e-6 beside a block of
// 1e8).  Left are kappa rounded to q, at most q / 2 per unit of length, and the few
// roundings of the final sum, carried in two doubles; kink_quantum says for which bands
// q is small enough, the others take the merged march (march_tets.h).  The sum does not
// depend on the end that the ray is walked from.
//
// Bound by the gathers of the table and by integer arithmetic: 18 vector
// instructions and one 8-byte load per crossing, the loads of kMarchAhead
// crossings independent.  A march that merges the six families and samples
// kappa on every piece costs 86 instructions and 32 bytes of loads that wait for
// the merge: ACA entry launches of 41^3 138 -> 67.8 ms (volume) and 37.1 -> 15.6
// (surface), of 13x21x13 with three walls and the hole 42.3 -> 17.4.  Jumps and sums in
// FP64 instead of integers would take 67.1, 15.3 and 16.8.
#pragma once

#include <cstdint>

namespace rte {

// Table of one band's kinks: [6 families][n0 + 1][n1 + 1][n2 + 1] in some order of
// the axes, in units of the quantum q, and kappa itself.  The families x_a and
// x_a - x_b, (a, b, c) a rotation of the axes, are stored [v_a][v_b][v_c]: a wavefront
// marches from one vertex to (or from) a cluster of neighbours, so its lanes meet a
// family's k-th plane side by side, spread over a few cells of the plane, and the
// coordinate that varies fastest within the plane is contiguous.  ACA entry
// launches against one natural order for all families: 41^3 FP64 68.8 -> 67.3 ms.
struct KinkTab {
    const int64_t *__restrict__ tab;
    const double *__restrict__ kappa;   // [N], natural order
    double q;
};

// Crossings in flight per loop step of a family: their loads are independent
// (the indices need no loaded value), so this many are issued before the first
// is used.  A lane that walks one family of a ray for a group (kink_one) takes
// more: there the latency of a launch counts, not its issue slots.  The depth
// does not depend on it.
constexpr int kMarchAhead = 4, kMarchAheadOne = 8;

// a b rounded before it is added to anything: the same wherever the sum is formed
template <typename T>
__device__ __forceinline__ T rounded_product(T a, T b) {
#pragma clang fp contract(off)
    return a * b;
}

// An unevaluated sum h + l of about 106 bits.  add and mul_add do not round h's terms
// away (TwoSum, and the product's own remainder by fma).
struct Dd {
    double h, l;
};
__device__ __forceinline__ Dd dd_add(Dd a, double b) {
#pragma clang fp contract(off)
    const double s = a.h + b, t = s - a.h;
    return {s, ((a.h - (s - t)) + (b - t)) + a.l};
}
__device__ __forceinline__ Dd dd_add(Dd a, Dd b) {
#pragma clang fp contract(off)
    const double s = a.h + b.h, t = s - a.h;
    return {s, ((a.h - (s - t)) + (b.h - t)) + (a.l + b.l)};
}
__device__ __forceinline__ Dd dd_mul_add(Dd a, double x, double y) {   // a + x y
    const double p = rounded_product(x, y);
    return dd_add(a, Dd{p, fma(x, y, -p)});
}

// (1/N) sum_{k < A / M} J(v_k) k (A - k M) of one family, in quanta.  Flat index of v_k: idx0 + k K0 + floor1 S1 +
// floor2 S2, floor_i the floor of k d_i / N, of the value just below when neg_i (the
// moved ray is on the lower side of a lattice plane that the ray itself touches).
template <int AHEAD>
__device__ __forceinline__ Dd kink_family(const int64_t *__restrict__ tab, uint32_t idx, int N, int K0, int d1, int S1,
                                          bool neg1, int d2, int S2, bool neg2, int A, int M) {
    const double Nd = (double)N, rN = N > 0 ? recip(Nd) : 0.0;
    // floor division: (d + 1/2) / N keeps 1/(2 N) away from every integer
    const double q1 = floor(((double)d1 + 0.5) * rN), q2 = floor(((double)d2 + 0.5) * rN);
    const int s1 = (int)fma(-q1, Nd, (double)d1), s2 = (int)fma(-q2, Nd, (double)d2);
    const int step = (int)fma(q1, (double)S1, fma(q2, (double)S2, (double)K0));
    const int last = M == 1 ? A - 1 : (int)floor(((double)A - 0.5) * recip((double)M));   // the largest k < A / M
    // remainders minus N: in [-N, -1], a carry when they reach 0
    int r1 = neg1 ? -1 : -N, r2 = neg2 ? -1 : -N;
    idx -= (uint32_t)((neg1 ? S1 : 0) + (neg2 ? S2 : 0));
    int w = 0, dw = A - M;   // k (A - k M) and its next difference
    int64_t hi = 0;
    uint64_t lo = 0;
    for (int k = 1; k <= last; k += AHEAD) {
        int64_t J[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            r1 += s1;
            r2 += s2;
            const bool c1 = r1 >= 0, c2 = r2 >= 0;
            idx += (uint32_t)(step + (c1 ? S1 : 0) + (c2 ? S2 : 0));
            r1 -= c1 ? N : 0;
            r2 -= c2 ? N : 0;
            // past the last crossing: entry 0, with weight 0
            J[u] = tab[k + u <= last ? idx : 0u];
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            w += dw;
            dw -= 2 * M;
            const int wu = max(w, 0);
            hi += (int64_t)(int32_t)(J[u] >> 32) * wu;
            lo += (uint64_t)(uint32_t)J[u] * (uint32_t)wu;
        }
    }
    // the sum 2^32 hi + lo as two doubles (exact), over N
    hi += (int64_t)(lo >> 32);
    const double h = (double)hi, h32 = h * 4294967296.0;
    const double l = fma((double)(hi - (int64_t)h), 4294967296.0, (double)(uint32_t)lo);
    const double q = rounded_product(h32, rN);
    return {q, rounded_product(fma(-q, Nd, h32) + l, rN)};
}

// One family with slope dG and offset oG of the moved ray along its
// coordinate, up to s = p / M (p = M: the whole segment); the companion
// coordinates have slopes d and offsets o.  M times the family's sum.
template <int AHEAD>
__device__ __forceinline__ Dd kink_plane(const int64_t *__restrict__ tab, uint32_t idx, int dG, double oG, int K, int d1,
                                         double o1, int S1, int d2, double o2, int S2, int p, int M) {
    const int N = dG < 0 ? -dG : dG;
    // a companion coordinate meets the family's plane at the offset o - oG d / dG
    const double gd = (double)dG, sg = dG < 0 ? -1.0 : 1.0;
    const bool neg1 = (o1 * gd - oG * (double)d1) * sg < 0.0, neg2 = (o2 * gd - oG * (double)d2) * sg < 0.0;
    return kink_family<AHEAD>(tab, idx, N, dG < 0 ? -K : K, d1, S1, neg1, d2, S2, neg2, N * p, M);
}

// the moved ray's offsets along the axes, with no integer relation (1, 1/sqrt 2, 1/sqrt 3)
constexpr double kOff0 = 1.0, kOff1 = 0.70710678118654752, kOff2 = 0.57735026918962576;

// M times the sum over the families of (1/N) sum_{k < w N} J k (w N - k) along V + s D, s < w = p / M (p = M:
// the whole segment to the vertex V + D), in quanta.  The axes rotate through one
// loop body (axis a with x_a and x_a - x_b), which keeps the registers of one
// family live at a time (six unrolled families spill).
__device__ __forceinline__ Dd kink_sum(const GridDev &g, const int64_t *__restrict__ tab, const int V[3],
                                       const int D[3], int p, int M) {
    int na = g.n[0] + 1, nb = g.n[1] + 1, nc = g.n[2] + 1;
    const int64_t fam = (int64_t)na * nb * nc;
    int Va = V[0], Vb = V[1], Vc = V[2], Da = D[0], Db = D[1], Dc = D[2];
    double oa = kOff0, ob = kOff1, oc = kOff2;
    Dd sum{0.0, 0.0};
#pragma nounroll
    for (int f = 0; f < 3; ++f) {
        const int Sb = nc, Sa = nb * nc, base = Va * Sa + Vb * Sb + Vc;
        sum = dd_add(sum, kink_plane<kMarchAhead>(tab, (uint32_t)base, Da, oa, Sa, Db, ob, Sb, Dc, oc, 1, p, M));
        sum = dd_add(sum, kink_plane<kMarchAhead>(tab + 3 * fam, (uint32_t)(base + 1), Da - Db, oa - ob, -Sb, Da, oa,
                                                  Sa + Sb + 1, Dc - Da, oc - oa, 1, p, M));
        tab += fam;
        const int n0 = na, v0 = Va, d0 = Da;
        const double o0 = oa;
        na = nb, nb = nc, nc = n0;
        Va = Vb, Vb = Vc, Vc = v0;
        Da = Db, Db = Dc, Dc = d0;
        oa = ob, ob = oc, oc = o0;
    }
    return sum;
}

// length of the grid vector D
__device__ __forceinline__ double grid_length(const GridDev &g, double d0, double d1, double d2) {
    const double x = d0 * g.h[0], y = d1 * g.h[1], z = d2 * g.h[2];
    return sqrt(fma(x, x, fma(y, y, rounded_product(z, z))));
}

__device__ __forceinline__ double vertex_kappa(const GridDev &g, const KinkTab &kt, const int V[3]) {
    return kt.kappa[(int64_t)V[0] * g.stride[0] + V[1] * g.stride[1] + V[2]];
}

// half the length of D times the sum s (at least 0: a path through a vacuum may be
// left with the quanta's rounding)
__device__ __forceinline__ double half_length_times(const GridDev &g, const int D[3], Dd s) {
    return 0.5 * grid_length(g, D[0], D[1], D[2]) * fmax(s.h + s.l, 0.0);
}

// the depth of the segment between vertices P and Q from its kinks
__device__ __forceinline__ double direct_depth(const GridDev &g, const KinkTab &kt, const int P[3], const int Q[3],
                                               Dd kinks) {
    const int D[3] = {Q[0] - P[0], Q[1] - P[1], Q[2] - P[2]};
    const Dd ends = dd_add(Dd{vertex_kappa(g, kt, P), 0.0}, vertex_kappa(g, kt, Q));
    return half_length_times(g, D, dd_add(ends, Dd{-kt.q * kinks.h, -kt.q * kinks.l}));
}

// optical depth of the segment between vertices P and Q
__device__ __forceinline__ double tau_direct(const GridDev &g, const KinkTab &kt, const int P[3], const int Q[3]) {
    const int D[3] = {Q[0] - P[0], Q[1] - P[1], Q[2] - P[2]};
    return direct_depth(g, kt, P, Q, kink_sum(g, kt.tab, P, D, 1, 1));
}

// s + M kappa at X = P + (p / M) (Q - P) on the lattice plane x_a = C (a grid face), where P1 is linear on the
// two triangles of each square's low-to-high diagonal; X's coordinates in its square
// are i / M, so M kappa is a sum of integers times kappa.
__device__ __forceinline__ Dd add_face_kappa(Dd s, const GridDev &g, const KinkTab &kt, int a, int C, const int P[3],
                                             const int Q[3], int p, int M) {
    int64_t v = 0, s1 = 0, s2 = 0;
    double i1 = 0.0, i2 = 0.0;
    bool first = true;
    const double Md = (double)M;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        if (b == a) {
            v += (int64_t)C * g.stride[b];
            continue;
        }
        const double num = (double)(Q[b] - P[b]) * (double)p, q = floor(num / Md);
        int cell = P[b] + (int)q;
        double i = num - q * Md;
        if (cell > g.n[b] - 2) {   // on the upper edge of the face
            i += Md * (double)(cell - (g.n[b] - 2));
            cell = g.n[b] - 2;
        }
        v += (int64_t)cell * g.stride[b];
        if (first) { i1 = i; s1 = g.stride[b]; first = false; }
        else { i2 = i; s2 = g.stride[b]; }
    }
    const double hi = fmax(i1, i2), lo = fmin(i1, i2);
    s = dd_mul_add(s, Md - hi, kt.kappa[v]);
    s = dd_mul_add(s, hi - lo, kt.kappa[v + (i1 >= i2 ? s1 : s2)]);
    return dd_mul_add(s, lo, kt.kappa[v + s1 + s2]);
}

// The two legs of a path reflected at the plane x_a = C: from P and from Q
// towards the wall (p, q their distances from it), along the unfolded segment
// of p + q planes.
struct Legs {
    int p, q, D1[3], D2[3];
};
__device__ __forceinline__ Legs reflect_legs(int a, int C, const int P[3], const int Q[3]) {
    Legs l;
    l.p = l.q = 0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        l.D1[b] = Q[b] - P[b];
        l.D2[b] = P[b] - Q[b];
        if (b == a) {
            l.p = P[b] < C ? C - P[b] : P[b] - C;
            l.q = Q[b] < C ? C - Q[b] : Q[b] - C;
            l.D1[b] = l.D2[b] = C > 0 ? l.p + l.q : -(l.p + l.q);   // C > 0: the upper wall
        }
    }
    return l;
}

// The depth of a reflected path from the kinks of its two legs (M times their sum,
// M = p + q).
__device__ __forceinline__ double reflected_depth(const GridDev &g, const KinkTab &kt, int a, int C, const int P[3],
                                                  const int Q[3], const Legs &l, Dd kinks) {
    const int M = l.p + l.q;
    // the terms of P and Q alike, so that the depth is the same from either end
    const double kp = vertex_kappa(g, kt, P), kq = vertex_kappa(g, kt, Q);
    const double xp = rounded_product((double)l.p, kp), xq = rounded_product((double)l.q, kq);
    const Dd rp{xp, fma((double)l.p, kp, -xp)}, rq{xq, fma((double)l.q, kq, -xq)};
    Dd s = add_face_kappa(dd_add(rp, rq), g, kt, a, C, P, Q, l.p, M);
    s = dd_add(s, Dd{-kt.q * kinks.h, -kt.q * kinks.l});
    return half_length_times(g, l.D1, s) / (double)M;
}

// Optical depth of the path from P to the plane x_a = C and on to Q, reflected
// there: two legs from the vertices to the wall point X, which is p / M of the
// unfolded segment from P (M = p + q).
__device__ __forceinline__ double tau_reflected(const GridDev &g, const KinkTab &kt, int a, int C, const int P[3],
                                                const int Q[3]) {
    const Legs l = reflect_legs(a, C, P, Q);
    const int M = l.p + l.q;
    if (M == 0) return tau_direct(g, kt, P, Q);   // both vertices on the wall: the path lies in it
    const Dd k1 = kink_sum(g, kt.tab, P, l.D1, l.p, M), k2 = kink_sum(g, kt.tab, Q, l.D2, l.q, M);
    return reflected_depth(g, kt, a, C, P, Q, l, dd_add(k1, k2));
}

// Family f (0..5) alone of the segment V + s D, s < p / M, for one lane of a
// group that shares a ray; add_families adds the six as kink_sum does, bit for
// bit.
__device__ __forceinline__ Dd kink_one(const GridDev &g, const int64_t *__restrict__ tab, const int V[3],
                                       const int D[3], int p, int M, int f) {
    const int n0 = g.n[0] + 1, n1 = g.n[1] + 1, n2 = g.n[2] + 1;
    const int64_t fam = (int64_t)n0 * n1 * n2;
    const bool diag = f >= 3;
    const int r = diag ? f - 3 : f;
    const int nb = r == 0 ? n1 : (r == 1 ? n2 : n0), nc = r == 0 ? n2 : (r == 1 ? n0 : n1);
    const int Va = r == 0 ? V[0] : (r == 1 ? V[1] : V[2]), Vb = r == 0 ? V[1] : (r == 1 ? V[2] : V[0]),
              Vc = r == 0 ? V[2] : (r == 1 ? V[0] : V[1]);
    const int Da = r == 0 ? D[0] : (r == 1 ? D[1] : D[2]), Db = r == 0 ? D[1] : (r == 1 ? D[2] : D[0]),
              Dc = r == 0 ? D[2] : (r == 1 ? D[0] : D[1]);
    const double oa = r == 0 ? kOff0 : (r == 1 ? kOff1 : kOff2), ob = r == 0 ? kOff1 : (r == 1 ? kOff2 : kOff0),
                 oc = r == 0 ? kOff2 : (r == 1 ? kOff0 : kOff1);
    const int Sb = nc, Sa = nb * nc, base = Va * Sa + Vb * Sb + Vc;
    return kink_plane<kMarchAheadOne>(tab + f * fam, (uint32_t)(diag ? base + 1 : base), diag ? Da - Db : Da,
                                      diag ? oa - ob : oa, diag ? -Sb : Sa, diag ? Da : Db, diag ? oa : ob,
                                      diag ? Sa + Sb + 1 : Sb, diag ? Dc - Da : Dc, diag ? oc - oa : oc, 1, p, M);
}

__device__ __forceinline__ Dd add_families(const Dd *f) {
    Dd s = dd_add(Dd{0.0, 0.0}, f[0]);
    s = dd_add(s, f[3]);
    s = dd_add(s, f[1]);
    s = dd_add(s, f[4]);
    s = dd_add(s, f[2]);
    return dd_add(s, f[5]);
}

}  // namespace rte
