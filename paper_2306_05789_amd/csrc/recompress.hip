// Recompression of the ACA factors of the admissible blocks.
//
// Section "Compression": the partially pivoted ACA approximates the first
// terms of a block's SVD.  Its factors U (m x k) and V (n x k) are not
// orthogonal, and the rank at which its stopping test fires is usually
// longer than what the SVD of U V^T needs for the same relative Frobenius
// tolerance.  The recompression replaces them by the shortest truncation of
// that SVD within eps (eps: the ACA tolerance), so every later matvec streams
// fewer bytes:
//
//   1. Gram matrices Gu = U^T U and Gv = V^T V (k x k, FP64);
//   2. with D the square roots of their diagonals, the Cholesky factors of the
//      scaled Grams D^-1 G D^-1 = L L^T, so that U = Qu Ru with
//      Ru = L_u^T D_u and Qu = U Ru^-1 (the scaling keeps the Cholesky away
//      from the spread of the ACA columns' norms);
//   3. the core M = Ru Rv^T (U V^T = Qu M Qv^T) and its SVD by one-sided
//      Jacobi rotations of M's columns: M Z = B with orthogonal columns of
//      norms sigma_j (the rotations themselves are not kept, Z = M^T B S^-2, S
//      the diagonal of sigma);
//   4. r = the fewest columns of B, by decreasing sigma, whose dropped sigmas
//      have a norm <= eps ||sigma||;
//   5. U' = U Ru^-1 B_r, V' = V Rv^-1 Z_r = V Ru^T B_r S_r^-2 (a triangular
//      solve and a triangular product on the small matrices, then one product
//      per factor, written in place).
//
// A block whose scaled Gram is numerically singular, or that would not get
// shorter, keeps its ACA factors.  The Gram matrices and the core are FP64
// whatever the storage type; every reduction has a fixed order, so results
// are bitwise reproducible.
#include <cmath>
#include <type_traits>

#include "kernels.h"

namespace rte {

namespace {

constexpr int kRcMax = 96;   // recompressed ranks: up to 96 (larger blocks, a few in a band, keep their factors)

struct RcTask {
    int64_t uoff, voff;   // U^T [kcap][m] and V^T [kcap][n] in the ACA scratch (elements)
    int64_t woff;         // FP64 workspace of the block: Gu, Gv, Mt, Zt (k x k each)
    int32_t m, n, k, idx; // idx: the block's slot in the rank output
};

struct RcApply {
    int32_t task, side, i0, i1;   // rows [i0, i1) of U (side 0) or V (side 1)
};

// Launches go by rank bucket, each with the threads and the LDS its largest rank
// needs (k_rc_gram and k_rc_apply: factor tiles of kb x 33 doubles), so that small
// ranks keep many workgroups per CU.

constexpr int kRcBuckets[] = {16, 32, 48, 64, kRcMax};
constexpr int kRcStaticLds = 7168;   // k_rc_core's fixed LDS (per-rank vectors, flags), rounded up

// Step 1: one workgroup per (block, factor).  The factor's rows are staged
// 32 columns at a time in LDS (FP64); a thread accumulates a 4 x 4 tile of
// the lower triangle of the Gram matrix, passes of 256 tiles cover it.
template <typename T>
__global__ __launch_bounds__(256) void k_rc_gram(const RcTask *__restrict__ tasks, const T *__restrict__ Us,
                                                 const T *__restrict__ Vs, double *__restrict__ W) {
    extern __shared__ double sx[];   // [4 kt][33]
    const RcTask t = tasks[blockIdx.x];
    const int side = blockIdx.y;
    const T *__restrict__ X = side ? Vs + t.voff : Us + t.uoff;
    const int L = side ? t.n : t.m, k = t.k;
    double *__restrict__ G = W + t.woff + (int64_t)side * k * k;
    const int kt = (k + 3) / 4, ntile = kt * (kt + 1) / 2;
    for (int p0 = 0; p0 < ntile; p0 += 256) {
        const int p = p0 + (int)threadIdx.x;
        int a = 0, b = 0;
        if (p < ntile) {   // tile (a, b), a >= b, of lower-triangle index p = a (a + 1) / 2 + b
            a = (int)((sqrt(8.0 * p + 1.0) - 1.0) * 0.5);
            while (a * (a + 1) / 2 > p) --a;
            while ((a + 1) * (a + 2) / 2 <= p) ++a;
            b = p - a * (a + 1) / 2;
        }
        double acc[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
        for (int i0 = 0; i0 < L; i0 += 32) {
            __syncthreads();
            for (int e = threadIdx.x; e < kt * 4 * 32; e += 256) {
                const int l = e >> 5, i = e & 31;
                sx[l * 33 + i] = (l < k && i0 + i < L) ? (double)X[(int64_t)l * L + i0 + i] : 0.0;
            }
            __syncthreads();
            if (p < ntile) {
                for (int i = 0; i < 32; ++i) {
                    double xa[4], xb[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        xa[u] = sx[(4 * a + u) * 33 + i];
                        xb[u] = sx[(4 * b + u) * 33 + i];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[u][v] = fma(xa[u], xb[v], acc[u][v]);
                }
            }
        }
        if (p < ntile) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 4 * a + u, c = 4 * b + v;
                    if (r < k && c < k) {
                        G[(int64_t)r * k + c] = acc[u][v];
                        G[(int64_t)c * k + r] = acc[u][v];
                    }
                }
        }
    }
}

// Steps 2 to 5 (small matrices): one workgroup of 4 KB lanes per block of rank
// k <= KB.  Output: the new rank (-1: keep the ACA factors), and over the global
// Mt and Zt the transforms of U and V, where k_rc_apply reads them.
//
// Bound by the latency of the Jacobi rounds (k - 1 per sweep, about 8 sweeps, a
// barrier each).  8 lanes hold a pair of columns in registers from its dot products
// to its rotation, so a round is one pass over all pairs: a read and a write of M,
// three sums over 8 lanes, one square root, one quotient and one reciprocal root.
// Two matrices in LDS: the core M, and both Cholesky factors in the triangles of
// one square; M's columns lie 8 doubles apart (mod 16), so that the 4 groups that
// an LDS access serves at a time meet different banks.
// 29^3 in 2 bands of mixed precision, recompression in all: 72 -> 20 ms (the Jacobi
// with its rotations accumulated, 16 lanes per pair and 4 matrices in LDS: 280 ms of
// kernels in 4 steps).  U' V'^T against the truncated SVD of 20x18x22 at eps 1e-5:
// 1.1e-14 of the block's norm at most, 5.5e-14 with accumulated rotations.
template <int KB>
struct RcCore {
    static constexpr int E = KB / 8;               // elements of a column per lane
    static constexpr int LD = (KB / 16) * 16 + 8;  // stride of M's columns (KB a multiple of 16)
    static constexpr int LS = KB + 1;              // stride of the factors' square
    static constexpr size_t lds = sizeof(double) * KB * (LD + LS);
};

// sum over a group of 8 lanes (every lane gets it)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double sum8(double v) {
    v = dpp_add<0xB1>(v);     // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E>(v);     // quad_perm [2, 3, 0, 1]
    return dpp_add<0x141>(v); // row_half_mirror: the other quad of the 8
}

// 1 / sqrt(x) and 1 / x for normal x far from the ends of the range, to about one ulp
__device__ __forceinline__ double rsqrt_n(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}
__device__ __forceinline__ double recip_n(double x) {
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(fma(-x, y, 1.0), y, y);
    return y;
}

template <int KB>
__global__ __launch_bounds__(4 * KB) void k_rc_core(const RcTask *__restrict__ tasks, double *__restrict__ W,
                                                    int *__restrict__ rnew, double eps) {
    constexpr int NT = 4 * KB, E = RcCore<KB>::E, LD = RcCore<KB>::LD, LS = RcCore<KB>::LS;
    extern __shared__ double smem[];
    __shared__ double du[KB], dv[KB], dw[KB], dl[2][KB], run[2][KB], sig[KB], wmax[NT / 64];
    __shared__ int order[KB];
    __shared__ int fail, rotated, rk;
    double *const M = smem;            // M[j * LD + i] = M(i, j), zero for k <= i < KB
    double *const S = smem + KB * LD;  // S[p * LS + i] = L_u(p, i), S[i * LS + p] = L_v(p, i), p > i; diagonals in dl
    const RcTask t = tasks[blockIdx.x];
    const int k = t.k, tid = threadIdx.x, grp = tid >> 3, sl = tid & 7;
    const int64_t kk = (int64_t)k * k;
    const double *const Gu = W + t.woff, *const Gv = Gu + kk;
    double *const Tu = W + t.woff + 2 * kk, *const Tv = Tu + kk;   // transforms, column c at c * k
    if (tid == 0) {
        fail = 0;
        rk = k;
    }
    __syncthreads();
    for (int l = tid; l < k; l += NT) {
        du[l] = sqrt(Gu[(int64_t)l * k + l]);
        dv[l] = sqrt(Gv[(int64_t)l * k + l]);
        if (!(du[l] > 0.0) || !(dv[l] > 0.0)) fail = 1;
        dw[l] = du[l] * dv[l];
    }
    __syncthreads();
    if (fail) {
        if (tid == 0) rnew[t.idx] = -1;
        return;
    }
    for (int e = tid; e < k * k; e += NT) {
        const int i = e / k, j = e - i * k;
        // the Grams are symmetric: the lower triangle from Gu, the upper one from Gv
        const double gu = Gu[e] / (du[i] * du[j]), gv = Gv[e] / (dv[i] * dv[j]);
        S[i * LS + j] = i > j ? gu : gv;
        if (i == j) {
            run[0][i] = gu;
            run[1][i] = gv;
        }
    }
    __syncthreads();
    // Cholesky of both scaled Grams at once, column by column, a thread per row
    // (threads 0 .. 2 KB - 1: L_u, the others: L_v); run: the diagonal left
    {
        const int half = tid >= NT / 2 ? 1 : 0, i = tid - half * (NT / 2);
        const int si = half ? 1 : LS, sj = half ? LS : 1;
        for (int j = 0; j < k; ++j) {
            double d = run[half][j];
            const bool bad = !(d > 1e-13);   // numerically dependent columns
            d = bad ? 1.0 : d;
            if (i > j && i < k) {
                double s = S[i * si + j * sj];
#pragma unroll 4
                for (int p = 0; p < j; ++p) s = fma(-S[i * si + p * sj], S[j * si + p * sj], s);
                s *= rsqrt_n(d);
                S[i * si + j * sj] = s;
                run[half][i] = fma(-s, s, run[half][i]);
            } else if (i == j) {
                dl[half][j] = sqrt(d);
                if (bad) fail = 1;
            }
            __syncthreads();
        }
    }
    if (fail) {
        if (tid == 0) rnew[t.idx] = -1;
        return;
    }
    // core M = Ru Rv^T, Ru(i, p) = L_u(p, i) du(p) for p >= i, times a power of two
    // that brings its largest element to [1/2, 1)
    double mx = 0.0;
    for (int e = tid; e < k * KB; e += NT) {
        const int j = e / KB, i = e - j * KB, p0 = i > j ? i : j;
        double s = 0.0;
        if (i < k) {
            s = (p0 == i ? dl[0][i] : S[p0 * LS + i]) * (p0 == j ? dl[1][j] : S[j * LS + p0]) * dw[p0];
#pragma unroll 4
            for (int p = p0 + 1; p < k; ++p) s = fma(S[p * LS + i] * S[j * LS + p], dw[p], s);
        }
        M[j * LD + i] = s;
        mx = fmax(mx, fabs(s));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if ((tid & 63) == 0) wmax[tid >> 6] = mx;
    __syncthreads();
    mx = wmax[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) mx = fmax(mx, wmax[w]);
    if (!(mx > 0.0 && mx < HUGE_VAL)) {   // underflow or overflow of the core
        if (tid == 0) rnew[t.idx] = -1;
        return;
    }
    int ex;
    (void)frexp(mx, &ex);
    for (int e = tid; e < k * KB; e += NT) {
        const int j = e / KB, i = e - j * KB;
        M[j * LD + i] = ldexp(M[j * LD + i], -ex);
    }
    __syncthreads();
    // one-sided Jacobi: sweeps of the round-robin pairing of the columns (a
    // dummy column when k is odd) until a sweep rotates nothing.  A pair is
    // rotated when its columns are not orthogonal to 3e-15 of their norms (V' takes
    // up sigma_1 / sigma_j times what is left; 1e-12 costs 4 % less and leaves 230
    // times as much); couplings below (1e-12 s)^2, s the largest column norm of M,
    // are left: such columns are far beyond any truncation and would only trade
    // rounding noise with the large ones.
    auto column_norms = [&]() {
        for (int j = grp; j < k; j += NT / 8) {
            double c2 = 0.0;
#pragma unroll
            for (int u = 0; u < E; ++u) c2 = fma(M[j * LD + sl + 8 * u], M[j * LD + sl + 8 * u], c2);
            c2 = sum8(c2);
            if (sl == 0) sig[j] = c2;
        }
        __syncthreads();
    };
    column_norms();
    double s2 = 0.0;
    for (int j = 0; j < k; ++j) s2 = fmax(s2, sig[j]);
    const double floor2 = 1e-24 * s2;
    const int n = k + (k & 1);
    for (int sweep = 0; sweep < 30; ++sweep) {
        __syncthreads();
        if (tid == 0) rotated = 0;
        __syncthreads();
        for (int r = 0; r < n - 1; ++r) {
            if (grp < n / 2) {
                int a = grp - 1 + r, b = n - 2 - grp + r;
                a = grp == 0 ? 0 : (a >= n - 1 ? a - (n - 1) : a) + 1;
                b = (b >= n - 1 ? b - (n - 1) : b) + 1;
                if (a < k && b < k) {   // not the dummy column
                    double *const ca = M + a * LD + sl, *const cb = M + b * LD + sl;
                    double x[E], y[E], al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll
                    for (int u = 0; u < E; ++u) {
                        x[u] = ca[8 * u];
                        y[u] = cb[8 * u];
                    }
#pragma unroll
                    for (int u = 0; u < E; ++u) {
                        al = fma(x[u], x[u], al);
                        be = fma(y[u], y[u], be);
                        ga = fma(x[u], y[u], ga);
                    }
                    al = sum8(al);
                    be = sum8(be);
                    ga = sum8(ga);
                    if (ga * ga > 9e-30 * (al * be) && fabs(ga) > floor2) {
                        // t = tan of the angle: the smaller root of t^2 + 2 z t - 1, z = (be - al) / (2 ga)
                        const double d = be - al, h2 = fma(d, d, 4.0 * (ga * ga)), h = h2 * rsqrt_n(h2);
                        const double tt = 2.0 * ga * recip_n(d + copysign(h, d));
                        const double c = rsqrt_n(fma(tt, tt, 1.0)), s = c * tt;
#pragma unroll
                        for (int u = 0; u < E; ++u) {
                            ca[8 * u] = c * x[u] - s * y[u];
                            cb[8 * u] = s * x[u] + c * y[u];
                        }
                        if (sl == 0) rotated = 1;
                    }
                }
            }
            __syncthreads();
        }
        if (!rotated) break;   // read by every thread after the round's barrier
    }
    __syncthreads();
    // singular values (sig: their squares), their decreasing order, the truncation
    // rank: the first c >= 1 whose tail c .. k - 1 is within eps
    column_norms();
    for (int j = tid; j < k; j += NT) {
        int pos = 0;
        for (int i = 0; i < k; ++i) pos += (sig[i] > sig[j] || (sig[i] == sig[j] && i < j)) ? 1 : 0;
        order[pos] = j;
    }
    __syncthreads();
    if (tid < k) {
        double total = 0.0, tail = 0.0;
        for (int c = 0; c < k; ++c) total += sig[order[c]];
        for (int c = k - 1; c >= tid; --c) tail += sig[order[c]];
        if (tid >= 1 && tail <= eps * eps * total) atomicMin(&rk, tid);
    }
    __syncthreads();
    const int r = rk;
    if (r >= k) {
        if (tid == 0) rnew[t.idx] = -1;
        return;
    }
    // transforms, columns c < r by decreasing sigma, b = B(:, order[c]):
    // V: Ru^T b / sigma^2
    for (int e = tid; e < r * k; e += NT) {
        const int c = e / k, p = e - c * k;
        const double *b = M + order[c] * LD;
        double s = dl[0][p] * b[p];
#pragma unroll 4
        for (int i = 0; i < p; ++i) s = fma(S[p * LS + i], b[i], s);
        Tv[(int64_t)c * k + p] = ldexp(du[p] * s / sig[order[c]], -ex);
    }
    __syncthreads();
    // U: Ru^-1 b = D_u^-1 L_u^-T b, solved in place by a group of 8 lanes per column
    for (int c = grp; c < r; c += NT / 8) {
        double *y = M + order[c] * LD;
        for (int i = k - 1; i >= 0; --i) {
            const double v = y[i] * recip_n(dl[0][i]);
            for (int p = sl; p < i; p += 8) y[p] = fma(-S[i * LS + p], v, y[p]);
            if (sl == 0) Tu[(int64_t)c * k + i] = ldexp(v / du[i], ex);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the group's next read of y
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (tid == 0) rnew[t.idx] = r;
}

// Step 5, the products: rows [i0, i1) of a factor, all k of its columns
// staged in LDS, times the kept transform columns; written in place (columns
// 0..r-1 of the factor's transposed storage).
template <typename T>
__global__ __launch_bounds__(256) void k_rc_apply(const RcApply *__restrict__ ap, const RcTask *__restrict__ tasks,
                                                  T *__restrict__ Us, T *__restrict__ Vs, const double *__restrict__ W,
                                                  const int *__restrict__ rnew) {
    extern __shared__ double sx[];   // [k][33]
    const RcApply a = ap[blockIdx.x];
    const RcTask t = tasks[a.task];
    const int r = rnew[t.idx];
    if (r <= 0) return;   // uniform: the block keeps its factors
    T *__restrict__ X = a.side ? Vs + t.voff : Us + t.uoff;
    const int L = a.side ? t.n : t.m, k = t.k, w = a.i1 - a.i0;
    const double *__restrict__ Tm = W + t.woff + (int64_t)(2 + a.side) * k * k;
    for (int e = threadIdx.x; e < k * 32; e += 256) {
        const int l = e >> 5, i = e & 31;
        sx[l * 33 + i] = i < w ? (double)X[(int64_t)l * L + a.i0 + i] : 0.0;
    }
    __syncthreads();
    const int i = threadIdx.x & 31, g = threadIdx.x >> 5;
    if (i >= w) return;
    for (int c = g; c < r; c += 8) {
        const double *__restrict__ col = Tm + (int64_t)c * k;
        double s = 0.0;
        for (int l = 0; l < k; ++l) s = fma(sx[l * 33 + i], col[l], s);
        X[(int64_t)c * L + a.i0 + i] = (T)s;
    }
}

}  // namespace

template <typename T>
void recompress_batch(const std::vector<AcaTask> &tasks, std::vector<int> &rk, T *Us, T *Vs, double eps,
                      BandStore &B, hipStream_t s) {
    // candidates, by rank bucket
    constexpr int NB = sizeof(kRcBuckets) / sizeof(kRcBuckets[0]);
    std::vector<size_t> cand;
    for (int bk = 0; bk < NB; ++bk)
        for (size_t t = 0; t < tasks.size(); ++t) {
            const int k = rk[t], lo = bk ? kRcBuckets[bk - 1] : 1;
            if (k >= 2 && k > lo && k <= kRcBuckets[bk]) cand.push_back(t);
        }
    if (cand.empty()) return;
    EventTimer timer(s);
    timer.start();
    // the LDS a workgroup may ask for (the core of the largest bucket takes 158 KiB of the 160)
    int dev = 0, lds_max = 0;
    HIP_CHECK(hipGetDevice(&dev));
    HIP_CHECK(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    // rounds whose FP64 workspace (4 k^2 per block) stays within 1 GiB
    const int64_t cap_words = (int64_t)1 << 27;
    size_t c0 = 0;
    while (c0 < cand.size()) {
        std::vector<RcTask> rt;
        std::vector<RcApply> ap;
        std::vector<int> bucket_end(NB, 0), apply_end(NB, 0);   // prefix ends per bucket
        int64_t words = 0;
        size_t c1 = c0;
        for (; c1 < cand.size(); ++c1) {
            const AcaTask &a = tasks[cand[c1]];
            const int64_t k = rk[cand[c1]];
            if (!rt.empty() && words + 4 * k * k > cap_words) break;
            const int32_t idx = (int32_t)rt.size();
            rt.push_back({a.uoff, a.voff, words, a.m, a.n, (int32_t)k, idx});
            words += 4 * k * k;
            for (int side = 0; side < 2; ++side) {
                const int L = side ? a.n : a.m;
                for (int i0 = 0; i0 < L; i0 += 32) ap.push_back({idx, side, i0, std::min(L, i0 + 32)});
            }
            int bk = 0;
            while (k > kRcBuckets[bk]) ++bk;
            for (int q = bk; q < NB; ++q) {
                bucket_end[q] = (int)rt.size();
                apply_end[q] = (int)ap.size();
            }
        }
        const int nt = (int)rt.size();
        DevBuf dt = upload_scratch(rt, s), dap = upload_scratch(ap, s);
        DevBuf W = DevBuf::scratch(sizeof(double) * (size_t)words);
        DevBuf dr = DevBuf::scratch(sizeof(int) * (size_t)nt);
        const RcTask *tp = dt.as<RcTask>();
        const RcApply *app = dap.as<RcApply>();
        int t0 = 0, a0 = 0;
        for (int bk = 0; bk < NB; ++bk) {   // the blocks of a bucket: t0..t1, their products a0..a1
            const int t1 = bucket_end[bk], a1 = apply_end[bk], kb = kRcBuckets[bk];
            if (t1 > t0) {
                const size_t tile = sizeof(double) * (size_t)((kb + 3) / 4 * 4) * 33;
                k_rc_gram<T><<<dim3((unsigned)(t1 - t0), 2), 256, tile, s>>>(tp + t0, Us, Vs, W.as<double>());
                auto core = [&](auto kb_c) {
                    constexpr int KB = decltype(kb_c)::value;
                    RTE_REQUIRE(RcCore<KB>::lds + kRcStaticLds <= (size_t)lds_max, "recompression: LDS of the device");
                    k_rc_core<KB><<<(unsigned)(t1 - t0), 4 * KB, RcCore<KB>::lds, s>>>(tp + t0, W.as<double>(),
                                                                                       dr.as<int>(), eps);
                };
                switch (bk) {
                    case 0: core(std::integral_constant<int, kRcBuckets[0]>()); break;
                    case 1: core(std::integral_constant<int, kRcBuckets[1]>()); break;
                    case 2: core(std::integral_constant<int, kRcBuckets[2]>()); break;
                    case 3: core(std::integral_constant<int, kRcBuckets[3]>()); break;
                    default: core(std::integral_constant<int, kRcBuckets[4]>()); break;
                }
                k_rc_apply<T><<<(unsigned)(a1 - a0), 256, sizeof(double) * kb * 33, s>>>(
                    app + a0, tp, Us, Vs, W.as<double>(), dr.as<int>());
                HIP_LAUNCH_CHECK();
            }
            t0 = std::max(t0, t1);
            a0 = std::max(a0, a1);
        }
        std::vector<int> rn(nt);
        HIP_CHECK(hipMemcpyAsync(rn.data(), dr.p, sizeof(int) * nt, hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
        for (int q = 0; q < nt; ++q) {
            const size_t t = cand[c0 + q];
            const int64_t mn = (int64_t)tasks[t].m + tasks[t].n;
            B.rc_before += rk[t] * mn;
            if (rn[q] > 0) rk[t] = rn[q];
            B.rc_after += rk[t] * mn;
        }
        for (DevBuf *d : {&dt, &dap, &W, &dr}) B.retire.push_back(std::move(*d));
        c0 = c1;
    }
    timer.stop();
    B.rc_ms += timer.ms();
    B.rc_blocks += (int64_t)cand.size();
}

template void recompress_batch<double>(const std::vector<AcaTask> &, std::vector<int> &, double *, double *, double,
                                       BandStore &, hipStream_t);
template void recompress_batch<float>(const std::vector<AcaTask> &, std::vector<int> &, float *, float *, double,
                                      BandStore &, hipStream_t);

}  // namespace rte
