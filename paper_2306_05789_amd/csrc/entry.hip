// Kernels that evaluate kernel entries directly: arbitrary (row, col) pairs,
// and the dense near-field leaves of the H-matrix (Section "Compression": a
// block that reaches the leaves without being admissible is computed in full).
#include <algorithm>
#include <cmath>

#include "entry_dev.h"

namespace rte {

template <typename T, bool K, int KIND>
__global__ __launch_bounds__(256) void k_entries(EntryCtx<T, K> c, int64_t n, const int64_t *__restrict__ rows,
                                                 const int64_t *__restrict__ cols, double *__restrict__ out) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    out[k] = (double)entry<KIND>(c, rows[k], cols[k]);
}

// One task = up to kFillChunk consecutive entries (column-major) of one
// dense block: the lanes of a wavefront march rays from a cluster of targets
// to one source and write contiguous rows of the leaf-sliced storage.  FP64:
// a task is spread over kFillChunk / 256 workgroups of one entry per thread
// (with a loop over entries the compiler hoists the quadrature tables'
// uniform loads into scalar registers, which spill at FP64 width and cost
// an occupancy step).  FP32: one workgroup loops over the task's entries,
// the hoisted tables being the cheaper form there (measured: 2x faster).
template <typename T>
constexpr int fill_split() { return sizeof(T) == 8 ? kFillChunk / 256 : 1; }
static_assert(kFillChunk % 256 == 0, "fill tasks are whole workgroups");

// KIND of the tasks that fill a volume block and its transpose together
constexpr int kPairedVolume = 2;

template <typename T, bool K, int KIND, bool SPLIT, int NW>
__device__ __forceinline__ void fill_one(const EntryCtx<T, K> &c, const FillTask &tk, int64_t e,
                                         const int64_t *__restrict__ tgt_nat, const int64_t *__restrict__ src_nat,
                                         const SliceMap &sm) {
    const int64_t jl = e / tk.m, il = e - jl * tk.m;
    auto put = [&](void *out, void *outlo, int64_t o, T v) {
        if constexpr (SPLIT) {
            const uint16_t h = f2bf((float)v);
            static_cast<uint16_t *>(out)[o] = h;
            static_cast<uint16_t *>(outlo)[o] = f2bf((float)v - bf2f(h));
        } else {
            static_cast<T *>(out)[o] = v;
        }
    };
    // the stored positions are looked up after the entries (not live through the march)
    if constexpr (KIND == kPairedVolume) {
        // this entry and its transpose (the volume tree's targets and sources coincide)
        T v, vt;
        volume_entry_pair<T, K, NW>(c, tgt_nat[tk.t0 + il], tgt_nat[tk.s0 + jl], v, vt);
        put(tk.out, tk.outlo,
            slice_offset(sm, tk.li0, tk.t0 + il, tk.kw, sm.src_p[tk.s0 + jl] - sm.src_p[tk.s0], tk.li0 + (int)il + 1),
            v);
        put(tk.out_t, tk.outlo_t,
            slice_offset(sm, tk.li0_t, tk.s0 + jl, tk.kw_t, sm.src_p[tk.t0 + il] - sm.src_p[tk.t0],
                         tk.li0_t + (int)jl + 1),
            vt);
    } else {
        const T v = entry<KIND, NW, true>(c, tgt_nat[tk.t0 + il], src_nat[tk.s0 + jl]);
        put(tk.out, tk.outlo,
            slice_offset(sm, tk.li0, tk.t0 + il, tk.kw, sm.src_p[tk.s0 + jl] - sm.src_p[tk.s0], tk.li0 + (int)il + 1),
            v);
    }
}

template <typename T, bool K, int KIND, bool SPLIT, int NW>
__global__ __launch_bounds__(256, sizeof(T) == 8 ? 4 : 3) void k_dense_fill(EntryCtx<T, K> c,
                                                                        const FillTask *__restrict__ tasks,
                                                                        const int64_t *__restrict__ tgt_nat,
                                                                        const int64_t *__restrict__ src_nat,
                                                                        SliceMap sm) {
    constexpr int split = fill_split<T>();
    const FillTask tk = tasks[blockIdx.x / split];
    const int64_t total = (int64_t)tk.m * tk.n;
    if constexpr (split == kFillChunk / 256) {
        const int64_t e = tk.first + (int64_t)(blockIdx.x % split) * 256 + threadIdx.x;
        if (e < total) fill_one<T, K, KIND, SPLIT, NW>(c, tk, e, tgt_nat, src_nat, sm);
    } else {
        const int64_t end = min(total, tk.first + (int64_t)kFillChunk);
        for (int64_t e = tk.first + threadIdx.x; e < end; e += blockDim.x)
            fill_one<T, K, KIND, SPLIT, NW>(c, tk, e, tgt_nat, src_nat, sm);
    }
}

__global__ void k_to_float(const double *__restrict__ in, float *__restrict__ out, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) out[k] = (float)in[k];
}

void to_float(const double *in, float *out, int64_t n, hipStream_t s) {
    if (n == 0) return;
    k_to_float<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(in, out, n);
    HIP_LAUNCH_CHECK();
}

// The bounds that kink_family's integers need and the quantum's error, over every
// path of the mesh: the straight ones and those reflected at each wall (two legs of the
// unfolded segment, cut at p / M with M = twice the wall axis' cells at most; N, the
// slope of a family, at most the two largest extents together).
//   q / 2 per unit of length is at most 2^-53 on the longest path, half a unit in the
//   last place of 1: exp(-depth) cannot show it;
//   kappa / q <= 2^61, so a jump's upper 32 bits are below 2^30, and the weights
//   k (A - k M), each below N^2 M / 4, sum to at most N^3 M / 6 < 2^32: both halves of a
//   family's sum fit 64 bits.
// On the unit cube this holds below kappa = 256 (128 with a wall) and to 1400 vertices
// per axis (146 with a wall).  Largest error of the depth at 41^3 by kinks and by the march: 1.1e-16
// and 5.6e-16 on a field in [0.3, 0.6], 9e-16 and 7e-15 beside a block of 100; at 1e4,
// where the quantum's bound is 6e-15, still 4e-15 and 4e-14; at 1e8 3e-11 and 3e-16.
double kink_quantum(const GridDev &g, double kmax) {
    int e = 0;
    (void)std::frexp(kmax, &e);   // kmax < 2^e
    if (!std::isfinite(kmax) || e < -900) return 0.0;
    for (int w = -1; w < g.n_walls; ++w) {
        double ext[3], len2 = 0.0, M = 1.0, big = 0.0, next = 0.0;
        for (int a = 0; a < 3; ++a) {
            ext[a] = g.n[a] - 1;
            if (w >= 0 && g.wall_axis[w] == a) {
                ext[a] *= 2.0;
                M = ext[a];
            }
            len2 += ext[a] * ext[a] * g.h[a] * g.h[a];
            next = std::fmax(next, std::fmin(big, ext[a]));
            big = std::fmax(big, ext[a]);
        }
        const double N = big + next;
        if (N * N * N * M / 6.0 >= 4294967296.0 || N * N * M / 4.0 >= 2147483648.0) return 0.0;
        if (!(std::ldexp(std::sqrt(len2), e) <= 512.0)) return 0.0;
    }
    return std::ldexp(1.0, e - 61);
}

// The kinks of kappa (march.h): per family and vertex v of the grid extended by
// one plane on its upper sides, where kappa continues by its nearest value.
// per_q: 1 / q, a power of two.
__global__ void k_kink_table(GridDev g, const double *__restrict__ kap, double per_q, int64_t *__restrict__ out) {
    const int64_t S0 = (int64_t)(g.n[1] + 1) * (g.n[2] + 1), S1 = g.n[2] + 1, M = (g.n[0] + 1) * S0;
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= M) return;
    const int x = (int)(o / S0), y = (int)(o % S0 / S1), z = (int)(o % S1);
    auto k = [&](int dx, int dy, int dz) {
        const int i = min(max(x + dx, 0), g.n[0] - 1), j = min(max(y + dy, 0), g.n[1] - 1),
                  l = min(max(z + dz, 0), g.n[2] - 1);
        return (int64_t)__double2ll_rn(kap[(int64_t)i * g.stride[0] + (int64_t)j * g.stride[1] + l] * per_q);
    };
    const int64_t v = k(0, 0, 0), all = k(1, 1, 1);
    const int64_t x1 = k(1, 0, 0), y1 = k(0, 1, 0), z1 = k(0, 0, 1);
    const int64_t xy = k(1, 1, 0), yz = k(0, 1, 1), xz = k(1, 0, 1);
    // a family of rotation (a, b, c) is stored [v_a][v_b][v_c]
    const int64_t r1 = ((int64_t)y * (g.n[2] + 1) + z) * (g.n[0] + 1) + x, r2 = ((int64_t)z * (g.n[0] + 1) + x) * (g.n[1] + 1) + y;
    out[0 * M + o] = all - yz - v + k(-1, 0, 0);
    out[1 * M + r1] = all - xz - v + k(0, -1, 0);
    out[2 * M + r2] = all - xy - v + k(0, 0, -1);
    out[3 * M + o] = x1 + y1 - v - xy;
    out[4 * M + r1] = y1 + z1 - v - yz;
    out[5 * M + r2] = x1 + z1 - v - xz;
}

DevBuf kink_table(const Mesh &m, const double *kappa, double q, hipStream_t s) {
    const int64_t M = (int64_t)(m.dev.n[0] + 1) * (m.dev.n[1] + 1) * (m.dev.n[2] + 1);
    DevBuf d = DevBuf::scratch(sizeof(int64_t) * 6 * (size_t)M);
    k_kink_table<<<(unsigned)((M + 255) / 256), 256, 0, s>>>(m.dev, kappa, 1.0 / q, d.as<int64_t>());
    HIP_LAUNCH_CHECK();
    return d;
}

// The four vertex values of every (cell base b, Kuhn tetrahedron t) pair, in
// the order tet_sample reads them: b, b + s_L, b + s0 + s1 + 1 - s_S and
// b + s0 + s1 + 1, L and S the tetrahedron's largest and smallest axes
// (t = 2 L + (S > L ? S - 1 : S)).  A vertex past the grid (bases on the
// upper faces) gives 0.
__global__ void k_tet_table(GridDev g, const float *__restrict__ kap, float *__restrict__ out) {
    const int64_t N = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N * 6) return;
    const int64_t b = k / 6;
    const int t = (int)(k - b * 6), L = t >> 1, r = t & 1, S = r < L ? r : r + 1;
    const int64_t s0 = g.stride[0], s1 = g.stride[1];
    const int64_t sL = L == 0 ? s0 : (L == 1 ? s1 : 1), sS = S == 0 ? s0 : (S == 1 ? s1 : 1);
    const int64_t v3 = b + s0 + s1 + 1;
    const int64_t v1 = b + sL, v2 = v3 - sS;
    out[4 * k + 0] = kap[b];
    out[4 * k + 1] = v1 < N ? kap[v1] : 0.0f;
    out[4 * k + 2] = v2 < N ? kap[v2] : 0.0f;
    out[4 * k + 3] = v3 < N ? kap[v3] : 0.0f;
}

// FP64: the eight corner values of every cell base b, in the order of tet_sample (a
// vertex past the grid gives 0)
__global__ void k_cell_table(GridDev g, const double *__restrict__ kap, double *__restrict__ out) {
    const int64_t N = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= N) return;
    const int64_t s0 = g.stride[0], s1 = g.stride[1];
    const int64_t v[8] = {b, b + s0 + s1 + 1, b + s0, b + s1, b + 1, b + s0 + s1, b + s1 + 1, b + s0 + 1};
#pragma unroll
    for (int q = 0; q < 8; ++q) out[8 * b + q] = v[q] < N ? kap[v[q]] : 0.0;
}

template <typename T>
DevBuf march_table(const Mesh &m, const T *kappa, hipStream_t s) {
    if constexpr (std::is_same<T, float>::value) {
        DevBuf d = DevBuf::scratch(sizeof(float) * (size_t)m.N * 24);
        const int64_t n = m.N * 6;
        k_tet_table<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(m.dev, kappa, d.as<float>());
        HIP_LAUNCH_CHECK();
        return d;
    } else {
        DevBuf d = DevBuf::scratch(sizeof(double) * (size_t)m.N * 8);
        k_cell_table<<<(unsigned)((m.N + 255) / 256), 256, 0, s>>>(m.dev, kappa, d.as<double>());
        HIP_LAUNCH_CHECK();
        return d;
    }
}
template DevBuf march_table<double>(const Mesh &, const double *, hipStream_t);
template DevBuf march_table<float>(const Mesh &, const float *, hipStream_t);

// Rows of the star table (StarTab) from the mesh's near and far tables: a workgroup
// takes 64 offsets d, a wavefront of it one of the cells around the source, whose corner
// weights it adds in LDS; then the rows' 16 sums over the cells.  11^3 14 us, 41^3 (340
// MB) 114; a lane per offset: 32 and 140.
constexpr int kStarRows = 64;   // rows per workgroup
__global__ __launch_bounds__(kStarRows * 8) void k_star_table(GridDev g, StarTab st, int64_t rows,
                                                              const double *__restrict__ near, double *__restrict__ w,
                                                              double *__restrict__ cell) {
    __shared__ double c[8][8][kStarRows + 1];   // [cell][corner][row]
    const int r = threadIdx.x & 63, bits = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * kStarRows, row = row0 + r;
    if (row < rows) {
        const int d[3] = {(int)(row / st.st0) + st.lo[0], (int)(row % st.st0 / st.st1) + st.lo[1],
                          (int)(row % st.st1) + st.lo[2]};
        if (max(max(abs(d[0]), abs(d[1])), abs(d[2])) <= kNearCheb) {
            const double *nr = near + ((d[0] + 2) * 25 + (d[1] + 2) * 5 + (d[2] + 2)) * 64 + bits * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) c[bits][e][r] = nr[e];
        } else {
            const double *far = near + kNearSize;
            const double D2 = g.h[0] * g.h[0] * d[0] * d[0] + g.h[1] * g.h[1] * d[1] * d[1] + g.h[2] * g.h[2] * d[2] * d[2];
#pragma unroll
            for (int e = 0; e < 8; ++e) c[bits][e][r] = 0.0;
            for (int t = 0; t < kTets; ++t) {
                const TetInfo &ti = kStarDev.tet[t];
                if (ti.bits != bits) continue;
                double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double *e = far + (t * 4 + q) * 8;
                    const double ri = 1.0 / (D2 + e[3] + e[0] * d[0] + e[1] * d[1] + e[2] * d[2]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) a[k] += e[4 + k] * ri;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) c[bits][corner_of(ti.slot[k], bits)][r] += a[k];
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) cell[row * 64 + bits * 8 + e] = c[bits][e][r] * g.vol_scale;
    }
    __syncthreads();
    for (int x = threadIdx.x; x < kStarRows * kStarWeights; x += kStarRows * 8) {
        const int rr = x / kStarWeights, v = x % kStarWeights;
        if (row0 + rr >= rows) break;
        double sum = 0.0;
        if (v < 15) {
            const int slot = star_slot(v), p0 = slot / 9 - 1, p1 = slot / 3 % 3 - 1, p2 = slot % 3 - 1;
#pragma unroll
            for (int o = 0; o < 8; ++o) {   // the vertex j + p is a corner of the cell j - o
                const int e0 = p0 + (o & 1), e1 = p1 + ((o >> 1) & 1), e2 = p2 + ((o >> 2) & 1);
                if (((e0 | e1 | e2) & ~1) == 0) sum += c[o][e0 | (e1 << 1) | (e2 << 2)][rr];
            }
        }
        w[(row0 + rr) * kStarWeights + v] = sum * g.vol_scale;
    }
}

StarBuf star_table(const Mesh &m, size_t room, hipStream_t s) {
    // checking aid: RTE_STAR_TABLE=0 in the environment sums the rules point by point
    if (const char *e = std::getenv("RTE_STAR_TABLE"))
        if (std::atoi(e) == 0) return StarBuf{};
    StarBuf r;
    StarTab &t = r.tab;
    const GridDev &g = m.dev;
    int64_t n[3], rows = 1;
    for (int a = 0; a < 3; ++a) {
        int64_t lo = -(g.n[a] - 1), hi = g.n[a] - 1;   // mirror images reach one box further
        for (int w = 0; w < g.n_walls; ++w)
            if (g.wall_axis[w] == a) (g.wall_side[w] ? hi : lo) *= 2;
        t.lo[a] = (int)lo;
        n[a] = hi - lo + 1;
        rows *= n[a];
    }
    if ((double)rows * kStarRow * sizeof(double) > (double)room) return StarBuf{};
    t.st0 = (int)(n[1] * n[2]);
    t.st1 = (int)n[2];
    const double *near = static_cast<const double *>(m.near_table(true));
    try {
        r.buf = DevBuf::scratch((size_t)rows * kStarRow * sizeof(double));
    } catch (const Error &) {   // no room for it now
        (void)hipGetLastError();
        return StarBuf{};
    }
    double *p = r.buf.as<double>();
    t.w = p;
    t.cell = p + rows * kStarWeights;
    poison(r.buf, s);
    k_star_table<<<(unsigned)((rows + kStarRows - 1) / kStarRows), kStarRows * 8, 0, s>>>(g, t, rows, near, p,
                                                                                         p + rows * kStarWeights);
    HIP_LAUNCH_CHECK();
    return r;
}

template <typename T, bool K>
EntryCtx<T, K> make_ctx(const Mesh &m, BandKappa<T, K> kappa) {
    EntryCtx<T, K> c;
    c.g = m.dev;
    c.kappa = kappa.v;
    c.tab = kappa.tab;
    c.q = kappa.q;
    c.near = static_cast<const T *>(m.near_table(std::is_same<T, double>::value));
    if constexpr (std::is_same<T, double>::value) {
        c.star = kappa.star;
        c.st = stencil_device().d;
    } else {
        c.st = stencil_device().f;
    }
    return c;
}
template EntryCtx<double, true> make_ctx(const Mesh &, BandKappa<double, true>);
template EntryCtx<double, false> make_ctx(const Mesh &, BandKappa<double, false>);
template EntryCtx<float, false> make_ctx(const Mesh &, BandKappa<float, false>);

void entries_launch(const Mesh &m, int kind, const double *kappa, double kmax, int64_t n, const int64_t *rows,
                    const int64_t *cols, double *out, int precision, hipStream_t s) {
    if (n == 0) return;
    const unsigned grid = (unsigned)((n + 255) / 256);
    auto launch = [&](auto bk) {   // the band's tables are released after it
        auto c = make_ctx(m, bk);
        using T = std::remove_const_t<std::remove_pointer_t<decltype(bk.v)>>;
        constexpr bool K = std::is_same<decltype(bk), BandKappa<T, true>>::value;
        if (kind == RTE_VOLUME) k_entries<T, K, RTE_VOLUME><<<grid, 256, 0, s>>>(c, n, rows, cols, out);
        else k_entries<T, K, RTE_SURFACE><<<grid, 256, 0, s>>>(c, n, rows, cols, out);
        HIP_LAUNCH_CHECK();
        HIP_CHECK(hipStreamSynchronize(s));
    };
    if (precision == RTE_FP64) {
        const double q = kink_quantum(m.dev, kmax);
        DevBuf kt = q > 0.0 ? kink_table(m, kappa, q, s) : march_table(m, kappa, s);
        // The quadrature's table, for fewer entries than vertices only when it is small: 16 entries of 6x5x7
        // with three walls take 182 us point by point and 136 with it; 25^3 (31 us for 66 MB) and larger
        // are as fast without
        StarBuf star;
        if (kind == RTE_VOLUME) {
            size_t room = (size_t)16 << 20, free_b = 0, total_b = 0;
            if (n >= m.N) {
                HIP_CHECK(hipMemGetInfo(&free_b, &total_b));
                room = std::max(room, (free_b + pool_idle_bytes()) / 16);
            }
            star = star_table(m, room, s);
        }
        if (q > 0.0) launch(BandKappa<double, true>{kappa, kt.as<int64_t>(), q, star.tab});
        else launch(BandKappa<double, false>{kappa, kt.as<double>(), 0.0, star.tab});
        settle({&kt, &star.buf});
    } else {
        DevBuf kf = DevBuf::scratch(sizeof(float) * (size_t)m.N);
        to_float(kappa, kf.as<float>(), m.N, s);
        DevBuf kt = march_table(m, kf.as<float>(), s);
        launch(BandKappa<float, false>{kf.as<float>(), kt.as<float>()});
        settle({&kf, &kt});
    }
}

template <typename T, bool K>
void dense_fill_launch(const Mesh &m, int kind, BandKappa<T, K> kappa, const std::vector<FillTask> &tasks,
                       const int64_t *tgt_nat, const int64_t *src_nat, SliceMap sm, bool split, BandStore &B,
                       hipStream_t s) {
    if (tasks.empty()) return;
    // the paired tasks (volume block and transpose) first, then the single ones
    std::vector<FillTask> order;
    order.reserve(tasks.size());
    for (const FillTask &t : tasks)
        if (t.out_t) order.push_back(t);
    const size_t npair = order.size();
    for (const FillTask &t : tasks)
        if (!t.out_t) order.push_back(t);
    RTE_REQUIRE(npair == 0 || kind == RTE_VOLUME, "dense fill: paired tasks are for the volume operator");
    if (order.size() > ((size_t)1 << 31) / fill_split<T>())
        throw std::runtime_error("dense fill: too many tasks for one grid");
    DevBuf dt = upload_scratch(order, s);
    auto c = make_ctx(m, kappa);
    const FillTask *d = dt.as<FillTask>();
    const unsigned gp = (unsigned)(npair * fill_split<T>()), gs = (unsigned)((order.size() - npair) * fill_split<T>());
    const FillTask *ds = d + npair;
    EventPair ev;
    HIP_CHECK(hipEventRecord(ev.a, s));
    auto launch = [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        if (split) {
            if constexpr (sizeof(T) == 4) {   // BF16 parts of FP32 entries
                if (gp) k_dense_fill<T, K, kPairedVolume, true, NW><<<gp, 256, 0, s>>>(c, d, tgt_nat, src_nat, sm);
                if (gs && kind == RTE_VOLUME) k_dense_fill<T, K, RTE_VOLUME, true, NW><<<gs, 256, 0, s>>>(c, ds, tgt_nat, src_nat, sm);
                else if (gs) k_dense_fill<T, K, RTE_SURFACE, true, NW><<<gs, 256, 0, s>>>(c, ds, tgt_nat, src_nat, sm);
            }
        } else {
            if (gp) k_dense_fill<T, K, kPairedVolume, false, NW><<<gp, 256, 0, s>>>(c, d, tgt_nat, src_nat, sm);
            if (gs && kind == RTE_VOLUME) k_dense_fill<T, K, RTE_VOLUME, false, NW><<<gs, 256, 0, s>>>(c, ds, tgt_nat, src_nat, sm);
            else if (gs) k_dense_fill<T, K, RTE_SURFACE, false, NW><<<gs, 256, 0, s>>>(c, ds, tgt_nat, src_nat, sm);
        }
    };
    switch (wall_mode(m.dev)) {
        case kNoWall: launch(std::integral_constant<int, kNoWall>()); break;
        case kOneWall: launch(std::integral_constant<int, kOneWall>()); break;
        default: launch(std::integral_constant<int, kAnyWalls>()); break;
    }
    HIP_LAUNCH_CHECK();
    HIP_CHECK(hipEventRecord(ev.b, s));
    B.fill_events.push_back(std::move(ev));
    B.retire.push_back(std::move(dt));   // read by the queued launches
}
template void dense_fill_launch(const Mesh &, int, BandKappa<double, true>, const std::vector<FillTask> &, const int64_t *,
                                const int64_t *, SliceMap, bool, BandStore &, hipStream_t);
template void dense_fill_launch(const Mesh &, int, BandKappa<double, false>, const std::vector<FillTask> &, const int64_t *,
                                const int64_t *, SliceMap, bool, BandStore &, hipStream_t);
template void dense_fill_launch(const Mesh &, int, BandKappa<float, false>, const std::vector<FillTask> &, const int64_t *,
                                const int64_t *, SliceMap, bool, BandStore &, hipStream_t);

}  // namespace rte
