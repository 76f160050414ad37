// Block conjugate gradients for (alpha L + I) X = B with up to 64 right-hand
// sides (the linear system of Algorithm 1, and the CG ground truth of the
// paper's experiments).  All vectors are row-major (row v holds the k values of
// vertex v), so a neighbour row is one contiguous, coalesced load.  The inner
// vectors r, p, q, d are padded to kp columns (k rounded up to a whole vector
// load of V values; the padding stays zero), so their rows are always loaded 16
// bytes a lane where k allows it; X, B and the residual keep the caller's k.
//
// Mapping: a group of lanes (kp / V rounded up to a power of two) covers one
// row, a wave 64 / group rows.  Rows of more than kLongRow neighbours are cut
// into segments of kSegment entries that a workgroup each sums beforehand; the
// row's own group then adds the segments' sums in order, so that no hub is
// walked by one group alone.
//
// Per-column dot products are reduced in two deterministic stages: each block
// writes its partial sums column by column, then one block per column adds them
// in a fixed order and updates that column's CG scalars.  The host polls the
// columns' activity every few iterations; the kernels of an iteration that
// starts with no active column return at once.
//
// Streams per iteration: p gathered by rows, p read and q written (apply); r, q
// read and r written (update); r, p, d read and p, d written (direction, where
// z = Minv r is formed again rather than stored).
//
// Measured on BA(2 000 000, 8), 64 columns in binary32 (512 MB a vector): apply
// 1.28 ms a pass (9.2 GB asked for, part of it served by the last-level cache),
// segments 0.11, update 0.29, direction 0.57 (both at the rate of a large copy);
// 2.08 ms for apply while each row was one group's, 0.65 + 0.28 ms for the
// vector passes while z was stored and single values loaded.  On BA(200 000, 5),
// 8 columns in binary64, a hub of 3000 neighbours held apply at 230 us; now 36.
// Whole solves (rtol 1e-9 refined, 1e-10): 118.5 -> 62.4 ms and 7.26 -> 2.17 ms.
// Lines lie at 128 entries because eight gathers in flight cover them in 16
// dependent rounds, about the time of one pass over an ordinary wave's rows, and
// a 256-lane segment of 128 entries is one round of loads at 64 columns.
#include <type_traits>

#include "fc_kernels.hpp"

#pragma clang fp contract(off)

namespace fc {

namespace {

constexpr uint32_t kThreads = 256;
constexpr uint32_t kWaves = kThreads / 64u;
constexpr uint32_t kLongRow = kCgLongRow, kSegment = kCgSegment;

// Offsets of the per-column scalars.
constexpr uint32_t kRz = 0, kTol2 = 256, kStep = 320, kBeta = 384, kActive = 448, kIters = 512;

template <typename T, int V>
struct alignas(sizeof(T) * V) Vec {
    T x[V];
};

template <typename T, int V>
__device__ __forceinline__ Vec<T, V> load(const T *p) {
    return *reinterpret_cast<const Vec<T, V> *>(p);
}
template <typename T, int V>
__device__ __forceinline__ void store(T *p, const Vec<T, V> &v) {
    *reinterpret_cast<Vec<T, V> *>(p) = v;
}

struct Lane {
    uint32_t group;  // lanes per row (power of two, <= 64)
    uint32_t sub;    // row within the wave
    uint32_t col;    // first column of this lane
    bool valid;      // col < cols
};

__device__ __forceinline__ Lane lane_map(uint32_t cols, uint32_t V) {
    uint32_t group = 1;
    while (group * V < cols) group <<= 1;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t col = (lane & (group - 1u)) * V;
    return {group, lane / group, col, col < cols};
}

// Rows handled by a wave: step g covers rows g * (64 / group) .. + 64 / group - 1.
__device__ __forceinline__ void row_range(uint32_t *first, uint32_t *stride) {
    *first = blockIdx.x * (blockDim.x / 64u) + (threadIdx.x >> 6);
    *stride = gridDim.x * (blockDim.x / 64u);
}

// Whether any of the k columns is still active.
__device__ __forceinline__ bool any_of(const double *flags, uint32_t k) {
    const uint32_t lane = threadIdx.x & 63u;
    return __ballot(lane < k && flags[lane < k ? lane : 0u] != 0.0) != 0ull;
}

// sum over entries q, q + step, ... below e of w X[u][col ...] (w = 1 without
// weights): U independent gathers in flight, fixed association.
template <typename T, int V, bool kWeighted>
__device__ __forceinline__ Vec<T, V> neighbour_sum(const int32_t *__restrict__ col_idx,
                                                   const double *__restrict__ wt, int32_t q,
                                                   int32_t e, int32_t step,
                                                   const T *__restrict__ X, uint32_t ld,
                                                   uint32_t col) {
    constexpr int U = 8;
    Vec<T, V> s0 = {}, s1 = {};
    for (; e - q > (U - 1) * step; q += U * step) {
        Vec<T, V> x[U];
        T c[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            x[i] = load<T, V>(X + static_cast<size_t>(col_idx[q + i * step]) * ld + col);
            if (kWeighted) c[i] = static_cast<T>(wt[q + i * step]);
        }
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const T y = kWeighted ? c[i] * x[i].x[j] : x[i].x[j];
                if (i & 1) s1.x[j] += y;
                else s0.x[j] += y;
            }
    }
    // the rest: up to U - 1 entries, all loaded before the first is added
    Vec<T, V> x[U - 1];
    T c[U - 1];
#pragma unroll
    for (int i = 0; i < U - 1; ++i) {
        x[i] = {};
        c[i] = T(0);
        if (e - q > i * step) {
            x[i] = load<T, V>(X + static_cast<size_t>(col_idx[q + i * step]) * ld + col);
            if (kWeighted) c[i] = static_cast<T>(wt[q + i * step]);
        }
    }
#pragma unroll
    for (int i = 0; i < U - 1; ++i)
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const T y = kWeighted ? c[i] * x[i].x[j] : x[i].x[j];
            if (i & 1) s1.x[j] += y;
            else s0.x[j] += y;
        }
#pragma unroll
    for (int j = 0; j < V; ++j) s0.x[j] += s1.x[j];
    return s0;
}

// Rows of more than kLongRow entries: seg_base[v] = their first segment,
// seg[s] = {first entry, end} of segment s; *count segments in all.  Segments of
// a row are consecutive; the order of the rows is free (nothing depends on it).
__global__ __launch_bounds__(kThreads) void segments_kernel(const int32_t *__restrict__ row_ptr,
                                                            uint32_t n,
                                                            uint32_t *__restrict__ seg_base,
                                                            int2 *__restrict__ seg,
                                                            uint32_t *count) {
    const uint32_t v = blockIdx.x * kThreads + threadIdx.x;
    if (v >= n) return;
    const int32_t b = row_ptr[v], e = row_ptr[v + 1];
    const uint32_t d = static_cast<uint32_t>(e - b);
    if (d <= kLongRow) return;
    const uint32_t parts = (d + kSegment - 1u) / kSegment;
    const uint32_t base = atomicAdd(count, parts);
    seg_base[v] = base;
    for (uint32_t i = 0; i < parts; ++i) {
        const int64_t s0 = b + static_cast<int64_t>(i) * kSegment;
        const int64_t s1 = s0 + kSegment;
        seg[base + i] = make_int2(static_cast<int32_t>(s0),
                                  static_cast<int32_t>(s1 < e ? s1 : e));
    }
}

// One workgroup per segment (striding): its lane groups take its entries in
// turn, their sums are added in group order into out[segment * ld + column].
template <typename T, int V, bool kWeighted>
__global__ __launch_bounds__(kThreads) void segment_sum_kernel(
    const int32_t *__restrict__ col_idx, const double *__restrict__ wt,
    const int2 *__restrict__ seg, const uint32_t *__restrict__ count, uint32_t cols, uint32_t k,
    const T *__restrict__ X, uint32_t ld, T *__restrict__ out, const double *__restrict__ active) {
    if (active && !any_of(active, k)) return;
    __shared__ Vec<T, V> lds[kThreads];
    const Lane ln = lane_map(cols, V);
    const uint32_t groups = kThreads / ln.group, g = threadIdx.x / ln.group;
    const uint32_t total = *count;
    for (uint32_t s = blockIdx.x; s < total; s += gridDim.x) {
        const int2 r = seg[s];
        Vec<T, V> acc = {};
        if (ln.valid)
            acc = neighbour_sum<T, V, kWeighted>(col_idx, wt, r.x + static_cast<int32_t>(g), r.y,
                                                 static_cast<int32_t>(groups), X, ld, ln.col);
        lds[threadIdx.x] = acc;
        __syncthreads();
        for (uint32_t half = groups >> 1; half > 0; half >>= 1) {
            if (g < half)
#pragma unroll
                for (int j = 0; j < V; ++j)
                    lds[threadIdx.x].x[j] += lds[threadIdx.x + half * ln.group].x[j];
            __syncthreads();
        }
        if (g == 0 && ln.valid) store<T, V>(out + static_cast<size_t>(s) * ld + ln.col, lds[threadIdx.x]);
        __syncthreads();
    }
}

// The neighbour sum of row v, whose segments (if it is long) are already summed.
template <typename T, int V, bool kWeighted>
__device__ __forceinline__ Vec<T, V> row_sum(const CgRows &m, const int32_t *__restrict__ col_idx,
                                             const double *__restrict__ wt, uint32_t v, int32_t b,
                                             int32_t e, const T *__restrict__ X,
                                             const T *__restrict__ seg_sum, uint32_t ld,
                                             uint32_t col) {
    if (static_cast<uint32_t>(e - b) <= kLongRow)
        return neighbour_sum<T, V, kWeighted>(col_idx, wt, b, e, 1, X, ld, col);
    const uint32_t parts = (static_cast<uint32_t>(e - b) + kSegment - 1u) / kSegment;
    const T *p = seg_sum + static_cast<size_t>(m.seg_base[v]) * ld + col;
    Vec<T, V> s = {};
#pragma unroll 8
    for (uint32_t i = 0; i < parts; ++i) {
        const Vec<T, V> x = load<T, V>(p + static_cast<size_t>(i) * ld);
#pragma unroll
        for (int j = 0; j < V; ++j) s.x[j] += x.x[j];
    }
    return s;
}

// Block-level per-column sums of acc into partial[column * gridDim.x + blockIdx.x]:
// across the wave's rows by shuffles, then across the waves in order.
template <int V>
__device__ __forceinline__ void block_column_sum(double (&acc)[V], const Lane &ln, uint32_t k,
                                                 double *__restrict__ partial, double (*lds)[64]) {
#pragma unroll
    for (int j = 0; j < V; ++j) {
        double a = ln.valid ? acc[j] : 0.0;
        for (uint32_t off = 32; off >= ln.group; off >>= 1) a += __shfl_xor(a, off, 64);
        if (ln.sub == 0 && ln.col + j < 64u) lds[threadIdx.x >> 6][ln.col + j] = a;
    }
    __syncthreads();
    if (threadIdx.x < k) {
        double t = 0.0;
        for (uint32_t w = 0; w < kWaves; ++w) t += lds[w][threadIdx.x];
        partial[static_cast<size_t>(threadIdx.x) * gridDim.x + blockIdx.x] = t;
    }
    __syncthreads();
}

// q = A p with A = alpha L + I; partial sums of p.q.
template <typename T, int V, bool kWeighted>
__global__ __launch_bounds__(kThreads) void apply_kernel(
    CgRows m, const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
    const double *__restrict__ wt, const double *__restrict__ wdeg, uint32_t n, uint32_t k,
    uint32_t kp, double alpha, const T *__restrict__ p, const T *__restrict__ seg_sum,
    T *__restrict__ q, double *__restrict__ partial, const double *__restrict__ S) {
    if (!any_of(S + kActive, k)) return;
    __shared__ double lds[kWaves][64];
    const Lane ln = lane_map(kp, V);
    const uint32_t rows = 64u / ln.group;
    uint32_t g0, gs;
    row_range(&g0, &gs);
    const T a = static_cast<T>(alpha);
    double acc[V] = {};
    for (uint32_t g = g0; static_cast<size_t>(g) * rows < n; g += gs) {
        const size_t vl = static_cast<size_t>(g) * rows + ln.sub;
        if (vl < n && ln.valid) {
            const uint32_t v = static_cast<uint32_t>(vl);
            const int32_t b = row_ptr[v], e = row_ptr[v + 1];
            const size_t at = vl * kp + ln.col;
            const Vec<T, V> x = load<T, V>(p + at);
            const Vec<T, V> s =
                row_sum<T, V, kWeighted>(m, col_idx, wt, v, b, e, p, seg_sum, kp, ln.col);
            const T d = T(1) + a * (kWeighted ? static_cast<T>(wdeg[v]) : static_cast<T>(e - b));
            Vec<T, V> y;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                y.x[j] = d * x.x[j] - a * s.x[j];
                acc[j] += static_cast<double>(x.x[j]) * static_cast<double>(y.x[j]);
            }
            store<T, V>(q + at, y);
        }
    }
    block_column_sum<V>(acc, ln, k, partial, lds);
}

// Sets *flag when some value of x is not zero (NaN included).
__global__ __launch_bounds__(kThreads) void nonzero_kernel(const double *__restrict__ x,
                                                           size_t count, unsigned int *flag) {
    bool found = false;
    const size_t step = static_cast<size_t>(gridDim.x) * kThreads;
    size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    for (; i + 3 * step < count && !found; i += 4 * step) {
        const double a = x[i], b = x[i + step], c = x[i + 2 * step], d = x[i + 3 * step];
        found = !(a == 0.0 && b == 0.0 && c == 0.0 && d == 0.0);
    }
    for (; i < count && !found; i += step) found = !(x[i] == 0.0);
    if (__ballot(found) && (threadIdx.x & 63u) == 0) *flag = 1u;
}

// R = B - A X in binary64; partial sums of R_j . R_j (and of B_j . B_j).  With
// gather false (X is zero) R = B and X is not read.
template <int V, bool kWeighted>
__global__ __launch_bounds__(kThreads) void residual_kernel(
    CgRows m, const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
    const double *__restrict__ wt, const double *__restrict__ wdeg, uint32_t n, uint32_t k,
    double alpha, const double *__restrict__ B, const double *__restrict__ X,
    const double *__restrict__ seg_sum, double *__restrict__ R, bool gather,
    double *__restrict__ partial_rr, double *__restrict__ partial_bb) {
    __shared__ double lds[kWaves][64];
    const Lane ln = lane_map(k, V);
    const uint32_t rows = 64u / ln.group;
    uint32_t g0, gs;
    row_range(&g0, &gs);
    double rr[V] = {}, bb[V] = {};
    for (uint32_t g = g0; static_cast<size_t>(g) * rows < n; g += gs) {
        const size_t vl = static_cast<size_t>(g) * rows + ln.sub;
        if (vl < n && ln.valid) {
            const uint32_t v = static_cast<uint32_t>(vl);
            const size_t at = vl * k + ln.col;
            const Vec<double, V> rhs = load<double, V>(B + at);
            Vec<double, V> r = rhs;
            if (gather) {
                const int32_t b = row_ptr[v], e = row_ptr[v + 1];
                const Vec<double, V> x = load<double, V>(X + at);
                const Vec<double, V> s = row_sum<double, V, kWeighted>(m, col_idx, wt, v, b, e, X,
                                                                       seg_sum, k, ln.col);
                const double d = 1.0 + alpha * (kWeighted ? wdeg[v] : static_cast<double>(e - b));
#pragma unroll
                for (int j = 0; j < V; ++j) r.x[j] = rhs.x[j] - (d * x.x[j] - alpha * s.x[j]);
            }
            store<double, V>(R + at, r);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                rr[j] += r.x[j] * r.x[j];
                bb[j] += rhs.x[j] * rhs.x[j];
            }
        }
    }
    block_column_sum<V>(rr, ln, k, partial_rr, lds);
    if (partial_bb) block_column_sum<V>(bb, ln, k, partial_bb, lds);
}

// Sum of one column's partials in a fixed order, the same in every thread.
__device__ __forceinline__ double column_total(const double *__restrict__ partial, uint32_t blocks,
                                               double *lds) {
    double a = 0.0;
    for (uint32_t b = threadIdx.x; b < blocks; b += kThreads) a += partial[b];
    for (uint32_t off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
    if ((threadIdx.x & 63u) == 0) lds[threadIdx.x >> 6] = a;
    __syncthreads();
    double t = 0.0;
    for (uint32_t w = 0; w < kWaves; ++w) t += lds[w];
    __syncthreads();
    return t;
}

// out[j] = the total of column j (one block per column).
__global__ __launch_bounds__(kThreads) void column_sum_kernel(const double *__restrict__ partial,
                                                              uint32_t blocks,
                                                              double *__restrict__ out) {
    __shared__ double lds[kWaves];
    const double t = column_total(partial + static_cast<size_t>(blockIdx.x) * blocks, blocks, lds);
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

// The dot products of column blockIdx.x and, from them, its CG scalars:
//   mode 0 (after start):  rz = r.z; active = rz > 0 and r.r > tol2
//   mode 1 (after A p):    step = active ? rz / p.q : 0 (column 0 counts the iteration)
//   mode 2 (after update): beta = active ? r.z / rz : 0; rz = r.z; active &= r.r > tol2
__global__ __launch_bounds__(kThreads) void scalars_kernel(int mode, uint32_t k,
                                                           const double *__restrict__ pa,
                                                           const double *__restrict__ pb,
                                                           uint32_t blocks, double *S) {
    __shared__ double lds[kWaves];
    const uint32_t j = blockIdx.x;
    if (mode == 1 && j == 0 && any_of(S + kActive, k) && threadIdx.x == 0) S[kIters] += 1.0;
    if (mode != 0 && S[kActive + j] == 0.0) {  // nothing moves in this column any more
        if (threadIdx.x == 0) S[(mode == 1 ? kStep : kBeta) + j] = 0.0;
        return;
    }
    const double a = column_total(pa + static_cast<size_t>(j) * blocks, blocks, lds);
    const double b = mode == 1 ? 0.0 : column_total(pb + static_cast<size_t>(j) * blocks, blocks, lds);
    if (threadIdx.x != 0) return;
    const double rz = S[kRz + j];
    if (mode == 0) {
        if (j == 0) S[kIters] = 0.0;
        S[kRz + j] = a;
        S[kActive + j] = (a > 0.0 && b > S[kTol2 + j]) ? 1.0 : 0.0;
    } else if (mode == 1) {
        S[kStep + j] = a > 0.0 ? rz / a : 0.0;
    } else {
        S[kBeta + j] = rz > 0.0 ? a / rz : 0.0;
        S[kRz + j] = a;
        if (!(b > S[kTol2 + j])) S[kActive + j] = 0.0;
    }
}

// Jacobi preconditioner of every row in the inner precision.
template <typename T>
__global__ __launch_bounds__(kThreads) void minv_kernel(const int32_t *__restrict__ row_ptr,
                                                        const double *__restrict__ wdeg, uint32_t n,
                                                        double alpha, T *__restrict__ minv) {
    const uint32_t v = blockIdx.x * kThreads + threadIdx.x;
    if (v >= n) return;
    const double d = wdeg ? wdeg[v] : static_cast<double>(row_ptr[v + 1] - row_ptr[v]);
    minv[v] = static_cast<T>(1.0 / (1.0 + alpha * d));
}

// Inner CG start on the scaled residual: r = R64 / scale_j (as T; zero in the
// padding), d = 0, p = Minv r; partial sums of r.z and r.r.
template <typename T>
__global__ __launch_bounds__(kThreads) void start_kernel(
    uint32_t n, uint32_t k, uint32_t kp, const T *__restrict__ minv,
    const double *__restrict__ R64, const double *__restrict__ scale, T *__restrict__ r,
    T *__restrict__ p, T *__restrict__ d, double *__restrict__ partial,
    double *__restrict__ partial_rr) {
    __shared__ double lds[kWaves][64];
    const Lane ln = lane_map(kp, 1);
    const uint32_t rows = 64u / ln.group;
    uint32_t g0, gs;
    row_range(&g0, &gs);
    const double sc = ln.col < k ? scale[ln.col] : 0.0;
    double acc[1] = {}, rr[1] = {};
    for (uint32_t g = g0; static_cast<size_t>(g) * rows < n; g += gs) {
        const size_t v = static_cast<size_t>(g) * rows + ln.sub;
        if (v < n && ln.valid) {
            const T rv = static_cast<T>(sc > 0.0 ? R64[v * k + ln.col] / sc : 0.0);
            const T zv = minv[v] * rv;
            const size_t at = v * kp + ln.col;
            r[at] = rv;
            p[at] = zv;
            d[at] = T(0);
            acc[0] += static_cast<double>(rv) * static_cast<double>(zv);
            rr[0] += static_cast<double>(rv) * static_cast<double>(rv);
        }
    }
    block_column_sum<1>(acc, ln, k, partial, lds);
    block_column_sum<1>(rr, ln, k, partial_rr, lds);
}

// r -= step_j q; partial sums of r.z (z = Minv r) and r.r.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void update_kernel(
    uint32_t n, uint32_t k, uint32_t kp, const T *__restrict__ minv, const T *__restrict__ q,
    T *__restrict__ r, double *__restrict__ partial_rz, double *__restrict__ partial_rr,
    const double *__restrict__ S) {
    if (!any_of(S + kActive, k)) return;
    __shared__ double lds[kWaves][64];
    const Lane ln = lane_map(kp, V);
    const uint32_t rows = 64u / ln.group;
    uint32_t g0, gs;
    row_range(&g0, &gs);
    T a[V];
#pragma unroll
    for (int j = 0; j < V; ++j)
        a[j] = ln.col + j < k ? static_cast<T>(S[kStep + ln.col + j]) : T(0);
    double rz[V] = {}, rr[V] = {};
    for (uint32_t g = g0; static_cast<size_t>(g) * rows < n; g += gs) {
        const size_t v = static_cast<size_t>(g) * rows + ln.sub;
        if (v < n && ln.valid) {
            const size_t at = v * kp + ln.col;
            const Vec<T, V> qv = load<T, V>(q + at);
            Vec<T, V> rv = load<T, V>(r + at);
            const T mv = minv[v];
#pragma unroll
            for (int j = 0; j < V; ++j) {
                rv.x[j] = rv.x[j] - a[j] * qv.x[j];
                const T zv = mv * rv.x[j];
                rz[j] += static_cast<double>(rv.x[j]) * static_cast<double>(zv);
                rr[j] += static_cast<double>(rv.x[j]) * static_cast<double>(rv.x[j]);
            }
            store<T, V>(r + at, rv);
        }
    }
    block_column_sum<V>(rz, ln, k, partial_rz, lds);
    block_column_sum<V>(rr, ln, k, partial_rr, lds);
}

// d += step_j p; p = Minv r + beta_j p.  A column that this iteration has just
// finished still owes d its step.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void direction_kernel(
    uint32_t n, uint32_t k, uint32_t kp, const T *__restrict__ minv, const T *__restrict__ r,
    T *__restrict__ p, T *__restrict__ d, const double *__restrict__ S) {
    if (!any_of(S + kStep, k) && !any_of(S + kActive, k)) return;
    const Lane ln = lane_map(kp, V);
    const uint32_t rows = 64u / ln.group;
    uint32_t g0, gs;
    row_range(&g0, &gs);
    T a[V], b[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        a[j] = ln.col + j < k ? static_cast<T>(S[kStep + ln.col + j]) : T(0);
        b[j] = ln.col + j < k ? static_cast<T>(S[kBeta + ln.col + j]) : T(0);
    }
    for (uint32_t g = g0; static_cast<size_t>(g) * rows < n; g += gs) {
        const size_t v = static_cast<size_t>(g) * rows + ln.sub;
        if (v < n && ln.valid) {
            const size_t at = v * kp + ln.col;
            const Vec<T, V> rv = load<T, V>(r + at);
            Vec<T, V> pv = load<T, V>(p + at), dv = load<T, V>(d + at);
            const T mv = minv[v];
#pragma unroll
            for (int j = 0; j < V; ++j) {
                dv.x[j] = dv.x[j] + a[j] * pv.x[j];
                pv.x[j] = mv * rv.x[j] + b[j] * pv.x[j];
            }
            store<T, V>(d + at, dv);
            store<T, V>(p + at, pv);
        }
    }
}

// X += scale_j * d (binary64 refinement update)
template <typename T>
__global__ __launch_bounds__(kThreads) void correct_kernel(uint32_t n, uint32_t k, uint32_t kp,
                                                           const double *__restrict__ scale,
                                                           const T *__restrict__ d,
                                                           double *__restrict__ X) {
    const Lane ln = lane_map(k, 1);
    const uint32_t rows = 64u / ln.group;
    uint32_t g0, gs;
    row_range(&g0, &gs);
    const double sc = ln.valid ? scale[ln.col] : 0.0;
    for (uint32_t g = g0; static_cast<size_t>(g) * rows < n; g += gs) {
        const size_t v = static_cast<size_t>(g) * rows + ln.sub;
        if (v < n && ln.valid) {
            const size_t i = v * k + ln.col;
            X[i] = X[i] + sc * static_cast<double>(d[v * kp + ln.col]);
        }
    }
}

// Blocks of kWaves waves that cover n rows of `cols` columns, V a lane.
inline unsigned int grid_for(uint32_t n, uint32_t cols, uint32_t V, uint32_t max_blocks) {
    uint32_t group = 1;
    while (group * V < cols) group <<= 1;
    const uint32_t rows = 64u / group;
    size_t blocks = (static_cast<size_t>(n) + rows * kWaves - 1) / (rows * kWaves);
    if (blocks > max_blocks) blocks = max_blocks;
    if (blocks < 1) blocks = 1;
    return static_cast<unsigned int>(blocks);
}

template <typename T, int V, bool kWeighted>
hipError_t inner(const CgWork &w, uint32_t max_iters, uint32_t poll, uint32_t *iters,
                 hipStream_t stream) {
    const uint32_t n = w.n, k = w.k, kp = w.kp;
    const unsigned int blocks = grid_for(n, kp, V, w.max_blocks);
    const unsigned int blocks1 = grid_for(n, kp, 1, w.max_blocks);
    T *r = static_cast<T *>(w.r), *p = static_cast<T *>(w.p), *q = static_cast<T *>(w.q),
      *d = static_cast<T *>(w.d), *minv = static_cast<T *>(w.minv),
      *seg_sum = static_cast<T *>(w.seg_sum);
    double *S = w.scalars;
    hipError_t e;
    start_kernel<T><<<blocks1, kThreads, 0, stream>>>(n, k, kp, minv, w.R64, w.scale, r, p, d,
                                                      w.partial_a, w.partial_b);
    scalars_kernel<<<k, kThreads, 0, stream>>>(0, k, w.partial_a, w.partial_b, blocks1, S);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    uint32_t it = 0;
    double state[kIters + 1 - kActive];  // activity of the columns, iterations done
    while (it < max_iters) {
        if (w.segments)
            segment_sum_kernel<T, V, kWeighted>
                <<<w.segments < w.max_blocks ? w.segments : w.max_blocks, kThreads, 0, stream>>>(
                    w.col_idx, w.weights, w.rows.seg, w.rows.count, kp, k, p, kp, seg_sum,
                    S + kActive);
        apply_kernel<T, V, kWeighted><<<blocks, kThreads, 0, stream>>>(
            w.rows, w.row_ptr, w.col_idx, w.weights, w.wdeg, n, k, kp, w.alpha, p, seg_sum, q,
            w.partial_a, S);
        scalars_kernel<<<k, kThreads, 0, stream>>>(1, k, w.partial_a, nullptr, blocks, S);
        update_kernel<T, V><<<blocks, kThreads, 0, stream>>>(n, k, kp, minv, q, r, w.partial_a,
                                                             w.partial_b, S);
        scalars_kernel<<<k, kThreads, 0, stream>>>(2, k, w.partial_a, w.partial_b, blocks, S);
        direction_kernel<T, V><<<blocks, kThreads, 0, stream>>>(n, k, kp, minv, r, p, d, S);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        ++it;
        if (it % poll == 0 || it == max_iters) {
            if ((e = hipMemcpyAsync(state, S + kActive, sizeof(state), hipMemcpyDeviceToHost,
                                    stream)) != hipSuccess)
                return e;
            if ((e = hipStreamSynchronize(stream)) != hipSuccess) return e;
            bool any = false;
            for (uint32_t j = 0; j < k; ++j) any = any || state[j] != 0.0;
            if (!any) break;
        }
    }
    correct_kernel<T><<<grid_for(n, k, 1, w.max_blocks), kThreads, 0, stream>>>(n, k, kp, w.scale,
                                                                                d, w.X);
    *iters = it ? static_cast<uint32_t>(state[kIters - kActive]) : 0u;
    return hipGetLastError();
}

template <int V>
void residual(const CgWork &w, bool with_b, bool gather, unsigned int blocks, hipStream_t stream) {
    double *seg_sum = static_cast<double *>(w.seg_sum);
    const uint32_t segs = w.segments < w.max_blocks ? w.segments : w.max_blocks;
    auto go = [&](auto weighted) {
        constexpr bool kW = decltype(weighted)::value;
        if (segs && gather)
            segment_sum_kernel<double, V, kW><<<segs, kThreads, 0, stream>>>(
                w.col_idx, w.weights, w.rows.seg, w.rows.count, w.k, w.k, w.X, w.k, seg_sum,
                nullptr);
        residual_kernel<V, kW><<<blocks, kThreads, 0, stream>>>(
            w.rows, w.row_ptr, w.col_idx, w.weights, w.wdeg, w.n, w.k, w.alpha, w.B, w.X, seg_sum,
            w.R64, gather, w.partial_a, with_b ? w.partial_b : nullptr);
    };
    if (w.weights) go(std::true_type{});
    else go(std::false_type{});
}

}  // namespace

uint32_t cg_padded(uint32_t k, bool fp32) {
    const uint32_t widest = fp32 ? 4u : 2u;  // 16 bytes
    uint32_t V = 1;
    while (V < widest && V < k) V <<= 1;
    return (k + V - 1u) / V * V;
}

template <typename T>
hipError_t cg_inner(const CgWork &w, uint32_t max_iters, uint32_t poll, uint32_t *iters,
                    hipStream_t stream) {
    auto go = [&](auto V) {
        constexpr int kV = decltype(V)::value;
        return w.weights ? inner<T, kV, true>(w, max_iters, poll, iters, stream)
                         : inner<T, kV, false>(w, max_iters, poll, iters, stream);
    };
    if constexpr (sizeof(T) == 4)
        if (w.kp % 4u == 0) return go(std::integral_constant<int, 4>{});
    if (w.kp % 2u == 0) return go(std::integral_constant<int, 2>{});
    return go(std::integral_constant<int, 1>{});
}

template hipError_t cg_inner<float>(const CgWork &, uint32_t, uint32_t, uint32_t *, hipStream_t);
template hipError_t cg_inner<double>(const CgWork &, uint32_t, uint32_t, uint32_t *, hipStream_t);

hipError_t cg_prepare(const CgWork &w, bool fp32, hipStream_t stream) {
    const uint32_t blocks = (w.n + kThreads - 1u) / kThreads;
    segments_kernel<<<blocks, kThreads, 0, stream>>>(w.row_ptr, w.n, w.rows.seg_base, w.rows.seg,
                                                     w.rows.count);
    if (fp32)
        minv_kernel<float><<<blocks, kThreads, 0, stream>>>(w.row_ptr, w.wdeg, w.n, w.alpha,
                                                            static_cast<float *>(w.minv));
    else
        minv_kernel<double><<<blocks, kThreads, 0, stream>>>(w.row_ptr, w.wdeg, w.n, w.alpha,
                                                             static_cast<double *>(w.minv));
    const size_t nk = static_cast<size_t>(w.n) * w.k;
    const size_t nz = (nk + 4u * kThreads - 1u) / (4u * kThreads);
    nonzero_kernel<<<static_cast<unsigned int>(nz < w.max_blocks ? nz : w.max_blocks), kThreads, 0,
                     stream>>>(w.X, nk, w.nonzero);
    return hipGetLastError();
}

hipError_t cg_residual(const CgWork &w, bool with_b, bool gather, hipStream_t stream) {
    // two columns a lane where every row of B, X and R starts on 16 bytes
    const bool pairs = w.k % 2u == 0 && reinterpret_cast<uintptr_t>(w.B) % 16u == 0 &&
                       reinterpret_cast<uintptr_t>(w.X) % 16u == 0;
    const unsigned int blocks = grid_for(w.n, w.k, pairs ? 2 : 1, w.max_blocks);
    if (pairs) residual<2>(w, with_b, gather, blocks, stream);
    else residual<1>(w, with_b, gather, blocks, stream);
    column_sum_kernel<<<w.k, kThreads, 0, stream>>>(w.partial_a, blocks, w.res_rr);
    if (with_b) column_sum_kernel<<<w.k, kThreads, 0, stream>>>(w.partial_b, blocks, w.res_bb);
    return hipGetLastError();
}

}  // namespace fc
