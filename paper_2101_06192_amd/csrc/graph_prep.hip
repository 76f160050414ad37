// CSR validation and the per-vertex records of the augmented graph G*.
//
// G* (Section 4.1 of the paper) is never materialised: u* is the id n, the
// edges {u*, v} are implicit, and a walk leaves v to u* with probability
// 1 / (1 + alpha d_v) (edge weight 1 against d_v edges of weight alpha).
#include "fc_kernels.hpp"
#include "fc_rows.hpp"

#pragma clang fp contract(off)

namespace fc {

namespace {

// Whether row offset v (of n + 1) is wrong.
__device__ __forceinline__ bool bad_offset(const int32_t *__restrict__ row_ptr, int64_t v, int32_t n,
                                           int64_t nnz) {
    const int64_t a = row_ptr[v];
    bool bad = a < 0 || a > nnz;
    if (v == 0) bad |= (a != 0);
    if (v == n) bad |= (a != nnz);
    if (v < n) bad |= (row_ptr[v + 1] < a);
    return bad;
}

__global__ void validate_rows_kernel(const int32_t *__restrict__ row_ptr, int32_t n, int64_t nnz,
                                     unsigned int *err) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v > n) return;
    if (bad_offset(row_ptr, v, n, nnz)) atomicOr(err, kErrGraphRowPtr);
}

// Column checks, one CSR entry per lane and step (entries of a wave are
// consecutive, so col_idx is read coalesced).  Every entry is checked for
// range, self-loop and strict order against the previous entry of its row.
//
// Symmetry needs only half of the binary searches: order the vertices by
// (degree, id) and call an entry (v, u) downward when u is below v.  Rows that
// are strictly ascending hold no entry twice, so reversing entries maps the
// downward entries one to one into the upward ones as soon as each of them has
// its reverse entry; with as many downward as upward entries the map is onto,
// and then every upward entry has its reverse too.  So only downward entries
// search, always in the shorter of the two rows (a hub's row is never
// searched), and the difference of the two counts is added to sym_diff.
//
// Bound by the random lines of row_ptr[u] and u's row: R-MAT with 2^22
// vertices, 65 M entries: 9.70 ms (16 entries per thread, every entry
// searched) before, 2.99 ms now; 10 K entries of a small graph: 26 us
// (a chain of 16 searches per thread) before, 5.0 us now.
// Wide blocks of several steps: each block ends in one atomic on sym_diff, and
// 7800 of them on that one word took 94 us (2 M entries: 106 us a call, now
// 76); more blocks than fit at once, so that the ones with hub rows, which
// search for nearly every entry, even out.
constexpr uint32_t kColThreads = 512, kColBlocks = 1024;

// kFollow: the row offsets are known to be right.  Otherwise they are cut to the
// entries before they are followed, and what is found in a graph whose offsets are
// wrong means nothing.
template <bool kFollow>
__device__ __forceinline__ void check_columns(
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
    const double *__restrict__ weights, int32_t n, int64_t nnz, uint32_t steps, unsigned int *err,
    unsigned long long *sym_diff) {
    __shared__ long long s_diff;
    if (threadIdx.x == 0) s_diff = 0;
    __syncthreads();
    RowFinder rows;
    unsigned int e = 0;
    long long diff = 0;  // downward minus upward entries (wave-uniform)
    const int64_t first =
        (static_cast<int64_t>(blockIdx.x) * (kColThreads / 64u) + (threadIdx.x >> 6)) * 64 * steps;
    for (uint32_t t = 0; t < steps; ++t) {
        const int64_t j0 = first + static_cast<int64_t>(t) * 64;
        if (j0 >= nnz) break;
        const int64_t j = j0 + (threadIdx.x & 63u);
        const bool live = j < nnz;
        int32_t v = 0, vb = 0, ve = 0;
        rows.find(row_ptr, n, j0, nnz, &v, &vb, &ve);
        bool down = false, up = false;
        if (live) {
            const int32_t u = col_idx[j];
            if (u < 0 || u >= n) {
                e |= kErrGraphColumn;
            } else {
                if (u == v) e |= kErrGraphSelfLoop;
                if (j > vb && j > 0 && col_idx[j - 1] >= u) e |= kErrGraphOrder;
                int32_t a = row_ptr[u];
                int32_t end = row_ptr[u + 1];
                if (!kFollow) {
                    const int32_t most = static_cast<int32_t>(nnz);
                    a = a < 0 ? 0 : a > most ? most : a;
                    end = end < a ? a : end > most ? most : end;
                }
                const int32_t du = end - a;
                const int32_t dv = static_cast<int32_t>(static_cast<uint32_t>(ve) - static_cast<uint32_t>(vb));
                down = du < dv || (du == dv && u < v);
                up = !down && u != v;
                double w = 0.0;
                if (weights) {  // 0 or in [2^-64, 2^64] (NaN fails both)
                    w = weights[j];
                    if (!(w == 0.0 || (w >= 0x1p-64 && w <= 0x1p64))) e |= kErrGraphWeight;
                }
                if (down) {
                    int32_t b = end;
                    while (a < b) {
                        const int32_t mid = a + ((b - a) >> 1);
                        if (col_idx[mid] < v) a = mid + 1;
                        else b = mid;
                    }
                    if (a >= end || col_idx[a] != v) e |= kErrGraphAsymmetric;
                    else if (weights && !(weights[a] == w)) e |= kErrGraphWeightAsym;
                }
            }
        }
        diff += __popcll(__ballot(down));
        diff -= __popcll(__ballot(up));
    }
    if (e) atomicOr(err, e);
    if ((threadIdx.x & 63u) == 0 && diff)
        atomicAdd(reinterpret_cast<unsigned long long *>(&s_diff),
                  static_cast<unsigned long long>(diff));
    __syncthreads();
    if (threadIdx.x == 0 && s_diff)
        atomicAdd(sym_diff, static_cast<unsigned long long>(s_diff));
}

__global__ __launch_bounds__(kColThreads) void validate_cols_kernel(
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
    const double *__restrict__ weights, int32_t n, int64_t nnz, uint32_t steps, unsigned int *err,
    unsigned long long *sym_diff) {
    if (*err & kErrGraphRowPtr) return;  // row offsets that may not be followed
    check_columns<true>(row_ptr, col_idx, weights, n, nnz, steps, err, sym_diff);
}

// kColChunk consecutive entries per thread (step thresholds).
constexpr int64_t kColChunk = 16;

// thr(d) = floor(2^32 * (1 / ((alpha * d) + 1))), each operation rounded to
// binary64 (IEEE division; no contraction in this file).
// The weighted threshold is the same expression in the weighted degree W
// (an integer d is exact in binary64, so W = d gives thr(d)).
__device__ __forceinline__ unsigned long long root_threshold_w(double alpha, double W) {
    if (W == 0.0) return 1ull << 32;
    const double aw = alpha * W;
    const double den = aw + 1.0;
    const double p = 1.0 / den;
    return static_cast<unsigned long long>(p * 4294967296.0);
}
__device__ __forceinline__ unsigned long long root_threshold(double alpha, uint32_t d) {
    return root_threshold_w(alpha, static_cast<double>(d));
}

// One thread per row; the sum is sequential by definition (its rounding is
// part of the randomness contract), so rows are not split.
__global__ void row_wsum_kernel(const int32_t *__restrict__ row_ptr,
                                const double *__restrict__ weights, int32_t n,
                                double *__restrict__ S) {
    const int32_t v = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    if (v >= n) return;
    const int32_t b = row_ptr[v], e = row_ptr[v + 1];
    double s = 0.0;
#pragma unroll 8
    for (int32_t q = b; q < e; ++q) {
        s += weights[q];
        S[q] = s;
    }
}

// Step thresholds: entry-parallel like the column check (kColChunk entries
// per thread, the row of the first found by binary search over row_ptr).
__global__ void step_thr_kernel(const int32_t *__restrict__ row_ptr, const double *__restrict__ S,
                                int32_t n, int64_t nnz, uint32_t *__restrict__ T) {
    const int64_t e0 = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) * kColChunk;
    if (e0 >= nnz) return;
    const int64_t e1 = e0 + kColChunk < nnz ? e0 + kColChunk : nnz;
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo + 1) >> 1);
        if (row_ptr[mid] <= e0) lo = mid;
        else hi = mid - 1;
    }
    int32_t v = lo;
    int64_t row_end = row_ptr[v + 1];
    for (int64_t j = e0; j < e1; ++j) {
        while (j >= row_end) {
            ++v;
            row_end = row_ptr[v + 1];
        }
        const double W = S[row_end - 1], s = S[j];
        // smallest x in [0, 2^32] with (x * W) * 2^-32 >= s (x = 2^32 gives W >= s)
        uint64_t a = 0, b = 1ull << 32;
        while (a < b) {
            const uint64_t mid = (a + b) >> 1;
            if ((static_cast<double>(mid) * W) * 0x1p-32 >= s) b = mid;
            else a = mid + 1;
        }
        T[j] = static_cast<uint32_t>(a < 1 ? 1 : a > 0xFFFFFFFFull ? 0xFFFFFFFFull : a);
    }
}

__global__ void row_wdeg_kernel(const int32_t *__restrict__ row_ptr,
                                const double *__restrict__ weights, int32_t n,
                                double *__restrict__ W) {
    const int32_t v = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    if (v >= n) return;
    const int32_t b = row_ptr[v], e = row_ptr[v + 1];
    double s = 0.0;
#pragma unroll 8
    for (int32_t q = b; q < e; ++q) s += weights[q];
    W[v] = s;
}

// One pass over the rows: 8 bytes read and 16 written per vertex.  The maximum
// degree and the weighted volume are reduced per block (kVrecBlocks blocks at
// most, each walking the vertices in strides) before they touch their one
// global word: with an atomic per wave, 15.6 K atomics on one address took
// 182 us of a pass that streams 24 MB (10^6 vertices); now 10 us.
constexpr uint32_t kVrecThreads = 1024, kVrecBlocks = 256;

__global__ __launch_bounds__(kVrecThreads) void build_vrec_kernel(
    const int32_t *__restrict__ row_ptr, const double *__restrict__ S, int32_t n, double alpha,
    VRec *__restrict__ vrec, unsigned int *dmax, uint32_t *__restrict__ iso, double *wtotal,
    uint32_t *__restrict__ zero) {
    __shared__ uint32_t s_max[kVrecThreads / 64u];
    __shared__ double s_sum[kVrecThreads / 64u];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t m = 0;
    double sw = 0.0;
    // whole blocks of vertices per step, so that ballots cover 64 consecutive ids
    for (int64_t v0 = static_cast<int64_t>(blockIdx.x) * kVrecThreads; v0 < n;
         v0 += static_cast<int64_t>(gridDim.x) * kVrecThreads) {
        const int64_t vl = v0 + threadIdx.x;
        const int32_t v = static_cast<int32_t>(vl);
        const bool live = vl < n;
        uint32_t d = 0;
        int32_t a = 0;
        if (live) {
            a = row_ptr[v];
            d = static_cast<uint32_t>(row_ptr[v + 1] - a);
        }
        m = max(m, d);
        if (iso) {  // 64 vertices per wave: two bitmap words
            const uint64_t bits = __ballot(live && d == 0);
            const int64_t w0 = (vl - lane) >> 5, nw = (static_cast<int64_t>(n) + 31) >> 5;
            if (lane == 0 && w0 < nw) iso[w0] = static_cast<uint32_t>(bits);
            if (lane == 32 && w0 + 1 < nw) iso[w0 + 1] = static_cast<uint32_t>(bits >> 32);
        }
        const double W = S && d ? S[a + static_cast<int32_t>(d) - 1] : 0.0;
        sw += W;
        if (!live) continue;
        if (zero) zero[v] = 0u;
        const unsigned long long t = S ? root_threshold_w(alpha, W) : root_threshold(alpha, d);
        VRec r;
        r.start = a;
        r.deg = d;
        r.thr = static_cast<uint32_t>(t);
        r.always_root = (t >> 32) ? 1u : 0u;
        vrec[v] = r;
    }
    for (int off = 32; off > 0; off >>= 1) {
        m = max(m, static_cast<uint32_t>(__shfl_down(m, off, 64)));
        sw += __shfl_down(sw, off, 64);
    }
    if (lane == 0) {
        s_max[wave] = m;
        s_sum[wave] = sw;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (uint32_t w = 1; w < kVrecThreads / 64u; ++w) {
        m = max(m, s_max[w]);
        sw += s_sum[w];
    }
    if (m) atomicMax(dmax, m);
    // sum of the weighted degrees (bounds the expected walk length)
    if (S && wtotal && sw > 0.0) atomicAdd(wtotal, sw);
}

// The checks and the records of a small graph without weights in one launch: each
// block takes kColThreads row offsets and vertices, and its share of the entries.
// Between launches this small a call waits longer than it computes: with three
// kernels a farness call on 1000 vertices, 10 K entries and 576 trees took 123 us,
// with this one 97.  zero may be cleared before the checks are over, so it is no
// output of the call.
__global__ __launch_bounds__(kColThreads) void prepare_small_kernel(
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx, int32_t n, int64_t nnz,
    uint32_t steps, double alpha, VRec *__restrict__ vrec, GraphCheck *check,
    uint32_t *__restrict__ zero) {
    const int64_t v = static_cast<int64_t>(blockIdx.x) * kColThreads + threadIdx.x;
    if (v <= n && bad_offset(row_ptr, v, n, nnz)) atomicOr(&check->err, kErrGraphRowPtr);
    if (v < n) {
        const int32_t a = row_ptr[v];
        const uint32_t d = static_cast<uint32_t>(row_ptr[v + 1]) - static_cast<uint32_t>(a);
        const unsigned long long t = root_threshold(alpha, d);
        vrec[v] = {a, d, static_cast<uint32_t>(t), (t >> 32) ? 1u : 0u};
        if (zero) zero[v] = 0u;
    }
    if (nnz) check_columns<false>(row_ptr, col_idx, nullptr, n, nnz, steps, &check->err, &check->sym_diff);
}

__global__ void thresholds_kernel(double alpha, int32_t d_max, unsigned long long *out) {
    const int32_t d = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    if (d > d_max) return;
    out[d] = root_threshold(alpha, static_cast<uint32_t>(d));
}

inline unsigned int blocks_for(int64_t items, int threads) {
    return static_cast<unsigned int>((items + threads - 1) / threads);
}

}  // namespace

hipError_t launch_validate_rows(const int32_t *row_ptr, int32_t n, int64_t nnz,
                                unsigned int *err, hipStream_t stream) {
    validate_rows_kernel<<<blocks_for(static_cast<int64_t>(n) + 1, 256), 256, 0, stream>>>(
        row_ptr, n, nnz, err);
    return hipGetLastError();
}

// Up to 8 steps per wave once there are kColBlocks blocks.
static uint32_t column_steps(int64_t nnz) {
    const int64_t want = nnz / (static_cast<int64_t>(kColThreads) * kColBlocks);
    return static_cast<uint32_t>(want < 1 ? 1 : want > 8 ? 8 : want);
}

hipError_t launch_prepare_small(const int32_t *row_ptr, const int32_t *col_idx, int32_t n, int64_t nnz,
                                double alpha, VRec *vrec, GraphCheck *check, uint32_t *zero,
                                hipStream_t stream) {
    const uint32_t steps = column_steps(nnz);
    const unsigned int rows = blocks_for(static_cast<int64_t>(n) + 1, kColThreads);
    const unsigned int cols = blocks_for(nnz, static_cast<int>(kColThreads * steps));
    prepare_small_kernel<<<rows > cols ? rows : cols, kColThreads, 0, stream>>>(
        row_ptr, col_idx, n, nnz, steps, alpha, vrec, check, zero);
    return hipGetLastError();
}

hipError_t launch_validate_cols(const int32_t *row_ptr, const int32_t *col_idx,
                                const double *weights, int32_t n, int64_t nnz, unsigned int *err,
                                unsigned long long *sym_diff, hipStream_t stream) {
    if (n == 0 || nnz == 0) return hipSuccess;
    const uint32_t steps = column_steps(nnz);
    validate_cols_kernel<<<blocks_for(nnz, static_cast<int>(kColThreads * steps)), kColThreads, 0,
                           stream>>>(row_ptr, col_idx, weights, n, nnz, steps, err, sym_diff);
    return hipGetLastError();
}

hipError_t launch_row_wsum(const int32_t *row_ptr, const double *weights, int32_t n, double *S,
                           hipStream_t stream) {
    if (n == 0) return hipSuccess;
    row_wsum_kernel<<<blocks_for(n, 256), 256, 0, stream>>>(row_ptr, weights, n, S);
    return hipGetLastError();
}

hipError_t launch_step_thresholds(const int32_t *row_ptr, const double *S, int32_t n,
                                  int64_t nnz, uint32_t *T, hipStream_t stream) {
    if (n == 0 || nnz == 0) return hipSuccess;
    step_thr_kernel<<<blocks_for((nnz + kColChunk - 1) / kColChunk, 256), 256, 0, stream>>>(
        row_ptr, S, n, nnz, T);
    return hipGetLastError();
}

hipError_t launch_row_wdeg(const int32_t *row_ptr, const double *weights, int32_t n, double *W,
                           hipStream_t stream) {
    if (n == 0) return hipSuccess;
    row_wdeg_kernel<<<blocks_for(n, 256), 256, 0, stream>>>(row_ptr, weights, n, W);
    return hipGetLastError();
}

hipError_t launch_build_vrec(const int32_t *row_ptr, const double *S, int32_t n, double alpha,
                             VRec *vrec, unsigned int *dmax, uint32_t *iso, double *wtotal,
                             uint32_t *zero, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const unsigned int blocks = blocks_for(n, kVrecThreads);
    build_vrec_kernel<<<blocks < kVrecBlocks ? blocks : kVrecBlocks, kVrecThreads, 0, stream>>>(
        row_ptr, S, n, alpha, vrec, dmax, iso, wtotal, zero);
    return hipGetLastError();
}

hipError_t launch_thresholds(double alpha, int32_t d_max, unsigned long long *out,
                             hipStream_t stream) {
    thresholds_kernel<<<blocks_for(static_cast<int64_t>(d_max) + 1, 256), 256, 0, stream>>>(
        alpha, d_max, out);
    return hipGetLastError();
}

}  // namespace fc
