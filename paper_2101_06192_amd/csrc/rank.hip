// Ranking output: the vertex ranking by a score vector (stable LSD radix
// sort of order-preserving 64-bit keys, vertex ids as values) and Kendall's
// tau-b between two score vectors (exact integer pair counts).
//
// The top vertices of the forest closeness ranking are those with the lowest
// Omega_vv (Eq. "eq-fdistu-tr": farness grows with Omega_vv); the paper ranks
// the vertices by the estimate and reports Kendall's rank correlation against
// the ground truth (Section 6, "Vertex Ranking").
//
// Everything of one call is enqueued without waiting for the device: which bytes
// of the keys differ at all (the others need no pass), whether a score was NaN
// and whether a vector has ties is left in a small record that the later
// kernels read, returning at once where there is nothing to do.  (The host reads
// the bytes when they are there, and enqueues no more passes of the others.)
//
// At these sizes (n = 1000 .. a few million) a pass is launches and dependent
// loads, not bytes: n = 200 000, per byte pass 40 us (histogram 6, one
// workgroup's serial scan 18, scatter 16 over 49 workgroups) before, 12.7 us now;
// ranking and tau-b together 1.67 ms before, 0.55 ms now.
#include "fc_rank_kernels.hpp"

namespace fc {

namespace {

constexpr uint32_t kRankThreads = 256;
constexpr uint32_t kRankWaves = kRankThreads / 64u;
// The kernels that end in an atomic on one word per block (12 ns each, one after
// the other): wide blocks, two per CU at most, striding.
constexpr uint32_t kWideThreads = 1024, kWideBlocks = 512;

// Order-preserving map of a binary64 to uint64 (-0 and +0 map alike): flip
// every bit of a negative number, set the sign bit of a positive one.
__device__ __forceinline__ uint64_t order_key(double x) {
    uint64_t u = __double_as_longlong(x == 0.0 ? 0.0 : x);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// A byte in which the keys differ takes a pass; the passes alternate between
// the two buffers, the first reading buffer 0.
__device__ __forceinline__ bool byte_active(unsigned long long vary, uint32_t p) {
    return ((vary >> (8u * p)) & 255u) != 0;
}
__device__ __forceinline__ uint32_t passes_below(unsigned long long vary, uint32_t p) {
    uint32_t c = 0;
    for (uint32_t q = 0; q < p; ++q) c += byte_active(vary, q) ? 1u : 0u;
    return c;
}

// Keys, values and what is known of them: the bits in which any key differs
// from the first one's, and whether a score is NaN.
__global__ __launch_bounds__(kWideThreads) void keys_kernel(const double *__restrict__ score,
                                                            uint32_t n, uint32_t descending,
                                                            uint64_t *__restrict__ key,
                                                            int32_t *__restrict__ val,
                                                            SortInfo *info) {
    __shared__ unsigned long long s_vary[kWideThreads / 64u];
    const uint64_t k0 = order_key(score[0]);
    unsigned long long vary = 0;
    bool bad = false;
    for (size_t i = static_cast<size_t>(blockIdx.x) * kWideThreads + threadIdx.x; i < n;
         i += static_cast<size_t>(gridDim.x) * kWideThreads) {
        const double x = score[i];
        bad |= x != x;
        const uint64_t k = order_key(x);
        vary |= k ^ k0;
        key[i] = descending ? ~k : k;
        val[i] = static_cast<int32_t>(i);
    }
    if (__ballot(bad) && (threadIdx.x & 63u) == 0) info->bad = 1u;
    for (int off = 32; off > 0; off >>= 1) vary |= __shfl_xor(vary, off, 64);
    if ((threadIdx.x & 63u) == 0) s_vary[threadIdx.x >> 6] = vary;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (uint32_t w = 1; w < kWideThreads / 64u; ++w) vary |= s_vary[w];
    if (vary) atomicOr(&info->vary, vary);
}

// A tile is kRankWaves x R x 64 keys, wave after wave: wave w holds R runs of
// 64 consecutive keys, so the stable order inside a tile is (wave, run, lane).
template <uint32_t R>
__device__ __forceinline__ size_t tile_first() {
    return (static_cast<size_t>(blockIdx.x) * kRankWaves + (threadIdx.x >> 6)) * (R * 64u) +
           (threadIdx.x & 63u);
}

// Digit counts of one tile: thist[d * ntiles + tile], and total[d] over the tiles.
template <uint32_t R>
__global__ __launch_bounds__(kRankThreads) void tile_hist_kernel(SortBufs b, uint32_t n, uint32_t p,
                                                                 uint32_t ntiles,
                                                                 const SortInfo *info,
                                                                 unsigned int *__restrict__ thist,
                                                                 unsigned int *total, unsigned int *tell,
                                                                 unsigned int number) {
    const unsigned long long vary = info->vary;
    if (tell && blockIdx.x == 0 && threadIdx.x == 0) {
        unsigned int bytes = number << 8;
        for (uint32_t q = 0; q < 8u; ++q) bytes |= byte_active(vary, q) ? 1u << q : 0u;
        __hip_atomic_store(tell, bytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (!byte_active(vary, p)) return;
    const uint64_t *key = b.key[passes_below(vary, p) & 1u];
    __shared__ unsigned int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const size_t base = tile_first<R>();
    uint64_t k[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) k[r] = base + r * 64u < n ? key[base + r * 64u] : 0ull;
#pragma unroll
    for (uint32_t r = 0; r < R; ++r)
        if (base + r * 64u < n) atomicAdd(&h[(k[r] >> (8u * p)) & 255u], 1u);
    __syncthreads();
    const unsigned int c = h[threadIdx.x];
    thist[static_cast<size_t>(threadIdx.x) * ntiles + blockIdx.x] = c;
    if (c) atomicAdd(&total[threadIdx.x], c);
}

// One wave per digit: its tile counts become the position of each tile's first
// key with that digit (the keys with a smaller digit, then the tiles before).
__global__ __launch_bounds__(64) void tile_scan_kernel(unsigned int *__restrict__ thist,
                                                       uint32_t ntiles, uint32_t p,
                                                       const SortInfo *info,
                                                       const unsigned int *__restrict__ total) {
    if (!byte_active(info->vary, p)) return;
    const uint32_t d = blockIdx.x, lane = threadIdx.x;
    unsigned int run = 0;
#pragma unroll
    for (uint32_t q = 0; q < 4u; ++q) run += q * 64u + lane < d ? total[q * 64u + lane] : 0u;
    for (int off = 32; off > 0; off >>= 1) run += __shfl_xor(run, off, 64);
    unsigned int *row = thist + static_cast<size_t>(d) * ntiles;
    for (uint32_t t0 = 0; t0 < ntiles; t0 += 256u) {  // four loads in flight
        unsigned int c[4];
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) {
            const uint32_t t = t0 + q * 64u + lane;
            c[q] = t < ntiles ? row[t] : 0u;
        }
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) {
            const uint32_t t = t0 + q * 64u + lane;
            unsigned int x = c[q];
            for (uint32_t off = 1; off < 64u; off <<= 1) {
                const unsigned int y = __shfl_up(x, off, 64);
                if (lane >= off) x += y;
            }
            if (t < ntiles) row[t] = run + x - c[q];
            run += __shfl(x, 63, 64);
        }
    }
}

// Stable scatter of one tile.  Each wave counts its own keys run by run (the
// keys of a run with the same digit found with eight ballots), without a
// barrier; then the waves' counts give every key its place.
template <uint32_t R>
__global__ __launch_bounds__(kRankThreads) void tile_scatter_kernel(
    SortBufs b, uint32_t n, uint32_t p, uint32_t ntiles, const SortInfo *info,
    const unsigned int *__restrict__ thist) {
    const unsigned long long vary = info->vary;
    if (!byte_active(vary, p)) return;
    const uint32_t src = passes_below(vary, p) & 1u;
    const uint64_t *key = b.key[src];
    const int32_t *val = b.val[src];
    uint64_t *okey = b.key[src ^ 1u];
    int32_t *oval = b.val[src ^ 1u];
    __shared__ unsigned int cnt[kRankWaves][256];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const unsigned int start = thist[static_cast<size_t>(tid) * ntiles + blockIdx.x];
#pragma unroll
    for (uint32_t w = 0; w < kRankWaves; ++w) cnt[w][tid] = 0;
    const size_t base = tile_first<R>();
    const uint64_t below = (1ull << lane) - 1ull;
    uint64_t k[R];
    int32_t v[R];
    uint32_t place[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const bool valid = base + r * 64u < n;
        k[r] = valid ? key[base + r * 64u] : 0ull;
        v[r] = valid ? val[base + r * 64u] : 0;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const bool valid = base + r * 64u < n;
        const uint32_t d = static_cast<uint32_t>((k[r] >> (8u * p)) & 255u);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
            const uint64_t m = __ballot((d >> q) & 1u);
            peers &= ((d >> q) & 1u) ? m : ~m;
        }
        const uint32_t before = static_cast<uint32_t>(__popcll(peers & below));
        const uint32_t seen = cnt[wave][d];
        place[r] = seen + before;
        __builtin_amdgcn_wave_barrier();  // every lane has read before the leaders write
        if (valid && before == 0) cnt[wave][d] = seen + static_cast<uint32_t>(__popcll(peers));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    unsigned int run = start;  // thread d: digit d's place in each wave
#pragma unroll
    for (uint32_t w = 0; w < kRankWaves; ++w) {
        const unsigned int c = cnt[w][tid];
        cnt[w][tid] = run;
        run += c;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        if (base + r * 64u >= n) continue;
        const uint32_t d = static_cast<uint32_t>((k[r] >> (8u * p)) & 255u);
        const uint32_t at = cnt[wave][d] + place[r];
        okey[at] = k[r];
        oval[at] = v[r];
    }
}

// The sorted values as order and their inverse as rank (nothing when a score
// was NaN).
__global__ __launch_bounds__(kRankThreads) void order_kernel(SortBufs b, uint32_t n,
                                                             const SortInfo *info,
                                                             int32_t *__restrict__ order,
                                                             int32_t *__restrict__ rank) {
    if (info->bad) return;
    const int32_t *val = b.val[passes_below(info->vary, 8u) & 1u];
    const uint32_t i = blockIdx.x * kRankThreads + threadIdx.x;
    if (i >= n) return;
    const int32_t v = val[i];
    if (order) order[i] = v;
    if (rank) rank[v] = static_cast<int32_t>(i);
}

// Adds the block's sum of x to *out (one atomic).
__device__ __forceinline__ void block_add_u64(unsigned long long x, unsigned long long *out) {
    __shared__ unsigned long long red[kWideThreads / 64];
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    if ((threadIdx.x & 63u) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (uint32_t w = 0; w < kWideThreads / 64; ++w) t += red[w];
        if (t) atomicAdd(out, t);
    }
}

// First position of the run of equal elements that ends at i (same(j): whether
// j < i is in it; the run is contiguous): doubling steps back, then halving.
template <typename F>
__device__ __forceinline__ uint32_t run_start(uint32_t i, F same) {
    uint32_t in = i, step = 1;  // in: known to be in the run
    while (step <= i && same(i - step)) {
        in = i - step;
        step <<= 1;
    }
    // the run starts in (i - step, in], or at 0 when i < step
    uint32_t lo = step <= i ? i - step + 1u : 0u;
    while (lo < in) {
        const uint32_t mid = lo + ((in - lo) >> 1);
        if (same(mid)) in = mid;
        else lo = mid + 1u;
    }
    return in;
}

// Min-rank of every key after the sort: the number of keys strictly below it
// (equal keys share it), scattered to the key's original index.  Also adds sum
// over positions of (i - min-rank) into *ties: a run of t equal keys
// contributes 0 + 1 + ... + (t - 1) = t(t - 1)/2, its tied pairs.
__global__ __launch_bounds__(kWideThreads) void min_rank_kernel(SortBufs b, uint32_t n,
                                                                const SortInfo *info,
                                                                uint32_t *__restrict__ out,
                                                                unsigned long long *__restrict__ ties) {
    const uint32_t src = passes_below(info->vary, 8u) & 1u;
    const uint64_t *key = b.key[src];
    const int32_t *val = b.val[src];
    unsigned long long t = 0;
    for (size_t l = static_cast<size_t>(blockIdx.x) * kWideThreads + threadIdx.x; l < n;
         l += static_cast<size_t>(gridDim.x) * kWideThreads) {
        const uint32_t i = static_cast<uint32_t>(l);
        const uint64_t k = key[i];
        const uint32_t lo = run_start(i, [&](uint32_t j) { return key[j] == k; });
        out[val[i]] = lo;
        t += i - lo;
    }
    block_add_u64(t, ties);
}

// The order whose strict inversions are the discordant pairs, from both
// vectors' ranks and the order of b (buffer of the sort just done):
//   b without ties: s = rank a in the order of b;
//   a without ties: s = rank b in the order of a (its ranks are the places);
//   else the stable sort of b's order by rank a (three passes for 2^24 values:
//   the order by b is there already), keys and values for it in buffer 0.
// pair->vary = 0 tells the later kernels that s is complete.
__global__ __launch_bounds__(kRankThreads) void pair_keys_kernel(
    SortBufs b, uint32_t n, const SortInfo *info_b, const uint32_t *__restrict__ ra,
    const uint32_t *__restrict__ rb, const unsigned long long *__restrict__ ties, SortInfo *pair,
    uint32_t *__restrict__ s) {
    const bool b_free = ties[1] == 0, a_free = ties[0] == 0;
    const int32_t *ids = b.val[passes_below(info_b->vary, 8u) & 1u];
    const uint32_t i = blockIdx.x * kRankThreads + threadIdx.x;
    if (i == 0 && !a_free && !b_free) {
        unsigned long long m = n - 1u;
        for (uint32_t q = 1; q < 64u; q <<= 1) m |= m >> q;
        pair->vary = m;
    }
    if (i >= n) return;
    if (b_free) {
        s[i] = ra[ids[i]];
    } else if (a_free) {
        s[ra[i]] = rb[i];
    } else {  // the thread that overwrites ids[i] has read it
        const int32_t id = ids[i];
        b.key[0][i] = ra[id];
        b.val[0][i] = id;
    }
}

// After the pair passes: s = rank b in the order of (a, b).
__global__ __launch_bounds__(kRankThreads) void pair_order_kernel(SortBufs b, uint32_t n,
                                                                  const SortInfo *pair,
                                                                  const uint32_t *__restrict__ rb,
                                                                  uint32_t *__restrict__ s) {
    const unsigned long long vary = pair->vary;
    if (!vary) return;
    const int32_t *val = b.val[passes_below(vary, 8u) & 1u];
    const uint32_t i = blockIdx.x * kRankThreads + threadIdx.x;
    if (i < n) s[i] = rb[val[i]];
}

// Pairs tied in both: runs of equal (rank a, rank b) in that order.
__global__ __launch_bounds__(kWideThreads) void joint_ties_kernel(SortBufs b, uint32_t n,
                                                                  const SortInfo *pair,
                                                                  const uint32_t *__restrict__ s,
                                                                  unsigned long long *__restrict__ ties) {
    const unsigned long long vary = pair->vary;
    if (!vary) return;
    const uint64_t *key = b.key[passes_below(vary, 8u) & 1u];
    unsigned long long t = 0;
    for (size_t l = static_cast<size_t>(blockIdx.x) * kWideThreads + threadIdx.x; l < n;
         l += static_cast<size_t>(gridDim.x) * kWideThreads) {
        const uint32_t i = static_cast<uint32_t>(l);
        const uint64_t k = key[i];
        const uint32_t x = s[i];
        t += i - run_start(i, [&](uint32_t j) { return key[j] == k && s[j] == x; });
    }
    block_add_u64(t, ties);
}

// Strict inversions (pairs p < q with s_p > s_q) by a bottom-up merge sort.
// An element finds its place by binary search in the sibling runs: after the
// elements of earlier runs that are not above it and those of later runs that
// are below it, so equal values keep their order; the elements of earlier runs
// above it are its inversions.
//
// The first ten levels: 1024 elements in LDS, one per thread.
__global__ __launch_bounds__(kWideThreads) void merge_tile_kernel(uint32_t *__restrict__ s, uint32_t n,
                                                                   unsigned long long *__restrict__ inv) {
    __shared__ uint32_t x[2][kWideThreads];
    const uint32_t t = threadIdx.x;
    unsigned long long c = 0;
    for (size_t first = static_cast<size_t>(blockIdx.x) * kWideThreads; first < n;
         first += static_cast<size_t>(gridDim.x) * kWideThreads) {
        const uint32_t m = static_cast<uint32_t>(min(static_cast<size_t>(kWideThreads), n - first));
        __syncthreads();
        if (t < m) x[0][t] = s[first + t];
        __syncthreads();
        uint32_t at = 0;
        for (uint32_t w = 1; w < m; w <<= 1, at ^= 1u) {
            const uint32_t *in = x[at];
            if (t < m) {
                const uint32_t l0 = t & ~(2u * w - 1u);
                const uint32_t r0 = min(l0 + w, m), r1 = min(l0 + 2u * w, m);
                const bool left = t < r0;
                const uint32_t y = in[t];
                uint32_t lo = left ? r0 : l0, hi = left ? r1 : r0;
                const uint32_t from = lo;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (left ? in[mid] < y : in[mid] <= y) lo = mid + 1u;
                    else hi = mid;
                }
                const uint32_t before = lo - from;
                x[at ^ 1u][l0 + (t - (left ? l0 : r0)) + before] = y;
                if (!left) c += r0 - lo;
            }
            __syncthreads();
        }
        if (t < m) s[first + t] = x[at][t];
    }
    block_add_u64(c, inv);
}

// The levels above, four runs of `width` into one: the three searches of an
// element go on together (n = 200 000: 13.7 us for a level of four runs, against
// two of 6.7 us and a launch more for two runs at a time).
__global__ __launch_bounds__(kWideThreads) void merge_four_kernel(const uint32_t *__restrict__ in,
                                                                   uint32_t n, uint32_t width,
                                                                   uint32_t *__restrict__ out,
                                                                   unsigned long long *__restrict__ inv) {
    unsigned long long c = 0;
    for (uint64_t l = static_cast<uint64_t>(blockIdx.x) * kWideThreads + threadIdx.x; l < n;
         l += static_cast<uint64_t>(gridDim.x) * kWideThreads) {
        const uint32_t i = static_cast<uint32_t>(l);
        const uint64_t first = i / width / 4u * 4u * static_cast<uint64_t>(width);
        const uint32_t own = static_cast<uint32_t>((i - first) / width);
        const uint32_t x = in[i];
        uint32_t lo[3], hi[3], start[3], end[3];
        bool earlier[3];
#pragma unroll
        for (uint32_t q = 0; q < 3u; ++q) {  // the three other runs
            const uint32_t r = q < own ? q : q + 1u;
            const uint64_t a = first + r * static_cast<uint64_t>(width);
            const uint64_t b = a + width;
            start[q] = static_cast<uint32_t>(a < n ? a : n);
            end[q] = static_cast<uint32_t>(b < n ? b : n);
            earlier[q] = q < own;
            lo[q] = start[q];
            hi[q] = end[q];
        }
        while (lo[0] < hi[0] || lo[1] < hi[1] || lo[2] < hi[2]) {
            uint32_t y[3], mid[3];
#pragma unroll
            for (uint32_t q = 0; q < 3u; ++q) {
                mid[q] = lo[q] + ((hi[q] - lo[q]) >> 1);
                y[q] = lo[q] < hi[q] ? in[mid[q]] : 0u;
            }
#pragma unroll
            for (uint32_t q = 0; q < 3u; ++q) {
                if (lo[q] >= hi[q]) continue;
                if (earlier[q] ? y[q] <= x : y[q] < x) lo[q] = mid[q] + 1u;
                else hi[q] = mid[q];
            }
        }
        uint64_t at = first + (i - first) % width;
#pragma unroll
        for (uint32_t q = 0; q < 3u; ++q) {
            at += lo[q] - start[q];
            if (earlier[q]) c += end[q] - lo[q];
        }
        out[at] = x;
    }
    block_add_u64(c, inv);
}

// Kendall pair counts on min-ranks (ties exactly where the scores tie).
// Block (x, y): i-tile y (one vertex per thread), j-tiles x * kPairTiles ..
// (those not before the i-tile) staged in LDS.  Per pair, with
// da = sign(a_j - a_i), db = sign(b_j - b_i) in {-1, 0, 1} (ranks < 2^31, so
// the differences do not overflow): s += da db, qa += da^2, qb += db^2,
// qab += (da db)^2; then tied in a = pairs - qa, tied in b = pairs - qb, tied
// in both = pairs - qa - qb + qab.
constexpr uint32_t kPairTiles = 8;

// sign(x) as one v_med3_i32 (the compiler rewrites min/max into compares and
// selects); register-only, no memory operand.
__device__ __forceinline__ int32_t sign3(int32_t x) {
    int32_t r;
    asm("v_med3_i32 %0, %1, -1, 1" : "=v"(r) : "v"(x));
    return r;
}

__global__ __launch_bounds__(kRankThreads) void kendall_kernel(const uint32_t *__restrict__ ra,
                                                               const uint32_t *__restrict__ rb,
                                                               uint32_t n,
                                                               unsigned long long *__restrict__ out) {
    __shared__ uint2 sj[kRankThreads];
    __shared__ long long red[5][kRankThreads / 64];
    const uint32_t ti = blockIdx.y, tid = threadIdx.x;
    const uint32_t i = ti * kRankThreads + tid;
    const int32_t ai = i < n ? static_cast<int32_t>(ra[i]) : 0;
    const int32_t bi = i < n ? static_cast<int32_t>(rb[i]) : 0;
    int32_t s = 0, qa = 0, qb = 0, qab = 0, pairs = 0;
    const uint32_t ntiles = (n + kRankThreads - 1) / kRankThreads;
    auto pair = [&](uint2 j) {
        const int32_t da = sign3(static_cast<int32_t>(j.x) - ai);
        const int32_t db = sign3(static_cast<int32_t>(j.y) - bi);
        const int32_t p = da * db;
        s += p;
        qa += da * da;
        qb += db * db;
        qab += p * p;
    };
    for (uint32_t q = 0; q < kPairTiles; ++q) {
        const uint32_t tj = blockIdx.x * kPairTiles + q;
        if (tj >= ntiles) break;
        if (tj < ti) continue;  // uniform over the block
        const uint32_t j0 = tj * kRankThreads;
        __syncthreads();
        sj[tid] = j0 + tid < n ? make_uint2(ra[j0 + tid], rb[j0 + tid]) : make_uint2(0u, 0u);
        __syncthreads();
        if (i >= n) continue;
        if (tj != ti && j0 + kRankThreads <= n) {  // a full tile off the diagonal
#pragma unroll 8
            for (uint32_t jj = 0; jj < kRankThreads; ++jj) pair(sj[jj]);
            pairs += kRankThreads;
        } else {  // pairs (i, j), i < j < n
            const uint32_t jlo = tj == ti ? tid + 1 : 0, jhi = min(kRankThreads, n - j0);
            for (uint32_t jj = jlo; jj < jhi; ++jj) pair(sj[jj]);
            pairs += static_cast<int32_t>(jhi > jlo ? jhi - jlo : 0u);
        }
    }
    // block sums, one atomic each: s, tied in a, tied in b, tied in both
    const long long v[5] = {s, pairs - qa, pairs - qb, pairs - qa - qb + qab, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        long long x = v[c];
        for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
        if ((tid & 63u) == 0) red[c][tid >> 6] = x;
    }
    __syncthreads();
    if (tid < 4) {
        long long x = 0;
        for (uint32_t w = 0; w < kRankThreads / 64; ++w) x += red[tid][w];
        if (x) atomicAdd(&out[tid], static_cast<unsigned long long>(x));
    }
}

inline unsigned int blocks_for(uint64_t items, uint32_t threads) {
    return static_cast<unsigned int>((items + threads - 1) / threads);
}
inline unsigned int wide_blocks(uint64_t items) {
    const uint64_t b = (items + kWideThreads - 1) / kWideThreads;
    return static_cast<unsigned int>(b < kWideBlocks ? b : kWideBlocks);
}

// Runs of 64 keys per wave and tile: short tiles while the tiles are few, so
// that 200 000 keys still fill the CUs; long ones once there are thousands,
// whose counts would otherwise be as much work as the keys.
constexpr uint32_t kShortTile = 4, kLongTile = 16;
inline uint32_t tile_rounds(uint32_t n) { return n <= (1u << 20) ? kShortTile : kLongTile; }

}  // namespace

uint32_t rank_tiles(uint32_t n) {
    const uint32_t keys = tile_rounds(n) * kRankThreads;
    return n / keys + (n % keys ? 1u : 0u);
}

hipError_t launch_rank_keys(const double *score, uint32_t n, bool descending, const SortBufs &b,
                            SortInfo *info, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    keys_kernel<<<wide_blocks(n), kWideThreads, 0, stream>>>(
        score, n, descending ? 1u : 0u, b.key[0], b.val[0], info);
    return hipGetLastError();
}

hipError_t launch_sort_pass(const SortBufs &b, uint32_t n, uint32_t p, const SortInfo *info,
                            unsigned int *thist, unsigned int *total, unsigned int *tell,
                            unsigned int number, hipStream_t stream) {
    if (n < 2) return hipSuccess;
    const uint32_t ntiles = rank_tiles(n);
    const bool shorts = tile_rounds(n) == kShortTile;
    if (shorts)
        tile_hist_kernel<kShortTile><<<ntiles, kRankThreads, 0, stream>>>(b, n, p, ntiles, info, thist,
                                                                          total, tell, number);
    else
        tile_hist_kernel<kLongTile><<<ntiles, kRankThreads, 0, stream>>>(b, n, p, ntiles, info, thist,
                                                                         total, tell, number);
    tile_scan_kernel<<<256, 64, 0, stream>>>(thist, ntiles, p, info, total);
    if (shorts)
        tile_scatter_kernel<kShortTile><<<ntiles, kRankThreads, 0, stream>>>(b, n, p, ntiles, info, thist);
    else
        tile_scatter_kernel<kLongTile><<<ntiles, kRankThreads, 0, stream>>>(b, n, p, ntiles, info, thist);
    return hipGetLastError();
}

hipError_t launch_order(const SortBufs &b, uint32_t n, const SortInfo *info, int32_t *order,
                        int32_t *rank, hipStream_t stream) {
    if (n == 0 || (!order && !rank)) return hipSuccess;
    order_kernel<<<blocks_for(n, kRankThreads), kRankThreads, 0, stream>>>(b, n, info, order, rank);
    return hipGetLastError();
}

hipError_t launch_min_rank(const SortBufs &b, uint32_t n, const SortInfo *info, uint32_t *out,
                           unsigned long long *ties, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    min_rank_kernel<<<wide_blocks(n), kWideThreads, 0, stream>>>(b, n, info, out, ties);
    return hipGetLastError();
}

hipError_t launch_discordant(const SortBufs &b, uint32_t n, const SortInfo *info_b, SortInfo *pair,
                             const uint32_t *ra, const uint32_t *rb, unsigned int *thist,
                             unsigned int *totals, uint32_t *s, uint32_t *tmp,
                             unsigned long long *out, hipStream_t stream) {
    if (n < 2) return hipSuccess;
    pair_keys_kernel<<<blocks_for(n, kRankThreads), kRankThreads, 0, stream>>>(b, n, info_b, ra, rb,
                                                                              out + 1, pair, s);
    uint32_t bytes = 1;
    while (bytes < 4u && (static_cast<uint64_t>(n - 1u) >> (8u * bytes))) ++bytes;
    for (uint32_t p = 0; p < bytes; ++p) {
        const hipError_t e = launch_sort_pass(b, n, p, pair, thist, totals + 256u * p, nullptr, 0u,
                                              stream);
        if (e != hipSuccess) return e;
    }
    pair_order_kernel<<<blocks_for(n, kRankThreads), kRankThreads, 0, stream>>>(b, n, pair, rb, s);
    joint_ties_kernel<<<wide_blocks(n), kWideThreads, 0, stream>>>(b, n, pair, s, out + 3);
    merge_tile_kernel<<<wide_blocks(n), kWideThreads, 0, stream>>>(s, n, out);
    for (uint64_t w = kWideThreads; w < n; w *= 4) {
        merge_four_kernel<<<wide_blocks(n), kWideThreads, 0, stream>>>(
            s, n, static_cast<uint32_t>(w), tmp, out);
        uint32_t *t = s;
        s = tmp;
        tmp = t;
    }
    return hipGetLastError();
}

hipError_t launch_kendall(const uint32_t *ra, const uint32_t *rb, uint32_t n,
                          unsigned long long *out, hipStream_t stream) {
    if (n < 2) return hipSuccess;
    const uint32_t ntiles = (n + kRankThreads - 1) / kRankThreads;
    const dim3 grid((ntiles + kPairTiles - 1) / kPairTiles, ntiles);
    kendall_kernel<<<grid, kRankThreads, 0, stream>>>(ra, rb, n, out);
    return hipGetLastError();
}

}  // namespace fc
