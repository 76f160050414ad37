// Degree-class relabelling for the LDS-counter sampler.
//
// That sampler keeps the in-arrow count of every vertex of a tree in LDS.  A
// count never exceeds the vertex degree, so a vertex of degree d gets a field
// of 4 << c bits, c = class(d): 4 bits up to degree 15, 8 up to 255, 16 up to
// 65535, else 32 (the hubs-first sampler keeps no counts: its classes end at 15, 63
// and 255, to tell the hubs apart).  Isolated vertices form a fifth class with no field: they
// are never a target, and in every tree they are roots after one draw.
// Vertices are renumbered so that each class is a contiguous range of
// internal ids (class 0 first, isolated vertices last; original order kept
// inside a class), which makes a field's LDS word and shift plain arithmetic
// on the internal id.  Randomness and every output stay on original ids: the relabelled
// vertex record carries the original id, and the relabelled adjacency holds
// (internal, original) pairs of each neighbour at the same CSR positions
// (internal id in the low bits, original id shifted by 18 for the LDS sampler
// or 32 for the others), so the neighbour chosen by a draw is the one the
// original CSR gives.
#include "fc_kernels.hpp"

namespace fc {

namespace {

constexpr int kPlaceThreads = 1024;
constexpr uint32_t kClasses = kRelabelClasses;  // four field widths, then isolated vertices

__device__ __forceinline__ uint32_t deg_class(uint32_t d, ClassOrder order) {
    const uint32_t top1 = order == kHubsFirst ? 63u : 255u, top2 = order == kHubsFirst ? 255u : 65535u;
    return d == 0u ? 4u : d <= 15u ? 0u : d <= top1 ? 1u : d <= top2 ? 2u : 3u;
}

// Per block of kPlaceThreads vertices: how many fall in each class; with ends, the sums of
// the degrees from 2^b to 2^(b+1) - 1 (a block's fit 32 bits: row offsets do).
__global__ __launch_bounds__(kPlaceThreads) void class_count_kernel(
    const int32_t *__restrict__ row_ptr, uint32_t n, ClassOrder order, uint32_t *__restrict__ blk,
    unsigned long long *ends) {
    __shared__ uint32_t s[kClasses], s_ends[kDegreeBits];
    if (threadIdx.x < kDegreeBits) s_ends[threadIdx.x] = 0;
    if (threadIdx.x < kClasses) s[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t v = blockIdx.x * kPlaceThreads + threadIdx.x;
    const uint32_t d = v < n ? static_cast<uint32_t>(row_ptr[v + 1] - row_ptr[v]) : 0u;
    const uint32_t c = v < n ? deg_class(d, order) : kClasses;
    if (ends && d) atomicAdd(&s_ends[31 - __clz(d)], d);
    for (uint32_t k = 0; k < kClasses; ++k) {
        const uint64_t m = __ballot(c == k);
        if ((threadIdx.x & 63u) == 0 && m) atomicAdd(&s[k], static_cast<uint32_t>(__popcll(m)));
    }
    __syncthreads();
    if (threadIdx.x < kClasses) blk[blockIdx.x * kClasses + threadIdx.x] = s[threadIdx.x];
    if (ends && threadIdx.x < kDegreeBits && s_ends[threadIdx.x])
        atomicAdd(&ends[threadIdx.x], static_cast<unsigned long long>(s_ends[threadIdx.x]));
}

// Rank of class c in the id order: narrowest field first (LDS sampler) or
// widest first (hybrid and hubs-first samplers, whose LDS holds a prefix of the ids:
// the highest-degree vertices, which receive most arrows); isolated vertices last.
__device__ __forceinline__ uint32_t class_rank(uint32_t c, ClassOrder order) {
    return c == 4u || order == kNarrowFirst ? c : 3u - c;
}

// One block: base[b][k] = first internal id of class k in block b; bounds[r] =
// end of the class of rank r, r < 4 (bounds[3] = number of vertices that are
// not isolated).  Thread t owns a run of consecutive blocks: it sums its run,
// the run sums are scanned over the waves, and it walks its run again.  (One
// thread per class walking all blocks in turn took 35 us for 200 K vertices
// and 680 us for 4 M, a chain of dependent loads; now 4.0 us and 12.5 us.)
constexpr uint32_t kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void class_scan_kernel(
    const uint32_t *__restrict__ blk, uint32_t nb, ClassOrder order, uint32_t *__restrict__ base,
    uint32_t *__restrict__ bounds) {
    constexpr uint32_t kWaves = kScanThreads / 64u;
    __shared__ uint32_t s_wave[kClasses][kWaves];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t run = (nb + kScanThreads - 1u) / kScanThreads;
    const uint64_t b0 = static_cast<uint64_t>(threadIdx.x) * run;
    const uint64_t b1 = b0 + run < nb ? b0 + run : nb;
    uint32_t sum[kClasses] = {}, before[kClasses];
    for (uint64_t b = b0; b < b1; ++b)
        for (uint32_t k = 0; k < kClasses; ++k) sum[k] += blk[b * kClasses + k];
    for (uint32_t k = 0; k < kClasses; ++k) {  // inclusive scan over the wave's runs
        uint32_t x = sum[k];
        for (uint32_t off = 1; off < 64u; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (lane == 63u) s_wave[k][wave] = x;
        before[k] = x - sum[k];
    }
    __syncthreads();
    uint32_t total[kClasses];
    for (uint32_t k = 0; k < kClasses; ++k) {
        uint32_t t = 0;
        for (uint32_t w = 0; w < kWaves; ++w) {
            if (w == wave) before[k] += t;
            t += s_wave[k][w];
        }
        total[k] = t;
    }
    for (uint32_t k = 0; k < kClasses; ++k) {  // classes of a lower rank come first
        const uint32_t r = class_rank(k, order);
        uint32_t start = 0;
        for (uint32_t j = 0; j < kClasses; ++j)
            if (class_rank(j, order) < r) start += total[j];
        if (threadIdx.x == 0 && r + 1 < kClasses) bounds[r] = start + total[k];
        before[k] += start;
    }
    for (uint64_t b = b0; b < b1; ++b)
        for (uint32_t k = 0; k < kClasses; ++k) {
            base[b * kClasses + k] = before[k];
            before[k] += blk[b * kClasses + k];
        }
}

// inv[v] = internal id of v, orig[internal] = v: rank inside the block from
// per-wave ballots, waves in order.
__global__ __launch_bounds__(kPlaceThreads) void class_place_kernel(
    const int32_t *__restrict__ row_ptr, uint32_t n, ClassOrder order,
    const uint32_t *__restrict__ base, uint32_t *__restrict__ inv, uint32_t *__restrict__ orig) {
    constexpr uint32_t kWaves = kPlaceThreads / 64;
    __shared__ uint32_t s_wave[kWaves][kClasses];
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t v = blockIdx.x * kPlaceThreads + threadIdx.x;
    const uint32_t c =
        v < n ? deg_class(static_cast<uint32_t>(row_ptr[v + 1] - row_ptr[v]), order) : kClasses;
    uint64_t mine = 0;
    for (uint32_t k = 0; k < kClasses; ++k) {
        const uint64_t m = __ballot(c == k);
        if (c == k) mine = m;
        if (lane == 0) s_wave[wave][k] = static_cast<uint32_t>(__popcll(m));
    }
    __syncthreads();
    if (v >= n) return;
    uint32_t id = base[blockIdx.x * kClasses + c];
    for (uint32_t w = 0; w < wave; ++w) id += s_wave[w][c];
    id += static_cast<uint32_t>(__popcll(mine & ((1ull << lane) - 1ull)));
    inv[v] = id;
    orig[id] = v;
}

// Relabelled records: field always_root becomes original id | always_root << 31.
__global__ void relabel_vrec_kernel(const VRec *__restrict__ vrec, const uint32_t *__restrict__ inv,
                                    uint32_t n, VRec *__restrict__ out) {
    const uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    VRec r = vrec[v];
    r.always_root = v | (r.always_root ? 0x80000000u : 0u);
    out[inv[v]] = r;
}

__global__ void relabel_adj_kernel(const int32_t *__restrict__ col_idx, int64_t nnz,
                                   const uint32_t *__restrict__ inv, uint32_t orig_shift,
                                   unsigned long long *__restrict__ adj) {
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < nnz;
         e += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const uint32_t u = static_cast<uint32_t>(col_idx[e]);
        adj[e] = static_cast<unsigned long long>(inv[u]) |
                 (static_cast<unsigned long long>(u) << orig_shift);
    }
}

}  // namespace

uint32_t relabel_blocks(uint32_t n) { return (n + kPlaceThreads - 1) / kPlaceThreads; }

hipError_t launch_class_bounds(const int32_t *row_ptr, uint32_t n, ClassOrder order, uint32_t *blk,
                               uint32_t *base, uint32_t *bounds, unsigned long long *ends,
                               hipStream_t stream) {
    const uint32_t nb = relabel_blocks(n);
    if (nb == 0) return hipSuccess;
    class_count_kernel<<<nb, kPlaceThreads, 0, stream>>>(row_ptr, n, order, blk, ends);
    class_scan_kernel<<<1, kScanThreads, 0, stream>>>(blk, nb, order, base, bounds);
    return hipGetLastError();
}

hipError_t launch_relabel_vrec(const VRec *vrec, const uint32_t *inv, uint32_t n, VRec *vrec_r,
                               hipStream_t stream) {
    if (n == 0) return hipSuccess;
    relabel_vrec_kernel<<<(n + 255) / 256, 256, 0, stream>>>(vrec, inv, n, vrec_r);
    return hipGetLastError();
}

hipError_t launch_relabel_graph(const int32_t *row_ptr, const int32_t *col_idx, uint32_t n,
                                int64_t nnz, ClassOrder order, const uint32_t *base,
                                uint32_t orig_shift,
                                uint32_t *inv, uint32_t *orig, unsigned long long *adj,
                                hipStream_t stream) {
    const uint32_t nb = relabel_blocks(n);
    if (nb == 0) return hipSuccess;
    class_place_kernel<<<nb, kPlaceThreads, 0, stream>>>(row_ptr, n, order, base, inv, orig);
    if (nnz > 0) {
        int64_t blocks = (nnz + 255) / 256;
        if (blocks > 16384) blocks = 16384;
        relabel_adj_kernel<<<static_cast<unsigned int>(blocks), 256, 0, stream>>>(
            col_idx, nnz, inv, orig_shift, adj);
    }
    return hipGetLastError();
}

}  // namespace fc
