// Finding the rows of consecutive CSR entries, wave by wave (wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fc {

// Rows of 64 consecutive CSR entries at a time, entry j0 + lane for each lane.
// The lanes hold the bounds of 64 consecutive rows between calls, so entries
// that go on in those rows (or the next 64) cost six lane shuffles and no
// search; a wave that jumps finds its row by a 64-way search of row_ptr
// (four rounds of one load for 2^24 rows, instead of 24 dependent loads).
struct RowFinder {
    int32_t r = -1;           // first row held (wave-uniform), -1: none yet
    int32_t rb = 0, re = 0;   // this lane's row r + lane: its bounds (empty past the last row)

    // The row holding entry j: largest v in [0, n) with row_ptr[v] <= j.  j is
    // wave-uniform, 0 <= j < row_ptr[n], row_ptr monotone from 0.
    static __device__ int32_t search(const int32_t *__restrict__ row_ptr, int32_t n, int64_t j) {
        const uint32_t lane = threadIdx.x & 63u;
        int64_t lo = 0, hi = n;
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + 63) >> 6;
            const int64_t p = lo + static_cast<int64_t>(lane) * step;
            const bool le = p < hi && row_ptr[p] <= j;
            const int64_t c = __popcll(__ballot(le));  // a prefix of the lanes, lane 0 in it
            lo += (c > 0 ? c - 1 : 0) * step;
            hi = hi < lo + step ? hi : lo + step;
        }
        return static_cast<int32_t>(lo);
    }

    __device__ void hold(const int32_t *__restrict__ row_ptr, int32_t n, int32_t first) {
        const int64_t v = static_cast<int64_t>(first) + (threadIdx.x & 63u);
        r = first;
        rb = row_ptr[v < n ? v : n];
        re = row_ptr[v < n ? v + 1 : n];
    }

    // Row *v of entry j0 + lane and its bounds [*b, *e), for the lanes whose
    // entry is below nnz (and in a row); all 64 lanes of the wave call it
    // together with the same j0 < nnz, in ascending order of j0.
    __device__ void find(const int32_t *__restrict__ row_ptr, int32_t n, int64_t j0, int64_t nnz,
                         int32_t *v, int32_t *b, int32_t *e) {
        const uint32_t lane = threadIdx.x & 63u;
        const int64_t j = j0 + lane;
        bool open = j < nnz;
        if (r < 0) hold(row_ptr, n, search(row_ptr, n, j0));
        while (true) {
            // how many of the 64 held rows end at or before entry j
            uint32_t i = 0;
            for (uint32_t s = 32; s > 0; s >>= 1) {
                const int32_t end = __shfl(re, static_cast<int>(i + s - 1u), 64);
                if (end <= j) i += s;
            }
            const int32_t last = __shfl(re, 63, 64);
            const int32_t bi = __shfl(rb, static_cast<int>(i), 64);
            const int32_t ei = __shfl(re, static_cast<int>(i), 64);
            if (open && j < last) {
                *v = r + static_cast<int32_t>(i);
                *b = bi;
                *e = ei;
                open = false;
            }
            const uint64_t left = __ballot(open);
            if (!left) return;
            // the first entry without a row lies beyond the held rows: the next
            // 64 rows most often, found again when they are not enough
            const int64_t jl = j0 + static_cast<int64_t>(__ffsll(static_cast<unsigned long long>(left)) - 1);
            const int64_t next = static_cast<int64_t>(r) + 64;
            hold(row_ptr, n, static_cast<int32_t>(next < n ? next : n - 1));
            if (__shfl(re, 63, 64) <= jl) {
                hold(row_ptr, n, search(row_ptr, n, jl));
                if (__shfl(re, 63, 64) <= jl) return;  // row_ptr that ends before nnz (unchecked graph)
            }
        }
    }
};

}  // namespace fc
