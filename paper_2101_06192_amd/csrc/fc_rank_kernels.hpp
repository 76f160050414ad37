// Host-side launch wrappers of the ranking output kernels (rank.hip).  Every wrapper
// enqueues on `stream` and returns the launch status; none synchronises.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace fc {

// What one sort knows of its keys (device memory, zeroed by the caller): the
// bits in which any two keys differ, and whether a score was NaN.
struct SortInfo {
    unsigned long long vary;
    unsigned int bad;
    unsigned int pad;
};
// Keys and values in two buffers: a sort reads buffer 0 and alternates; the
// number of bytes in which the keys differ tells where it ends.
struct SortBufs {
    uint64_t *key[2];
    int32_t *val[2];
};

// Order-preserving keys of the scores (complemented when descending) and the
// values 0 .. n - 1 into buffer 0, and *info.
hipError_t launch_rank_keys(const double *score, uint32_t n, bool descending, const SortBufs &b,
                            SortInfo *info, hipStream_t stream);
// Tiles of the radix sort (thist holds 256 * rank_tiles(n) counters).
uint32_t rank_tiles(uint32_t n);
// Stable sort by byte p of the keys, after the bytes below (nothing where the keys do not
// differ in it); total: 256 zeroed counters; tell (or null): a word of coherent host
// memory that gets a bit for every byte in which the keys differ, and number << 8.
hipError_t launch_sort_pass(const SortBufs &b, uint32_t n, uint32_t p, const SortInfo *info,
                            unsigned int *thist, unsigned int *total, unsigned int *tell,
                            unsigned int number, hipStream_t stream);
// The sorted values into order and their inverse into rank (either may be
// null); nothing when info->bad.
hipError_t launch_order(const SortBufs &b, uint32_t n, const SortInfo *info, int32_t *order,
                        int32_t *rank, hipStream_t stream);
// out[val[i]] = the number of sorted keys below key[i]; *ties += pairs of equal keys.
hipError_t launch_min_rank(const SortBufs &b, uint32_t n, const SortInfo *info, uint32_t *out,
                           unsigned long long *ties, hipStream_t stream);
// Discordant pairs of two vectors from their min-ranks: out[0] += pairs ordered
// strictly the other way, out[3] += pairs tied in both; out[1], out[2] hold the
// pairs tied in a and in b.  b holds the order by vector b (its sort's info in
// info_b); pair and totals (4 x 256) are zero before; s and tmp: n scratch each.
hipError_t launch_discordant(const SortBufs &b, uint32_t n, const SortInfo *info_b, SortInfo *pair,
                             const uint32_t *ra, const uint32_t *rb, unsigned int *thist,
                             unsigned int *totals, uint32_t *s, uint32_t *tmp,
                             unsigned long long *out, hipStream_t stream);
// Kendall pair counts of two rank vectors (< 2^31) over all pairs i < j
// (n <= 65535 * 256): out[0] += sum of sign products, out[1..3] += pairs tied in
// a, in b, in both (out zeroed by the caller; out[0] is two's complement).
hipError_t launch_kendall(const uint32_t *ra, const uint32_t *rb, uint32_t n,
                          unsigned long long *out, hipStream_t stream);

}  // namespace fc
