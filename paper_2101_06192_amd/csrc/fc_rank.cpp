// fc_rank and fc_kendall_tau: the ranking output of the estimate (Section 6,
// "Vertex Ranking") on the device.
#include <cmath>
#include <cstddef>
#include <cstring>
#include <limits>

#include "fc_internal.hpp"
#include "fc_rank_kernels.hpp"

using namespace fc_host;

namespace {

// Counters of one call (rk_hist), zeroed together: the digit counts of up to
// three sorts (the third one of four bytes), what each knows of its keys, the
// four Kendall sums.
struct RankSmall {
    unsigned int totals[2][8 * 256];
    unsigned int pair_totals[4 * 256];
    fc::SortInfo info[2], pair;
    unsigned long long out[4];
};

int ensure_sort(fc_ctx *ctx, size_t n, fc::SortBufs *b, RankSmall **small) {
    int rc;
    if ((rc = ensure(ctx, ctx->rk_key0, 8 * n, "rank keys")) ||
        (rc = ensure(ctx, ctx->rk_key1, 8 * n, "rank keys")) ||
        (rc = ensure(ctx, ctx->rk_val0, 4 * n, "rank values")) ||
        (rc = ensure(ctx, ctx->rk_val1, 4 * n, "rank values")) ||
        (rc = ensure(ctx, ctx->rk_hist, sizeof(RankSmall), "digit counts")) ||
        (rc = ensure(ctx, ctx->rk_thist,
                     4 * 256 * static_cast<size_t>(fc::rank_tiles(static_cast<uint32_t>(n))),
                     "tile counts")))
        return rc;
    b->key[0] = static_cast<uint64_t *>(ctx->rk_key0.ptr);
    b->key[1] = static_cast<uint64_t *>(ctx->rk_key1.ptr);
    b->val[0] = static_cast<int32_t *>(ctx->rk_val0.ptr);
    b->val[1] = static_cast<int32_t *>(ctx->rk_val1.ptr);
    *small = static_cast<RankSmall *>(ctx->rk_hist.ptr);
    FC_HIP(ctx, hipMemsetAsync(*small, 0, sizeof(RankSmall), ctx->stream), "memset counts");
    return FC_OK;
}

// Stable sort of the scores; the vertices end in the buffers as their info says.
// The first pass tells the host the bytes in which the keys differ: the passes of the
// others are enqueued until then (they return at once) and left out from then on.  With
// all of them enqueued a ranking of 1000 scores took 133 us, however few bytes differ;
// so 137 (eight bytes), 97 (two) and 46 (none).  When the host waited for the digit
// counts: 190, 123 and 75.
int sort_scores(fc_ctx *ctx, const double *score, uint32_t n, bool descending,
                const fc::SortBufs &b, RankSmall *small, int which) {
    FC_HIP(ctx, fc::launch_rank_keys(score, n, descending, b, &small->info[which], ctx->stream),
           "rank keys");
    unsigned int *tell = nullptr, *told = &ctx->host_bytes[which];
    FC_HIP(ctx, hipHostGetDevicePointer(reinterpret_cast<void **>(&tell), told, 0), "host pointer");
    // (what an earlier call told, or one that failed tells still, has another number)
    ctx->sorts = (ctx->sorts + 1u) & 0xFFFFFFu;
    for (uint32_t p = 0; p < 8; ++p) {
        const unsigned int bytes = __atomic_load_n(told, __ATOMIC_ACQUIRE);
        if (bytes >> 8 == ctx->sorts && !((bytes >> p) & 1u)) continue;
        FC_HIP(ctx, fc::launch_sort_pass(b, n, p, &small->info[which],
                                         static_cast<unsigned int *>(ctx->rk_thist.ptr),
                                         small->totals[which] + 256u * p, p == 0 ? tell : nullptr,
                                         ctx->sorts, ctx->stream),
               "radix sort");
    }
    return FC_OK;
}

}  // namespace

extern "C" int fc_rank(fc_ctx *ctx, const double *score, int32_t n, int32_t descending,
                       int32_t *order, int32_t *rank) {
    int rc = begin(ctx);
    if (rc) return rc;
    if (n < 0) return set_err(ctx, FC_ERR_ARG, "n must be >= 0");
    if (n == 0) return FC_OK;
    if (!score) return set_err(ctx, FC_ERR_ARG, "score is NULL");
    const uint32_t un = static_cast<uint32_t>(n);
    fc::SortBufs b;
    RankSmall *small;
    if ((rc = ensure_sort(ctx, static_cast<size_t>(n), &b, &small)) ||
        (rc = sort_scores(ctx, score, un, descending != 0, b, small, 0)))
        return rc;
    FC_HIP(ctx, fc::launch_order(b, un, &small->info[0], order, rank, ctx->stream), "order");
    fc::SortInfo info{};
    FC_HIP(ctx, hipMemcpyAsync(&info, &small->info[0], sizeof(info), hipMemcpyDeviceToHost,
                               ctx->stream),
           "copy flag");
    FC_HIP(ctx, hipStreamSynchronize(ctx->stream), "rank");
    if (info.bad) return set_err(ctx, FC_ERR_ARG, "score contains NaN");
    return FC_OK;
}

extern "C" int fc_kendall_tau(fc_ctx *ctx, const double *a, const double *b, int32_t n,
                              double *tau_b, int64_t *counts) {
    int rc = begin(ctx);
    if (rc) return rc;
    if (n < 0) return set_err(ctx, FC_ERR_ARG, "n must be >= 0");
    if (static_cast<int64_t>(n) > 65535LL * 256)
        return set_err(ctx, FC_ERR_UNSUPPORTED, "n must be <= 65535 * 256");
    if (n > 0 && (!a || !b)) return set_err(ctx, FC_ERR_ARG, "a and b must be device pointers");
    const uint32_t un = static_cast<uint32_t>(n);
    // sums on the device: [0] n_c - n_d (pair kernel) or n_d (merge count),
    // [1] tied in a, [2] tied in b, [3] tied in both
    unsigned long long out[4] = {0, 0, 0, 0};
    const bool pairs = ctx->kendall_pairs;
    if (n > 0) {
        const size_t nn = static_cast<size_t>(n);
        fc::SortBufs bufs;
        RankSmall *small;
        if ((rc = ensure(ctx, ctx->rk_ra, 4 * nn, "ranks")) ||
            (rc = ensure(ctx, ctx->rk_rb, 4 * nn, "ranks")) ||
            (rc = ensure(ctx, ctx->rk_s, 8 * nn, "merge runs")) ||
            (rc = ensure_sort(ctx, nn, &bufs, &small)))
            return rc;
        uint32_t *ra = static_cast<uint32_t *>(ctx->rk_ra.ptr);
        uint32_t *rb = static_cast<uint32_t *>(ctx->rk_rb.ptr);
        // each vector's scores -> min-ranks (equal scores share a rank) and its ties
        if ((rc = sort_scores(ctx, a, un, false, bufs, small, 0))) return rc;
        FC_HIP(ctx, fc::launch_min_rank(bufs, un, &small->info[0], ra, &small->out[1], ctx->stream),
               "min ranks");
        if ((rc = sort_scores(ctx, b, un, false, bufs, small, 1))) return rc;
        FC_HIP(ctx, fc::launch_min_rank(bufs, un, &small->info[1], rb, &small->out[2], ctx->stream),
               "min ranks");
        if (pairs) {  // all n(n-1)/2 pairs compared (the definition, tiled)
            FC_HIP(ctx, hipMemsetAsync(small->out, 0, sizeof(out), ctx->stream), "memset sums");
            FC_HIP(ctx, fc::launch_kendall(ra, rb, un, small->out, ctx->stream), "kendall");
        } else {
            // discordant pairs: strict inversions of one vector's ranks in the order
            // of the other (ties there broken by the first); pairs tied in both
            uint32_t *s = static_cast<uint32_t *>(ctx->rk_s.ptr);
            FC_HIP(ctx, fc::launch_discordant(bufs, un, &small->info[1], &small->pair, ra, rb,
                                              static_cast<unsigned int *>(ctx->rk_thist.ptr),
                                              small->pair_totals, s, s + nn, small->out, ctx->stream),
                   "discordant pairs");
        }
        struct {
            fc::SortInfo info[2], pair;
            unsigned long long out[4];
        } got;
        static_assert(sizeof(got) == sizeof(RankSmall) - offsetof(RankSmall, info), "the tail of RankSmall");
        FC_HIP(ctx, hipMemcpyAsync(&got, small->info, sizeof(got), hipMemcpyDeviceToHost, ctx->stream),
               "copy sums");
        FC_HIP(ctx, hipStreamSynchronize(ctx->stream), "kendall");
        if (got.info[0].bad || got.info[1].bad) return set_err(ctx, FC_ERR_ARG, "score contains NaN");
        std::memcpy(out, got.out, sizeof(out));
    }
    const int64_t n0 = static_cast<int64_t>(n) * (n - 1) / 2;
    const int64_t ta = static_cast<int64_t>(out[1]), tb = static_cast<int64_t>(out[2]),
                  tab = static_cast<int64_t>(out[3]);
    const int64_t untied = n0 - ta - tb + tab;  // n_c + n_d
    const int64_t s = pairs ? static_cast<int64_t>(out[0]) : untied - 2 * static_cast<int64_t>(out[0]);
    if (counts) {
        counts[0] = (untied + s) / 2;
        counts[1] = (untied - s) / 2;
        counts[2] = ta;
        counts[3] = tb;
        counts[4] = tab;
    }
    if (tau_b) {
        const int64_t d1 = n0 - ta, d2 = n0 - tb;
        *tau_b = (d1 == 0 || d2 == 0)
                     ? std::numeric_limits<double>::quiet_NaN()
                     : static_cast<double>(s) /
                           std::sqrt(static_cast<double>(d1) * static_cast<double>(d2));
    }
    return FC_OK;
}
