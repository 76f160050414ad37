// Host-side internals shared by the C-ABI translation units: the context,
// device buffers and the graph preparation helpers.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <memory>
#include <string>

#include "fc.h"
#include "fc_kernels.hpp"

struct DevBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
};

struct Small {  // device-side counters of one call
    fc::Totals totals;
    unsigned int queue;
    unsigned int pad0;
    fc::GraphCheck check;
    unsigned long long cross;  // CSR entries that join different tiles
    unsigned int dmax;
    unsigned int pad;
    unsigned long long phase_ticks[8];
    unsigned int class_bounds[4];  // n0, n1, n2, n3 of the degree-class relabelling
    double wtotal;                 // sum of the weighted degrees (weighted graphs)
    // (last: left out of a call on a caller's array, which asks for none of it)
    unsigned long long ends[fc::kDegreeBits];  // sums of the degrees, by their highest bit
};

struct fc_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string last_error;
    std::string kernels;  // the sampling kernels of the last call
    DevBuf state, vrec, row_ptr, col_idx, small, rtmp, thr, cword, ckk, clists, clevels, cbits;
    DevBuf s_r64, s_r, s_p, s_q, s_d, s_pa, s_pb, s_small, s_wdeg;  // solver workspace
    DevBuf s_minv, s_segbase, s_seg, s_segsum;  // solver: preconditioner, long rows' segments
    DevBuf rl_blk, rl_base, rl_inv, rl_orig, rl_vrec, rl_adj;     // degree-class relabelling
    DevBuf iso;                                                   // isolated-vertex bitmap
    DevBuf corigt;                                                // hybrid: target ids per slot
    DevBuf crint;                                                 // hubs first: root counts
    DevBuf cpre;                                                  // pre-drawn tree words or arrows
    bool pre_used = false;                                        // (by the call under way)
    DevBuf weights, wsum, wthr;  // staged edge weights (host graphs), running row weight sums,
                                 // step thresholds
    DevBuf rk_key0, rk_key1, rk_val0, rk_val1, rk_hist, rk_thist, rk_ra, rk_rb, rk_s;  // ranking
    DevBuf g_mat, g_vec, g_part, g_taken, g_scr;  // group closeness: matrix, vectors, sums, flags, scratch
    DevBuf t_ex, t_tl, t_exl, t_ecnt, t_pc, t_sc, t_bl, t_xb;  // tile sampler (exits, counts, lists)
    hipEvent_t ev0 = nullptr, ev1 = nullptr, evm = nullptr;
    Small *host_small = nullptr;  // pinned: where a call's counters are read back
    unsigned int *host_bytes = nullptr;  // pinned, coherent: the bytes that two sorts have to look at
    unsigned int sorts = 0;              // the last one's number
    size_t state_budget = 0;      // bytes of per-tree state the sampler may use
    size_t scratch_limit = 0;     // most bytes of device memory to hold (0: what the device has)
    // what this context's buffers and its batches' take now (a batch may outlive its context)
    std::shared_ptr<std::atomic<size_t>> held = std::make_shared<std::atomic<size_t>>(0);
    uint32_t lanes_per_wave = 64; // active lanes per wave in the lane sampler
    uint32_t max_slots = 0;       // 0 = as many trees in flight as memory allows
    uint32_t cu_count = 256;
    size_t max_lds = 65536;       // dynamic LDS a workgroup may use
    uint32_t coop_threads = 512;  // threads per workgroup in the workgroup sampler
    uint32_t coop_wg_per_cu = 3;  // resident workgroups per CU in the workgroup sampler
    uint32_t force_sampler = 0;   // 0 auto, 1 lane, 2 coop, 3 lds, 4 hyb, 5 tile (environment override)
    bool coop_lds_bits = true;    // settled bitmap in LDS when it fits
    bool coop_word32 = true;      // 32-bit tree words when target and count fit
    bool coop_in_bits = true;     // in-arrow bitmap in LDS when both bitmaps fit
    bool phase_timing = false;    // per-phase wall-clock ticks of the workgroup sampler
    uint32_t max_draws = 0;       // per-vertex draw limit in one tree (0: each sampler's own)
    uint32_t hyb_hot_cap = 0x7FFFFFFF;  // hybrid sampler: cap on the LDS-resident id prefix
    bool coop_lds_counts = true;  // in-arrow counters in LDS when the tree's fields fit
    uint32_t lds_threads = 0;     // threads per workgroup of the LDS-counter sampler (0: by n)
    uint32_t lds_wg_per_cu = 0;   // its resident workgroups per CU (0: as many as fit)
    uint32_t predraw_mib = 32768;  // budget of pre-drawn first arrows (0: off)
    bool kendall_pairs = false;   // Kendall's tau by all pairs instead of merge-sort counts
    uint32_t lds_repop = 3;       // re-formed 2-cycle pops: 0 never, 1 weighted graphs, 2 always,
                                  // 3 always, and timed both ways by batch autotuning
    uint32_t coop_repop = 2;      // the same for the global-counter sampler
    uint32_t lds_lean = 0;        // LDS-counter sampler: the lean register shape for workgroups
                                  // of at most 512 threads (batch autotuning times both)
    uint32_t hub = 1;             // hubs-first sampler: 0 never, 1 by hub_applies where a tree does
                                  // not fit LDS whole, 2 wherever the tile sampler does not go ahead
    uint32_t hub_set = 0;         // its LDS set's vertices (0: the most that fit)
    uint32_t hub_hot = 130;       // of these, per mille, hubs at the start; the rest join later
    uint32_t hub_threads = 1024;  // its threads per workgroup
    uint32_t tile_size = 0;       // tile sampler: vertices per tile (0: the widest that fits LDS)
    uint32_t tile_cross_permille = 100;  // picked automatically when at most this share (per
                                         // mille) of the CSR entries cross tiles
    uint32_t tile_threads = 1024; // threads per workgroup of the tile sampler
    uint32_t tile_repop = 2;      // tile sampler's re-formed 2-cycle pops: 0 never, 1 weighted, 2 always
    uint32_t tile_bits_lds = 1;   // tile sampler's exit and settled bitmaps in LDS when they fit (0: global)
    double wall_khz = 100000.0;   // device wall clock rate
    // Arena mode (fc_sample_noalloc): every buffer of one call is carved from
    // this device range instead of being allocated; null in ordinary contexts.
    char *arena = nullptr;
    size_t arena_size = 0, arena_off = 0;
};


#define FC_HIP(ctx, expr, what)                          \
    do {                                                 \
        hipError_t e_ = (expr);                          \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, what); \
    } while (0)


namespace fc_host {

// static LDS of the LDS-counter kernel (item, tails, totals, phase clocks) with margin
constexpr size_t kLdsStaticBytes = 1024;
// Largest "tile_size" that the tile sampler takes (6 bytes of LDS a vertex).
constexpr uint32_t kTileAsk = 26432;
// fewest non-isolated vertices for which the LDS sampler draws first arrows ahead
constexpr uint32_t kPredrawMinVertices = 16384;

int set_err(fc_ctx *ctx, int code, const std::string &msg);
int hip_fail(fc_ctx *ctx, hipError_t e, const char *what);
// Grow-only device buffer: (re)allocates when `bytes` exceeds its size; in
// arena mode carves it from the context's arena instead (never allocates).  Pre-drawn
// arrows that an earlier call left are given back before an allocation is refused.
int ensure(fc_ctx *ctx, DevBuf &b, size_t bytes, const char *what);
// Frees a buffer that ensure() allocated (held: its context's).
void release(std::atomic<size_t> &held, DevBuf &b);
// Bytes of Small that a context's calls use.
size_t small_bytes(const fc_ctx *ctx);
// Bytes of per-tree state the sampler may use now: the context's budget, or
// in arena mode what is left of the arena.
size_t state_budget_now(const fc_ctx *ctx);
uint32_t env_u32(const char *name, uint32_t dflt);
bool valid_alpha(double a);

// Resolved device view of a graph for one call.
struct GraphView {
    int32_t n = 0;
    int64_t nnz = 0;
    const int32_t *row_ptr = nullptr;
    const int32_t *col_idx = nullptr;
    const double *weights = nullptr;  // device edge weights, or null (unit weights)
    bool pending = false;  // the checks are enqueued (into Small::check, the rest of Small
                           // zeroed) but not read: kernels that follow the graph must look
};

int check_graph_args(fc_ctx *ctx, const fc_graph *g);
// Stage (if on the host) and validate the CSR (and weights) on the device.
// defer: leave the outcome of the checks on the device (out->pending).
int prepare_graph(fc_ctx *ctx, const fc_graph *g, bool trusted, GraphView *out, bool defer = false);
// The error for what the checks found (FC_OK: a valid graph).
int check_outcome(fc_ctx *ctx, const fc::GraphCheck &found);
// Running row weight sums and step thresholds of a weighted graph into the two
// buffers (both null for an unweighted graph).
int weight_tables(fc_ctx *ctx, const GraphView &g, DevBuf &sbuf, DevBuf &tbuf, const double **S,
                  const uint32_t **T);
double now_ms();
int begin(fc_ctx *ctx);
// Threads per workgroup of the LDS-counter sampler for `trees` trees whose
// counters and bitmap take lds_words words of LDS.
uint32_t lds_threads_for(const fc_ctx *ctx, uint64_t trees, uint32_t lds_words);
struct HubShape {
    uint32_t set, lds_bits;
    size_t lds;
};
bool hub_applies(bool fits, uint32_t nl, uint64_t nnz, const unsigned long long *ends, double reach);
HubShape hub_shape(const fc_ctx *ctx, uint32_t nl, uint32_t threads, uint32_t per_cu);
// Threads per workgroup of the small-graph sampler for `trees` trees of n vertices.
uint32_t jump_threads_for(const fc_ctx *ctx, uint32_t n, uint64_t trees);
// Bits of the target field so that n < 2^tshift, and whether a 32-bit tree
// word also holds an in-arrow count up to dmax.
void word_layout(uint32_t n, uint32_t dmax, bool allow32, uint32_t *tshift, bool *word32);
// Global-counter sampler: LDS words of the re-pop filter for a launch of
// `threads` x `per_cu` workgroups (0 when the option is off or nothing fits).
uint32_t coop_repop_words(const fc_ctx *ctx, uint32_t threads, uint32_t per_cu, bool lds_bits,
                          bool in_bits, bool word32, uint32_t n, bool weighted);

}  // namespace fc_host
