// Workgroup-per-tree sampler for small graphs: the whole tree in LDS.
//
// Cycle popping as in the other workgroup samplers (Wilson's theorem: pop any
// cycle of the current arrows until none is left; the tree and the number of
// arrows drawn at every vertex do not depend on the order), but with nothing
// of the tree outside LDS, so that paths can be followed by pointer jumping
// instead of peeling the arrow forest level by level.  On a graph of 1000
// vertices peeling is a chain of dozens to hundreds of levels, each with a
// load from memory and barriers; jumping takes log2 of the longest path, in
// steps of two LDS reads.
//
// A tree goes through
//   draw     the first arrow of every vertex
//   2-cycles every vertex whose target points back at it draws again; the
//            vertices that drew are checked again among themselves and their
//            targets until no 2-cycle is left (most cycles are 2-cycles, and a
//            check is two LDS reads)
//   jump     J[v] <- J[J[v]] from J = arrow; a vertex that reaches u* (or a
//            settled vertex) is settled.  A pass that settles nobody means that
//            nobody left can reach u*: if v still could, some vertex on its
//            chain of jumps would be next to one that reached
//   cycles   the others stand on a cycle or hang off one.  Each marks J of
//            itself; a marked vertex follows the arrows, and if it comes back
//            to itself before meeting a marked vertex of a smaller id, that
//            cycle is popped.  (A mark that is not on a cycle yet, after few
//            jumps on a long path, finds no cycle; a round that pops nothing
//            is followed by one with enough jumps and no bound on the walk.)
// and back to the 2-cycles with the vertices that drew, until all are settled.
//
// LDS (n vertices on the caller's ids, u* = n; 6.25 bytes a vertex):
//   mark   bitmap: marks, or the vertices of the 2-cycle check under way
//   spill  bitmap: draw counts that left 16 bits (their high parts are in
//          global memory, set when the bit is)
//   T      u16 target | settled << 15
//   J      u16 jump; between the jumps the list of vertices that draw again
//   K      u16 low half of the draw count
// A thread owns the vertices tid, tid + T, ...: at most 32, with a bit each in
// a register for "not settled yet".
#include "fc_kernels.hpp"
#include "fc_wave.hpp"

namespace fc {

namespace {

constexpr uint32_t kSettled = 0x8000u;
constexpr uint32_t kIdMask = 0x7FFFu;
constexpr uint32_t kMinJumps = 5;    // passes before marks are worth following
constexpr uint32_t kFullJumps = 16;  // passes that cover any path (n < 2^15)
constexpr uint32_t kWalk = 64;       // arrows a mark follows in an ordinary round
constexpr uint32_t kU = 4;           // vertices a thread keeps in flight

// Offsets in LDS words / u16s for n vertices.
struct JumpLayout {
    uint32_t nb, half;  // words of a bitmap; u16s of T and of J (with u*), even
};
__host__ __device__ inline JumpLayout jump_layout(uint32_t n) {
    return {(n + 31u) >> 5, (n + 2u) & ~1u};
}

template <bool kWeighted>
__global__ __launch_bounds__(1024) void wilson_jump_kernel(CoopArgs a) {
    extern __shared__ uint32_t s_dyn[];
    __shared__ uint32_t s_item, s_cnt, s_flags[4];
    __shared__ unsigned long long s_digest, s_roots;

    const uint32_t T = blockDim.x, tid = threadIdx.x, lane = tid & 63u;
    unsigned int err = 0;

    for (;;) {
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(a.queue, 1u);
        __syncthreads();
        const uint32_t item = uniform(s_item);
        if (item >= a.item_count) break;
        const CoopJob job = a.jobs ? a.jobs[uniform(a.item_job[item])] : a.single;
        const uint32_t ti = item - job.first_item;
        const uint32_t t = job.tree_begin + ti;
        const uint32_t n = job.n;
        const JumpLayout L = jump_layout(n);
        uint32_t *__restrict__ mark = s_dyn;
        uint32_t *__restrict__ spill = s_dyn + L.nb;
        uint16_t *arrow = reinterpret_cast<uint16_t *>(s_dyn + 2u * L.nb);
        uint16_t *jump = arrow + L.half;
        uint16_t *list = jump;
        uint16_t *drawn = jump + L.half;
        uint32_t *__restrict__ high = static_cast<uint32_t *>(a.word) + static_cast<size_t>(blockIdx.x) * a.n_max;

        auto marked = [&](uint32_t v) { return (mark[v >> 5] >> (v & 31u)) & 1u; };
        // Arrow of v from its next draw; the draw count goes up by one.
        auto redraw = [&](uint32_t v) {
            uint32_t k = drawn[v];
            if ((spill[v >> 5] >> (v & 31u)) & 1u) k |= high[v] << 16;
            VRec r = load_vrec(job.vrec, v);
            hold_vrec(r);
            if (k >= a.k_limit) {  // the error ends the tree here: as if v were a root
                err |= kErrVisitOverflow;
                arrow[v] = static_cast<uint16_t>(n | kSettled);
                return;
            }
            const Philox4 x = philox4x32_10(v, k, t, job.stream_id, a.key0, a.key1);
            const uint32_t tg = arrow_target<kWeighted>(r, x.x0, x.x1, job.col_idx, job.wsum, job.wthr, n);
            // a target seen settled settles v: its path to u* is final
            const bool done = tg == n || (arrow[tg] & kSettled);
            arrow[v] = static_cast<uint16_t>(tg | (done ? kSettled : 0u));
            drawn[v] = static_cast<uint16_t>(k + 1u);
            if (((k + 1u) & 0xFFFFu) == 0u) {
                high[v] = (k + 1u) >> 16;
                atomicOr(&spill[v >> 5], 1u << (v & 31u));
            }
        };
        // Appends v to the list (all lanes of the wave call it).
        auto append = [&](uint32_t v, bool pred) {
            const uint64_t m = __ballot(pred);
            if (m == 0ull) return;
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&s_cnt, static_cast<uint32_t>(__popcll(m)));
            base = uniform(base);
            if (pred)
                list[base + static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)))] =
                    static_cast<uint16_t>(v);
        };

        for (uint32_t i = tid; i < 2u * L.nb; i += T) s_dyn[i] = 0u;
        if (tid == 0) {
            s_cnt = 0;
            s_digest = 0;
            s_roots = 0;
            for (uint32_t i = 0; i < 4u; ++i) s_flags[i] = 0;
        }
        // first arrows
        uint32_t open = 0;  // bit i: vertex i T + tid is not settled
        for (uint32_t i0 = 0; i0 * T < n; i0 += kU) {
            VRec r[kU] = {};
            uint32_t tg[kU];
#pragma unroll
            for (uint32_t q = 0; q < kU; ++q) {
                const uint32_t v = (i0 + q) * T + tid;
                if (v < n) r[q] = load_vrec(job.vrec, v);
            }
#pragma unroll
            for (uint32_t q = 0; q < kU; ++q) {
                const uint32_t v = (i0 + q) * T + tid;
                tg[q] = n;
                if (v < n) {
                    const Philox4 x = philox4x32_10(v, 0u, t, job.stream_id, a.key0, a.key1);
                    tg[q] = arrow_target<kWeighted>(r[q], x.x0, x.x1, job.col_idx, job.wsum, job.wthr, n);
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < kU; ++q) {
                const uint32_t v = (i0 + q) * T + tid;
                if (v >= n) continue;
                arrow[v] = static_cast<uint16_t>(tg[q] | (tg[q] == n ? kSettled : 0u));
                drawn[v] = 1;
                if (tg[q] != n) open |= 1u << (i0 + q);
            }
        }
        __syncthreads();
        // 2-cycles of the first arrows: both ends find the pair for themselves
        {
            uint32_t pop = 0;
            for (uint32_t todo = open; todo; todo &= todo - 1u) {
                const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                const uint32_t v = b * T + tid;
                if ((arrow[arrow[v] & kIdMask] & kIdMask) == v) pop |= 1u << b;
            }
            while (__ballot(pop != 0u)) {
                const bool have = pop != 0u;
                append(have ? static_cast<uint32_t>(__builtin_ctz(pop)) * T + tid : 0u, have);
                pop &= pop - 1u;
            }
        }
        __syncthreads();
        unsigned long long draws = n;
        uint32_t rounds = 0;
        bool full = false;
        uint32_t cur = 0, ccur = uniform(s_cnt);  // the list's vertices that draw: [cur, cur + ccur)
        bool done = false;
        for (;;) {
            // pop what is listed, then the 2-cycles that the new arrows close
            while (ccur > 0u) {
                for (uint32_t i = tid; i < ccur; i += T) {
                    const uint32_t v = list[cur + i];
                    redraw(v);
                    atomicOr(&mark[v >> 5], 1u << (v & 31u));
                }
                draws += ccur;
                if (tid == 0) s_cnt = 0;
                __syncthreads();
                if (draws > job.step_cap) break;
                // pairs go to the larger part of the list that is free; pairs that
                // find no room there wait for the cycle search
                const uint32_t after = n + 1u - (cur + ccur);
                const uint32_t nxt = after >= cur ? cur + ccur : 0u;
                const uint32_t cap = after >= cur ? after : cur;
                for (uint32_t i0 = tid - lane; i0 < ccur; i0 += T) {
                    uint32_t u = 0, w = 0;
                    bool pair = false;
                    if (i0 + lane < ccur) {
                        u = list[cur + i0 + lane];
                        w = arrow[u];
                        if (!(w & kSettled)) {
                            w &= kIdMask;
                            // the pair belongs to its smaller end if both drew
                            pair = (arrow[w] & kIdMask) == u && (!marked(w) || u < w);
                        }
                    }
                    const uint64_t m = __ballot(pair);
                    if (m == 0ull) continue;
                    uint32_t base = 0;
                    if (lane == 0) base = atomicAdd(&s_cnt, 2u * static_cast<uint32_t>(__popcll(m)));
                    base = uniform(base) + 2u * static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)));
                    if (pair && base + 2u <= cap) {
                        list[nxt + base] = static_cast<uint16_t>(u);
                        list[nxt + base + 1u] = static_cast<uint16_t>(w);
                    }
                }
                __syncthreads();
                for (uint32_t i = tid; i < ccur; i += T) {
                    const uint32_t v = list[cur + i];
                    atomicAnd(&mark[v >> 5], ~(1u << (v & 31u)));
                }
                ccur = min(uniform(s_cnt), cap & ~1u);
                cur = nxt;
                __syncthreads();  // s_cnt is read, the marks are gone
            }
            if (++rounds > a.max_rounds || draws > job.step_cap) {
                err |= kErrStepCap;
                break;
            }
            // jumps; settled vertices are never anybody's jump
            for (uint32_t todo = open; todo; todo &= todo - 1u) {
                const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                const uint32_t v = b * T + tid;
                const uint32_t w = arrow[v];
                bool reached = (w & kSettled) != 0u;
                uint32_t to = w & kIdMask;
                if (!reached && (arrow[to] & kSettled)) {
                    reached = true;
                    arrow[v] = static_cast<uint16_t>(w | kSettled);
                }
                if (reached) {  // others may jump here before they see it settled
                    to = n;
                    open &= ~(1u << b);
                }
                jump[v] = static_cast<uint16_t>(to);
            }
            __syncthreads();
            for (uint32_t p = 0;; ++p) {
                bool settled = false;
                for (uint32_t todo = open; todo;) {
                    uint32_t b[kU], j[kU];
                    uint32_t have = 0;
#pragma unroll
                    for (uint32_t q = 0; q < kU; ++q) {
                        b[q] = 0;
                        j[q] = n;
                        if (todo) {
                            b[q] = static_cast<uint32_t>(__builtin_ctz(todo));
                            todo &= todo - 1u;
                            have |= 1u << q;
                            j[q] = jump[b[q] * T + tid];
                        }
                    }
#pragma unroll
                    for (uint32_t q = 0; q < kU; ++q)
                        if (have & (1u << q)) j[q] = jump[j[q]];
#pragma unroll
                    for (uint32_t q = 0; q < kU; ++q)
                        if (have & (1u << q)) {
                            const uint32_t v = b[q] * T + tid;
                            jump[v] = static_cast<uint16_t>(j[q]);
                            if (j[q] == n) {
                                arrow[v] = static_cast<uint16_t>(arrow[v] | kSettled);
                                open &= ~(1u << b[q]);
                                settled = true;
                            }
                        }
                }
                // bit 0: somebody is open, bit 1: somebody was settled in this pass
                const uint32_t f = (__ballot(open != 0u) ? 1u : 0u) | (__ballot(settled) ? 2u : 0u);
                if (lane == 0 && f) atomicOr(&s_flags[p & 3u], f);
                __syncthreads();
                const uint32_t all = uniform(s_flags[p & 3u]);
                if (tid == 0) s_flags[(p + 2u) & 3u] = 0;
                if (!(all & 1u)) {
                    done = true;
                    break;
                }
                if (!(all & 2u) && p + 1u >= (full ? kFullJumps : kMinJumps)) break;
            }
            __syncthreads();
            if (tid < 4u) s_flags[tid] = 0;
            if (done) break;
            // marks, then walks
            for (uint32_t todo = open; todo; todo &= todo - 1u) {
                const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                const uint32_t c = jump[b * T + tid];
                atomicOr(&mark[c >> 5], 1u << (c & 31u));
            }
            if (tid == 0) s_cnt = 0;
            __syncthreads();
            const uint32_t bound = full ? n + 1u : kWalk;
            for (uint32_t todo = open; todo; todo &= todo - 1u) {
                const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                const uint32_t c = b * T + tid;
                if (!marked(c)) continue;
                uint32_t x = arrow[c] & kIdMask, len = 1;
                while (x != c && len < bound && !(x < c && marked(x))) {
                    x = arrow[x] & kIdMask;
                    ++len;
                }
                if (x != c) continue;
                uint32_t at = atomicAdd(&s_cnt, len);
                do {
                    list[at++] = static_cast<uint16_t>(x);
                    x = arrow[x] & kIdMask;
                } while (x != c);
            }
            __syncthreads();
            for (uint32_t i = tid; i < L.nb; i += T) mark[i] = 0u;
            cur = 0;
            ccur = uniform(s_cnt);
            if (full && ccur == 0u) {  // cannot be: some cycle is left and its marks close it
                err |= kErrStepCap;
                break;
            }
            full = ccur == 0u;
            __syncthreads();
        }
        __syncthreads();
        if (err & kErrStepCap) break;

        unsigned long long my_digest = 0, my_roots = 0;
        for (uint32_t v = tid; v < n; v += T) {
            const uint32_t to = arrow[v] & kIdMask;
            my_digest += mix64((static_cast<unsigned long long>(v) << 32) | to);
            if (to == n) {
                ++my_roots;
                atomicAdd(&job.root_counts[v], 1u);
            }
            const size_t at = static_cast<size_t>(ti) * n + v;
            if (job.parents) job.parents[at] = static_cast<int32_t>(to);
            if (job.visit_counts || job.tree_visits) {
                uint32_t k = drawn[v];
                if ((spill[v >> 5] >> (v & 31u)) & 1u) k |= high[v] << 16;
                if (job.visit_counts)
                    atomicAdd(&job.visit_counts[v], static_cast<unsigned long long>(k));
                if (job.tree_visits) job.tree_visits[at] = k;
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            my_digest += __shfl_down(my_digest, off, 64);
            my_roots += __shfl_down(my_roots, off, 64);
        }
        if (lane == 0) {
            atomicAdd(&s_digest, my_digest);
            atomicAdd(&s_roots, my_roots);
        }
        __syncthreads();
        if (tid == 0) {
            if (job.tree_digests) job.tree_digests[ti] = s_digest;
            if (job.tree_steps) job.tree_steps[ti] = draws;
            atomicAdd(&a.totals->walk_steps, draws);
            atomicAdd(&a.totals->roots, s_roots);
            atomicAdd(&a.totals->digest_sum, s_digest);
        }
    }
    if (err) atomicOr(&a.totals->error, err);
}

const void *jump_kernel_of(bool weighted) {
    return weighted ? reinterpret_cast<const void *>(&wilson_jump_kernel<true>)
                    : reinterpret_cast<const void *>(&wilson_jump_kernel<false>);
}

}  // namespace

size_t jump_lds_bytes(uint32_t n) {
    const JumpLayout L = jump_layout(n);
    return 8u * static_cast<size_t>(L.nb) + 2u * (2u * static_cast<size_t>(L.half) + n);
}

hipError_t jump_set_limit(size_t bytes) {
    for (bool w : {false, true}) {
        const hipError_t e = hipFuncSetAttribute(jump_kernel_of(w), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(bytes));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int jump_max_active(uint32_t threads, size_t lds, bool weighted) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, jump_kernel_of(weighted),
                                                     static_cast<int>(threads), lds) != hipSuccess)
        return 0;
    return blocks;
}

hipError_t launch_wilson_jump(const CoopArgs &a, uint32_t threads, size_t lds, bool weighted,
                              hipStream_t stream) {
    if (a.n_max == 0 || a.item_count == 0 || a.slots == 0) return hipSuccess;
    if (a.n_max > kJumpMax || a.n_max > kJumpOwn * threads || lds < jump_lds_bytes(a.n_max))
        return hipErrorInvalidValue;
    void *args[] = {const_cast<CoopArgs *>(&a)};
    return hipLaunchKernel(jump_kernel_of(weighted), dim3(a.slots), dim3(threads), args, lds, stream);
}

}  // namespace fc
