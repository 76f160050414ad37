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
//            itself, and every marked vertex follows the arrows to the next
//            marked one.  If that map takes the marks onto all of themselves,
//            they all stand on cycles, and the paths walked are the cycles
//            whole: all of them are popped.  A mark that nobody walked to is
//            still on its way to a cycle (few jumps, long path): then a few
//            more jumps, and marks and walks again.  (Every cycle holds marks:
//            its own vertices' jumps stay on it.)
// and back to the 2-cycles with the vertices that drew, until all are settled.
//
// The jumps go over all unsettled vertices once.  After that every unsettled
// vertex that has drawn only once hangs, over others of its kind, off one that
// has drawn again: a cycle that forms later passes through one of those.  So the
// later rounds jump among the vertices that have drawn again alone, from the
// first of their kind that their arrows lead to (found by walking there), and
// the tree is finished when these are settled.  Where such a walk would be long
// (deep forests), the round jumps over all unsettled vertices again.
//
// What bounds it: small trees the latency of their passes, about 2 us for one that
// draws (list, draw count, record and neighbour, arrow, then the check) and 0.9 us for
// one that jumps; a tree of 20000 vertices on a CU of its own 16 us Philox, 22 us jumps
// (seven passes of random 2-byte LDS accesses), 13 us redraws, 8 us outputs.  Measured
// against in-arrow counts and a peel: 64 trees of 1000 vertices (Erdos-Renyi) 107 us
// then, 35 us now; 64 of BA(20000, 5) 197 and 67; 4096 of R-MAT(20000) at alpha 10
// 10.6 ms and 3.3.  Threads: as many as a CU's trees leave room for (jump_threads_for);
// one wave a tree, without barriers, was slower (56 us).
//
// LDS (n vertices on the caller's ids, u* = n; 6.4 bytes a vertex):
//   mark   bitmap: marks, or the vertices of the 2-cycle check under way
//   hit    bitmap: marks that a walk ended at
//   spill  bitmap: draw counts that left 15 bits (their high parts are in
//          global memory, set when the bit is)
//   T      u16 target | settled << 15
//   J      u16 jump; between the jumps the list of vertices that draw again
//   K      u16 low 15 bits of the draw count | drawn again << 15
// A thread owns the vertices tid, tid + T, ...: at most 32, with a bit each in
// a register for "not settled yet".
#include "fc_kernels.hpp"
#include "fc_wave.hpp"

namespace fc {

namespace {

constexpr uint32_t kSettled = 0x8000u;
constexpr uint32_t kIdMask = 0x7FFFu;
constexpr uint32_t kMinJumps = 4;   // passes before marks are tried
constexpr uint32_t kMoreJumps = 3;  // and after some were not on a cycle
constexpr uint32_t kU = 4, kD = 2;  // vertices a thread keeps in flight: jumping, drawing
constexpr uint32_t kWalk = 96;      // arrows a walk to the next vertex that drew again may take
constexpr uint32_t kAgain = 0x8000u;
constexpr uint32_t kLowBits = 15;

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

    if (failed(a.check)) return;
    const uint32_t T = blockDim.x, tid = threadIdx.x, lane = tid & 63u;
    unsigned int err = 0;
    // The totals and the queue are one line of memory for all workgroups, 12 ns an
    // addition: thread 0 keeps the totals and adds them once at the end, the first
    // tree is the workgroup's own number, and the next one is asked for while the
    // outputs are written.  (Four additions a tree took 200 of the 217 us of 4096
    // trees of 1000 vertices.)
    unsigned long long all_draws = 0, all_roots = 0, all_digests = 0;
    if (tid == 0) s_item = blockIdx.x;

    for (;;) {
        __syncthreads();
        const uint32_t item = uniform(s_item);
        if (item >= a.item_count) break;
        const CoopJob job = a.jobs ? a.jobs[uniform(a.item_job[item])] : a.single;
        const uint32_t ti = item - job.first_item;
        const uint32_t t = job.tree_begin + ti;
        const uint32_t n = job.n;
        const JumpLayout L = jump_layout(n);
        uint32_t *__restrict__ mark = s_dyn;
        uint32_t *__restrict__ hit = s_dyn + L.nb;
        uint32_t *__restrict__ spill = s_dyn + 2u * L.nb;
        uint16_t *arrow = reinterpret_cast<uint16_t *>(s_dyn + 3u * L.nb);
        uint16_t *jump = arrow + L.half;
        uint16_t *list = jump;
        uint16_t *drawn = jump + L.half;
        uint32_t *__restrict__ high = static_cast<uint32_t *>(a.word) + static_cast<size_t>(blockIdx.x) * a.n_max;

        auto marked = [&](uint32_t v) { return (mark[v >> 5] >> (v & 31u)) & 1u; };
        auto draws_of = [&](uint32_t v) {
            uint32_t k = drawn[v] & (kAgain - 1u);
            if ((spill[v >> 5] >> (v & 31u)) & 1u) k |= high[v] << kLowBits;
            return k;
        };
        // Arrow of v from its next draw; the draw count goes up by one.
        auto redraw = [&](uint32_t v) {
            const uint32_t k = draws_of(v);
            VRec r = load_vrec(job.vrec, v);  // on its way during the Philox rounds
            const Philox4 x = philox4x32_10(v, k, t, job.stream_id, a.key0, a.key1);
            hold_vrec(r);
            if (k >= a.k_limit) {  // the error ends the tree here: as if v were a root
                err |= kErrVisitOverflow;
                arrow[v] = static_cast<uint16_t>(n | kSettled);
                return;
            }
            const uint32_t tg = arrow_target<kWeighted>(r, x.x0, x.x1, job.col_idx, job.wsum, job.wthr, n);
            // a target seen settled settles v: its path to u* is final
            const bool done = tg == n || (arrow[tg] & kSettled);
            arrow[v] = static_cast<uint16_t>(tg | (done ? kSettled : 0u));
            drawn[v] = static_cast<uint16_t>(((k + 1u) & (kAgain - 1u)) | kAgain);
            if (((k + 1u) & (kAgain - 1u)) == 0u) {
                high[v] = (k + 1u) >> kLowBits;
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

        for (uint32_t i = tid; i < 3u * L.nb; i += T) s_dyn[i] = 0u;
        if (tid == 0) {
            s_cnt = 0;
            s_digest = 0;
            s_roots = 0;
            for (uint32_t i = 0; i < 4u; ++i) s_flags[i] = 0;
        }
        // first arrows
        uint32_t open = 0;  // bit i: vertex i T + tid is not settled
        for (uint32_t i0 = 0; i0 * T < n; i0 += kD) {
            VRec r[kD] = {};
            uint32_t tg[kD];
#pragma unroll
            for (uint32_t q = 0; q < kD; ++q) {
                const uint32_t v = (i0 + q) * T + tid;
                if (v < n) r[q] = load_vrec(job.vrec, v);
            }
#pragma unroll
            for (uint32_t q = 0; q < kD; ++q) {
                const uint32_t v = (i0 + q) * T + tid;
                tg[q] = n;
                if (v < n) {
                    const Philox4 x = philox4x32_10(v, 0u, t, job.stream_id, a.key0, a.key1);
                    tg[q] = arrow_target<kWeighted>(r[q], x.x0, x.x1, job.col_idx, job.wsum, job.wthr, n);
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < kD; ++q) {
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
        bool wide = true;  // this round's jumps go over all unsettled vertices
        uint32_t cur = 0, ccur = uniform(s_cnt);  // the list's vertices that draw: [cur, cur + ccur)
        bool done = false;
        __syncthreads();  // s_cnt is read
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
            // where each vertex's jumps start; settled vertices are never anybody's jump
            uint32_t work;  // the vertices of this round
            for (;;) {
                work = open;
                if (!wide)
                    for (uint32_t todo = open; todo; todo &= todo - 1u) {
                        const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                        if (!(drawn[b * T + tid] & kAgain)) work &= ~(1u << b);
                    }
                bool deep = false;
                for (uint32_t todo = work; todo; todo &= todo - 1u) {
                    const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                    const uint32_t v = b * T + tid;
                    const uint32_t w = arrow[v];
                    bool reached = (w & kSettled) != 0u;
                    uint32_t to = w & kIdMask;
                    if (!reached) {
                        uint32_t x = arrow[to];
                        if (!wide) {
                            uint32_t steps = 0;
                            for (uint32_t d = drawn[to]; !(x & kSettled) && !(d & kAgain);) {
                                if (++steps > kWalk) break;
                                to = x & kIdMask;
                                x = arrow[to];
                                d = drawn[to];
                            }
                            deep |= steps > kWalk;
                        }
                        reached = (x & kSettled) != 0u;
                        if (reached) arrow[v] = static_cast<uint16_t>(w | kSettled);
                    }
                    if (reached) {  // others may jump here before they see it settled
                        to = n;
                        open &= ~(1u << b);
                        work &= ~(1u << b);
                    }
                    jump[v] = static_cast<uint16_t>(to);
                }
                if (wide) break;
                if (__ballot(deep) && lane == 0) s_flags[3] = 1u;
                __syncthreads();
                wide = uniform(s_flags[3]) != 0u;
                if (!wide) break;
                __syncthreads();
                if (tid == 0) s_flags[3] = 0;
            }
            __syncthreads();
            // jumps until a pass settles nobody, marks, walks to the next mark; where
            // some mark turns out not to be on a cycle, a few more jumps
            uint32_t least = kMinJumps;
            for (;;) {
                for (uint32_t p = 0;; ++p) {
                    bool settled = false;
                    for (uint32_t todo = work; todo;) {
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
                                    work &= ~(1u << b[q]);
                                    settled = true;
                                }
                            }
                    }
                    // bit 0: somebody is left, bit 1: somebody was settled in this pass
                    const uint32_t f = (__ballot(work != 0u) ? 1u : 0u) | (__ballot(settled) ? 2u : 0u);
                    if (lane == 0 && f) atomicOr(&s_flags[p & 3u], f);
                    __syncthreads();
                    const uint32_t all = uniform(s_flags[p & 3u]);
                    if (tid == 0) s_flags[(p + 2u) & 3u] = 0;
                    if (!(all & 1u)) {
                        done = true;
                        break;
                    }
                    if (!(all & 2u) && p + 1u >= least) break;
                }
                __syncthreads();
                if (tid < 4u) s_flags[tid] = 0;
                if (done) break;
                for (uint32_t todo = work; todo; todo &= todo - 1u) {
                    const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                    const uint32_t c = jump[b * T + tid];
                    atomicOr(&mark[c >> 5], 1u << (c & 31u));
                }
                __syncthreads();
                uint32_t mine = 0;  // the vertices of this thread that are marked
                for (uint32_t todo = work; todo; todo &= todo - 1u) {
                    const uint32_t b = static_cast<uint32_t>(__builtin_ctz(todo));
                    if (marked(b * T + tid)) mine |= 1u << b;
                }
                for (uint32_t todo = mine; todo; todo &= todo - 1u) {
                    uint32_t x = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                    do {  // ends: the arrows lead to a cycle, which holds a mark
                        x = arrow[x] & kIdMask;
                    } while (!marked(x));
                    atomicOr(&hit[x >> 5], 1u << (x & 31u));
                }
                __syncthreads();
                bool stray = false;
                for (uint32_t todo = mine; todo; todo &= todo - 1u) {
                    const uint32_t c = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                    stray |= !((hit[c >> 5] >> (c & 31u)) & 1u);
                }
                if (__ballot(stray) && lane == 0) s_flags[3] = 1u;
                if (tid == 0) s_cnt = 0;
                __syncthreads();
                const bool again = uniform(s_flags[3]) != 0u;
                if (!again)  // the jumps are not needed any more: list the cycles there
                    for (uint32_t todo = mine; todo; todo &= todo - 1u) {
                        const uint32_t c = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                        uint32_t x = c, len = 0;
                        do {
                            x = arrow[x] & kIdMask;
                            ++len;
                        } while (!marked(x));
                        uint32_t at = atomicAdd(&s_cnt, len);
                        x = c;
                        do {
                            list[at++] = static_cast<uint16_t>(x);
                            x = arrow[x] & kIdMask;
                        } while (--len);
                    }
                __syncthreads();
                for (uint32_t i = tid; i < 2u * L.nb; i += T) mark[i] = 0u;  // and hit
                if (tid == 0) s_flags[3] = 0;
                if (!again) break;
                least = kMoreJumps;
                __syncthreads();
            }
            if (done) break;
            cur = 0;
            ccur = uniform(s_cnt);
            if (ccur == 0u) {  // cannot be: somebody is left, so is a cycle
                err |= kErrStepCap;
                break;
            }
            __syncthreads();
            wide = false;
        }
        __syncthreads();
        if (err & kErrStepCap) break;

        uint32_t next = a.item_count;
        if (tid == 0 && a.item_count > gridDim.x) next = gridDim.x + atomicAdd(a.queue, 1u);
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
                const uint32_t k = draws_of(v);
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
            all_draws += draws;
            all_roots += s_roots;
            all_digests += s_digest;
            s_item = next;
        }
    }
    if (tid == 0 && all_draws) {
        atomicAdd(&a.totals->walk_steps, all_draws);
        atomicAdd(&a.totals->roots, all_roots);
        atomicAdd(&a.totals->digest_sum, all_digests);
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
    return 12u * static_cast<size_t>(L.nb) + 2u * (2u * static_cast<size_t>(L.half) + n);
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
