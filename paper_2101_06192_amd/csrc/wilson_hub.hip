// Workgroup-per-tree sampler that settles the vertices of highest degree first.
//
// Cycle popping in an order of its own (the tree and every draw count are the same in
// any order).  Ids are relabelled highest degrees first, and every vertex's first
// arrow of the tree is drawn ahead.
//
// 1. Hubs.  The ids [0, hot) and whatever their arrows lead to are popped in LDS by
//    2-cycles, pointer jumping and cycle walks (wilson_jump.hip says how, and why it
//    finds every cycle).  A vertex outside that an arrow leads to joins the set: it is
//    claimed in st and gets the next local id.  So the set is closed, and ends settled.
//    (When it is full, an arrow to a newcomer ends its path there, undecided.)
// 2. Stream.  All vertices are read once in id order: the tree's outputs are counted,
//    and a vertex whose arrow goes to u* or to a settled vertex is settled, for good.
//    With the hubs settled that is most of them, at 8 bytes each.
// 3. List.  The others are gone through again, as (vertex, target) pairs, as long as
//    enough of them settle; when too few do, the 2-cycles among them are popped.
// 4. Sets.  As soon as the list fits the LDS arrays it finishes there like the hubs; when
//    few 2-cycles are left in a longer one, its first vertices do, with what they lead
//    to, and step 3 goes on.  (Where even 64 of them lead to more than fits, the cycles
//    that a peel of the in-arrow counts leaves are popped instead.)
//    A vertex drawn again after the stream corrects the outputs by itself.
//
// What bounds it: R-MAT of 2^22 vertices, alpha 1, 512 trees, two on each CU after the
// other, 20.3 ms (108 ms with in-arrow counts, and 300 bytes of lists, counts and words
// a vertex and tree moved over memory): first arrows 3.8 ms, Philox and 8 bytes
// written; hubs 0.9 ms, waits for one draw's loads after the other; stream 4.7 ms
// (8.3 before its loads went ahead by one step, the root counts to internal ids and the
// settled bits of a step were read together) and
// list 8.2 ms (9.4 before), latency and bandwidth of the arrows and pairs read and written; sets
// 1.9 ms.  130 per mille of a set are hubs at the start: with 100 the list takes longer
// (+0.8 ms), with 160 sets come close to full (-0.8 ms; with 300 they are, twice the
// time).  The list is read in id order, hubs first: backwards every other time it
// settles less, 17.8 ms.  One workgroup a CU with the widest set: two with half of it
// +10 ms.
//
// LDS in steps 1 and 4 as in wilson_tile.hip (6.4 bytes a vertex of the set); in 2 and
// 3 the settled bits of the lowest ids, as many as fit.
// Global, per tree slot (n vertices):
//   cur[v]  u64  the current arrow: internal target | original target << 32 (the
//                tree's own pre-drawn array, or the slot's)
//   st[v]   u64  epoch << 47 | id in the set << 31 | arrows drawn: of the vertices that
//                were in a set of this tree (epoch: the slot's set number)
//   lists   u64  (vertex, target) pairs: two lists and the peel order / pops
//   pc      u32  in-arrow counts of a peel
//   vid     u32  ids of a set's members, then the same with their outcome
//   gbits        settled bits: of the ids beyond those in LDS, and of all in step 4
// Per job: rint, the root counts on internal ids.
#include "fc_kernels.hpp"
#include "fc_wave.hpp"

namespace fc {

namespace {

constexpr uint32_t kRoot = 0x7FFFu;   // T: the arrow goes to u* or a vertex settled before
constexpr uint32_t kExt = 0x7FFEu;    // T: the arrow leaves the full set
constexpr uint32_t kAgain = 0x8000u;  // T: drawn more than once, or claimed
constexpr uint32_t kDone = 0x8000u;   // J: the end of the path is known
constexpr uint32_t kIdMask = 0x7FFFu;
constexpr uint32_t kMinJumps = 4;   // passes before marks are tried
constexpr uint32_t kMoreJumps = 3;  // and after some were not on a cycle
constexpr uint32_t kU = 4, kD = 2;  // vertices a thread keeps in flight: jumping, drawing
constexpr uint32_t kWalk = 96;      // arrows a walk to the next vertex that drew again may take
constexpr uint32_t kFewPairs = 64;  // 2-cycles of the first arrows: fewer vertices wait for the cycles
constexpr uint32_t kLowBits = 8;
constexpr int kS = 4, kR = 4, kP = 1;  // vertices a lane keeps in flight: stream, list, pops
constexpr uint32_t kNobody = 0xFFFFFFFFu;
constexpr uint32_t kLeastSeeds = 64;  // of a longer list, the vertices a set starts with, at least
constexpr uint32_t kEpochs = 1u << 17;  // values of a set's number
constexpr uint32_t kDrawMask = 0x7FFFFFFFu;

__device__ __forceinline__ uint32_t lo32(uint64_t w) { return static_cast<uint32_t>(w); }
__device__ __forceinline__ uint32_t hi32(uint64_t w) { return static_cast<uint32_t>(w >> 32); }
__device__ __forceinline__ uint64_t pair(uint32_t v, uint32_t tg) {
    return static_cast<uint64_t>(v) | (static_cast<uint64_t>(tg) << 32);
}

// LDS of a set of up to cap vertices (a multiple of 64), in words from the start.
struct SetLayout {
    uint32_t nb;                       // words of a bitmap
    uint32_t arrow, jump, list, cap;   // cap: entries of the list
    uint32_t drawn, words;
};
__host__ __device__ inline SetLayout set_layout(uint32_t set) {
    SetLayout L{};
    L.nb = set >> 5;
    L.arrow = 3u * L.nb;
    L.jump = L.arrow + (set >> 1);
    L.list = L.jump + (set >> 1);
    L.cap = set >> 1;
    L.drawn = L.list + (set >> 2);
    L.words = L.drawn + (set >> 2);
    return L;
}

// Per-phase clock sums: first arrows (when not drawn ahead), hubs: first arrows and
// claims, redraws, jumps, cycles; stream; list; rest.
enum Phase : int { kPhDraw = 0, kPhClaim, kPhPop, kPhJump, kPhCycle, kPhStream, kPhList, kPhRest,
                   kPhNum };

// Arrow number k of the vertex with (relabelled) record r in tree t:
// internal | original target (u* = n in both).
template <bool kWeighted>
__device__ __forceinline__ uint64_t hub_draw(const CoopJob &j, const VRec &r, uint32_t key0,
                                             uint32_t key1, uint32_t k, uint32_t t) {
    const uint32_t orig = r.always_root & 0x7FFFFFFFu;
    const Philox4 x = philox4x32_10(orig, k, t, j.stream_id, key0, key1);
    if ((r.always_root >> 31) || x.x0 < r.thr) return pair(j.n, j.n);
    const uint32_t idx = neighbour_entry<kWeighted>(r, x.x1, j.wsum, j.wthr);
    return j.adj[r.start + static_cast<int32_t>(idx)];
}

template <bool kWeighted>
__global__ __launch_bounds__(1024) void wilson_hub_kernel(CoopArgs a) {
    extern __shared__ uint32_t s_dyn[];
    __shared__ uint32_t s_item, s_u, s_c, s_cnt, s_over, s_set, s_ext, s_flags[4];
    __shared__ unsigned long long s_digest, s_roots;
    __shared__ unsigned long long s_ph[kPhNum + 1];

    const uint32_t T = blockDim.x;
    const uint32_t tid = threadIdx.x;
    const uint32_t wave_base = tid & ~63u;
    const uint32_t lane = tid & 63u;
    const size_t slot = blockIdx.x;
    const size_t stride = a.n_max;
    const SetLayout L = set_layout(a.set);
    uint32_t *__restrict__ mark = s_dyn;
    uint32_t *__restrict__ hit = s_dyn + L.nb;
    uint32_t *__restrict__ spill = s_dyn + 2u * L.nb;
    uint16_t *arrow = reinterpret_cast<uint16_t *>(s_dyn + L.arrow);
    uint16_t *jump = reinterpret_cast<uint16_t *>(s_dyn + L.jump);
    uint16_t *__restrict__ list = reinterpret_cast<uint16_t *>(s_dyn + L.list);
    uint8_t *__restrict__ drawn = reinterpret_cast<uint8_t *>(s_dyn + L.drawn);
    unsigned long long *const st = reinterpret_cast<unsigned long long *>(a.kk) + slot * stride;
    uint64_t *__restrict__ listA = a.lists + slot * (3ull * stride);
    uint64_t *__restrict__ listB = listA + stride;
    uint64_t *__restrict__ peel = listB + stride;
    uint32_t *__restrict__ pc = a.levels + slot * stride;
    uint32_t *__restrict__ vid = a.origt + slot * (2ull * a.set);
    uint32_t *__restrict__ fin = vid + a.set;
    uint32_t *const gbits = a.bits + slot * ((stride + 31u) >> 5);

    unsigned int err = 0;
    uint32_t epoch = 0;  // the slot's set number, from 1 (st is zero at launch)
    uint32_t iso_job = kNobody;
    unsigned long long iso_digest = 0;  // this thread's part, of the isolated vertices of iso_job
    const bool timing = a.phase_ticks != nullptr;
    if (tid == 0) s_over = 0;
    if (timing && tid == 0) {
        for (int i = 0; i < kPhNum; ++i) s_ph[i] = 0;
        s_ph[kPhNum] = wall_clock64();
    }
    auto mark_time = [&](int which) {
        if (timing && tid == 0) {
            const unsigned long long now = wall_clock64();
            s_ph[which] += now - s_ph[kPhNum];
            s_ph[kPhNum] = now;
        }
    };

    for (;;) {
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(a.queue, 1u);
        __syncthreads();
        const uint32_t item = uniform(s_item);
        if (item >= a.item_count) break;
        const CoopJob job = a.jobs ? a.jobs[uniform(a.item_job[item])] : a.single;
        const uint32_t ti = item - job.first_item;
        const uint32_t t = job.tree_begin + ti;
        const uint32_t n = job.n;      // also the id of u*
        const uint32_t nl = job.n3;    // ids [0, nl) are not isolated
        // ids [0, hot) are the hubs
        const uint32_t hot = nl <= a.set ? nl : a.set * a.hub_hot / 1000u;
        const uint32_t nb = (nl + 31u) >> 5;
        const uint32_t lb = min(nb, a.lds_bits >> 5);  // words of the bitmap that are in LDS
        uint64_t *__restrict__ cur = a.pre ? a.pre + static_cast<size_t>(item) * stride
                                           : static_cast<uint64_t *>(a.word) + slot * stride;
        if (epoch > kEpochs - kEpochs / 8u) {
            for (size_t i = tid; i < stride; i += T) st[i] = 0ull;
            epoch = 0;
            __syncthreads();
        }
        const uint32_t before_tree = epoch;
        unsigned long long draws = n;  // arrows drawn in this tree
        unsigned long long my_digest = 0, my_roots = 0;
        if (tid == 0) {
            s_digest = 0;
            s_roots = 0;
        }
        if (!a.pre) {  // first arrows
            for (uint32_t v0 = tid; v0 < nl; v0 += kD * T) {
                VRec r[kD];
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q)
                    if (v0 + q * T < nl) r[q] = load_vrec(job.vrec, v0 + q * T);
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q)
                    if (v0 + q * T < nl)
                        cur[v0 + q * T] = hub_draw<kWeighted>(job, r[q], a.key0, a.key1, 0u, t);
            }
            __syncthreads();
            mark_time(kPhDraw);
        }
        // Vertex v (original id ov) drew its arrow number k anew after the stream: the
        // outputs had the one before.
        auto correct = [&](uint32_t v, uint32_t ov, uint64_t was, uint64_t now, uint32_t k) {
            const unsigned long long hi = static_cast<unsigned long long>(ov) << 32;
            my_digest += mix64(hi | hi32(now)) - mix64(hi | hi32(was));
            if (lo32(now) == n) {
                ++my_roots;
                atomicAdd(&job.rint[v], 1u);
            }
            const size_t at = static_cast<size_t>(ti) * n + ov;
            if (job.parents) job.parents[at] = static_cast<int32_t>(hi32(now));
            if (job.visit_counts) atomicAdd(&job.visit_counts[ov], 1ull);
            if (job.tree_visits) job.tree_visits[at] = k + 1u;
        };
        auto draws_in = [&](unsigned long long s) -> uint32_t {  // arrows drawn, of an st entry
            return static_cast<uint32_t>(s >> 47) > before_tree ? lo32(s) & kDrawMask : 1u;
        };
        auto local_in = [&](unsigned long long s) -> uint32_t {
            return static_cast<uint32_t>(s >> 31) & 0xFFFFu;
        };
        auto settled = [&](uint32_t v) -> bool {  // steps 2 and 3
            if (v >= nl) return true;
            const uint32_t w = v >> 5;
            return ((w < lb ? s_dyn[w] : gbits[w]) >> (v & 31u)) & 1u;
        };
        // The same of several vertices, none of them left out: their words on the way
        // together, without branches where all bits are in LDS.
        auto settled_all = [&](const auto &v, auto &is) {
            constexpr int kN = static_cast<int>(sizeof(v) / sizeof(v[0]));
            uint32_t word[kN];
            bool far = false;
#pragma unroll
            for (int q = 0; q < kN; ++q) {
                const uint32_t x = min(v[q] >> 5, nb);
                far |= x >= lb && x < nb;
                word[q] = s_dyn[min(x, lb - 1u)];
            }
            if (__ballot(far)) {
#pragma unroll
                for (int q = 0; q < kN; ++q) {
                    const uint32_t x = v[q] >> 5;
                    if (x >= lb && x < nb) word[q] = gbits[x];
                }
            }
#pragma unroll
            for (int q = 0; q < kN; ++q) is[q] = v[q] >= nl || ((word[q] >> (v[q] & 31u)) & 1u);
        };
        auto settle = [&](uint32_t v) {
            const uint32_t w = v >> 5, bit = 1u << (v & 31u);
            if (w < lb) atomicOr(&s_dyn[w], bit);
            else (void)__hip_atomic_fetch_or(&gbits[w], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };

        // Cycle popping inside a set held in LDS, of b vertices to begin with: the hubs
        // (ids [0, b)), or (res) those in vid, with their st entries set.
        uint64_t *U = listA, *Unext = listB;
        unsigned long long tag = 0;
        auto pop_set = [&](uint32_t b, bool res, int ph_claim, int ph_pop, int ph_jump, int ph_cycle) {
            auto marked = [&](uint32_t i) { return (mark[i >> 5] >> (i & 31u)) & 1u; };
            auto id_of = [&](uint32_t i) -> uint32_t { return !res && i < b ? i : vid[i]; };
            // T of an arrow to tg
            auto code_of = [&](uint32_t tg) -> uint32_t {
                if (tg == n) return kRoot;
                if (!res && tg < b) return tg;
                const unsigned long long s = st[tg];
                if (res && ((gbits[tg >> 5] >> (tg & 31u)) & 1u)) return kRoot;
                if (static_cast<uint32_t>(s >> 47) == epoch) return local_in(s);
                const uint32_t i = atomicAdd(&s_set, 1u);  // claim it
                if (i >= a.set) {
                    s_ext = 1u;
                    return kExt;
                }
                const unsigned long long mine = tag | (static_cast<unsigned long long>(i) << 31) | draws_in(s);
                unsigned long long seen = s;
                if (__hip_atomic_compare_exchange_strong(&st[tg], &seen, mine, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
                    vid[i] = tg;
                    jump[i] = 0;
                    return i;
                }
                vid[i] = kNobody;  // another lane was first: the local id stays unused
                arrow[i] = static_cast<uint16_t>(kRoot);
                jump[i] = static_cast<uint16_t>(kDone | kRoot);
                return local_in(seen);
            };
            uint32_t have = 0;  // vertices of the set whose arrows are known
            auto set_arrow = [&](uint32_t i, uint32_t code, uint32_t again) {
                arrow[i] = static_cast<uint16_t>(code | again);
                if (code == kRoot) jump[i] = static_cast<uint16_t>(kDone | kRoot);
                else if (code == kExt) jump[i] = static_cast<uint16_t>(kDone | i);
            };
            // Arrows of set vertices at[0..m) from their next draws; the draw counts go
            // up by one.  The loads of kD draws are in flight together.
            auto redraw = [&](const uint32_t (&at)[kD], uint32_t m) {
                uint32_t k[kD], v[kD];
                uint64_t was[kD], now[kD];
                VRec r[kD];
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q) v[q] = q < m ? id_of(at[q]) : 0u;
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q) {
                    k[q] = 0;
                    was[q] = 0;
                    r[q] = {};
                    if (q >= m) continue;
                    const uint32_t i = at[q];
                    if (res) {
                        k[q] = lo32(st[v[q]]) & kDrawMask;
                        was[q] = cur[v[q]];
                    } else {
                        k[q] = drawn[i];
                        if ((spill[i >> 5] >> (i & 31u)) & 1u) k[q] |= lo32(st[v[q]]) << kLowBits;
                    }
                    r[q] = load_vrec(job.vrec, v[q]);
                }
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q) {
                    now[q] = pair(n, n);
                    if (q >= m) continue;
                    hold_vrec(r[q]);  // (its original id goes into Philox)
                    now[q] = hub_draw<kWeighted>(job, r[q], a.key0, a.key1, k[q], t);
                }
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q) {
                    if (q >= m) continue;
                    const uint32_t i = at[q];
                    if (k[q] >= a.k_limit) {  // the error ends the tree here: as if v were a root
                        err |= kErrVisitOverflow;
                        set_arrow(i, kRoot, kAgain);
                        continue;
                    }
                    cur[v[q]] = now[q];
                    const uint32_t code = code_of(lo32(now[q]));
                    set_arrow(i, code, kAgain);
                    if (code < have) {  // a target whose end is known: its path is final
                        const uint32_t j = jump[code];
                        if (j & kDone) jump[i] = static_cast<uint16_t>(j);
                    }
                    const unsigned long long where = tag | (static_cast<unsigned long long>(i) << 31);
                    if (res) {
                        correct(v[q], r[q].always_root & 0x7FFFFFFFu, was[q], now[q], k[q]);
                        st[v[q]] = where | (k[q] + 1u);
                    } else {
                        drawn[i] = static_cast<uint8_t>(k[q] + 1u);
                        if (((k[q] + 1u) & ((1u << kLowBits) - 1u)) == 0u) {
                            st[v[q]] = where | ((k[q] + 1u) >> kLowBits);
                            atomicOr(&spill[i >> 5], 1u << (i & 31u));
                        }
                    }
                }
            };
            // Appends the pair (u, w) at list[base + ...], of which cap entries are free
            // (all lanes of the wave call it); without room there it is left alone.
            auto append_pair = [&](uint32_t base, uint32_t cap, uint32_t u, uint32_t w, bool pred) {
                const uint64_t m = __ballot(pred);
                if (m == 0ull) return;
                uint32_t off = 0;
                if (lane == 0) off = atomicAdd(&s_cnt, 2u * static_cast<uint32_t>(__popcll(m)));
                off = uniform(off) + 2u * static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)));
                if (pred && off + 2u <= cap) {
                    list[base + off] = static_cast<uint16_t>(u);
                    list[base + off + 1u] = static_cast<uint16_t>(w);
                }
            };

            // First arrows of the vertices claimed since, and of those that they claim.
            auto grow = [&]() {
                for (;;) {
                    const uint32_t upto = min(uniform(s_set), a.set);
                    __syncthreads();  // everybody has read it
                    if (have >= upto) break;
                    for (uint32_t i = have + tid; i < upto; i += T) {
                        const uint32_t v = id_of(i);
                        if (v == kNobody) continue;
                        drawn[i] = 1;
                        const uint32_t code = code_of(lo32(cur[v]));
                        if (i < b) jump[i] = 0;
                        set_arrow(i, code, i < b ? 0u : kAgain);
                    }
                    have = upto;
                    __syncthreads();
                }
            };

            for (uint32_t i = tid; i < 3u * L.nb; i += T) s_dyn[i] = 0u;
            if (tid == 0) {
                s_cnt = 0;
                s_set = b;
                s_ext = 0;
            }
            if (tid < 4u) s_flags[tid] = 0;
            __syncthreads();
            uint32_t open = 0;  // bit q: the path of vertex q T + tid has no known end
            uint32_t seen = 0;  // vertices of the set that open covers
            grow();
            auto cover = [&]() {
                for (uint32_t q = seen / T; q * T + tid < have; ++q)
                    if (q * T + tid >= seen && !(jump[q * T + tid] & kDone)) open |= 1u << q;
                seen = have;
            };
            cover();
            mark_time(ph_claim);
            // 2-cycles of the first arrows, each listed by its smaller end
            {
                uint32_t pop = 0;
                for (uint32_t todo = open; todo; todo &= todo - 1u) {
                    const uint32_t q = static_cast<uint32_t>(__builtin_ctz(todo));
                    const uint32_t i = q * T + tid, w = arrow[i] & kIdMask;
                    if (i < w && (arrow[w] & kIdMask) == i) pop |= 1u << q;
                }
                while (__ballot(pop != 0u)) {
                    const bool some = pop != 0u;
                    const uint32_t u = some ? static_cast<uint32_t>(__builtin_ctz(pop)) * T + tid : 0u;
                    append_pair(0u, L.cap, u, some ? arrow[u] & kIdMask : 0u, some);
                    pop &= pop - 1u;
                }
            }
            __syncthreads();
            uint32_t rounds = 0;
            bool wide = true;  // this round's jumps go over all open vertices
            uint32_t head = 0, ccur = min(uniform(s_cnt), L.cap);  // list entries that draw
            bool done = false;
            __syncthreads();
            for (;;) {
                // pop what is listed, then the 2-cycles that the new arrows close
                while (ccur > (wide ? kFewPairs : 0u)) {
                    for (uint32_t j = tid; j < ccur; j += kD * T) {
                        uint32_t at[kD], m = 0;
#pragma unroll
                        for (uint32_t q = 0; q < kD; ++q) {
                            at[q] = 0;
                            if (j + q * T < ccur) {
                                at[q] = list[head + j + q * T];
                                m = q + 1u;
                            }
                        }
                        redraw(at, m);
#pragma unroll
                        for (uint32_t q = 0; q < kD; ++q)
                            if (q < m) atomicOr(&mark[at[q] >> 5], 1u << (at[q] & 31u));
                    }
                    draws += ccur;
                    if (tid == 0) s_cnt = 0;
                    __syncthreads();
                    grow();
                    if (draws > job.step_cap) break;
                    // pairs go to the larger part of the list that is free; pairs that
                    // find no room there wait for the cycle search
                    const uint32_t after = L.cap - (head + ccur);
                    const uint32_t nxt = after >= head ? head + ccur : 0u;
                    const uint32_t room = (after >= head ? after : head) & ~1u;
                    for (uint32_t j0 = wave_base; j0 < ccur; j0 += T) {
                        uint32_t u = 0, w = 0;
                        bool pair = false;
                        if (j0 + lane < ccur) {
                            u = list[head + j0 + lane];
                            w = arrow[u] & kIdMask;
                            // the pair belongs to its smaller end if both drew
                            if (w < kExt)
                                pair = (arrow[w] & kIdMask) == u && (!marked(w) || u < w);
                        }
                        append_pair(nxt, room, u, w, pair);
                    }
                    __syncthreads();
                    for (uint32_t j = tid; j < ccur; j += T) {
                        const uint32_t i = list[head + j];
                        atomicAnd(&mark[i >> 5], ~(1u << (i & 31u)));
                    }
                    ccur = min(uniform(s_cnt), room);
                    head = nxt;
                    __syncthreads();  // s_cnt is read, the marks are gone
                }
                cover();
                mark_time(ph_pop);
                if (++rounds > a.max_rounds || draws > job.step_cap) {
                    err |= kErrStepCap;
                    return;
                }
                // where each vertex's jumps start
                uint32_t work;  // the vertices of this round
                for (;;) {
                    work = open;
                    bool deep = false;
                    for (uint32_t todo = open; todo; todo &= todo - 1u) {
                        const uint32_t bit = todo & (0u - todo);
                        const uint32_t i = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                        const uint32_t c = arrow[i];
                        if (!wide && !(c & kAgain)) {
                            work &= ~bit;
                            continue;
                        }
                        uint32_t x = jump[i];
                        if (!(x & kDone)) {
                            uint32_t to = c & kIdMask;
                            x = jump[to];
                            if (!wide) {
                                uint32_t steps = 0;
                                for (uint32_t y = arrow[to]; !(x & kDone) && !(y & kAgain);) {
                                    if (++steps > kWalk) break;
                                    to = y;
                                    x = jump[to];
                                    y = arrow[to];
                                }
                                deep |= steps > kWalk;
                            }
                            jump[i] = static_cast<uint16_t>(x & kDone ? x : to);
                        }
                        if (x & kDone) {
                            open &= ~bit;
                            work &= ~bit;
                        }
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
                uint32_t total = 0;  // vertices on cycles
                for (;;) {
                    for (uint32_t p = 0;; ++p) {
                        bool settled = false;
                        for (uint32_t todo = work; todo;) {
                            uint32_t q[kU], j[kU];
#pragma unroll
                            for (uint32_t h = 0; h < kU; ++h) {
                                q[h] = 32u;
                                j[h] = 0;
                                if (todo) {
                                    q[h] = static_cast<uint32_t>(__builtin_ctz(todo));
                                    todo &= todo - 1u;
                                    j[h] = jump[q[h] * T + tid];
                                }
                            }
#pragma unroll
                            for (uint32_t h = 0; h < kU; ++h)
                                if (q[h] < 32u) j[h] = jump[j[h]];
#pragma unroll
                            for (uint32_t h = 0; h < kU; ++h)
                                if (q[h] < 32u) {
                                    jump[q[h] * T + tid] = static_cast<uint16_t>(j[h]);
                                    if (j[h] & kDone) {
                                        open &= ~(1u << q[h]);
                                        work &= ~(1u << q[h]);
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
                    mark_time(ph_jump);
                    if (done) break;
                    for (uint32_t todo = work; todo; todo &= todo - 1u) {
                        const uint32_t c = jump[static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid];
                        atomicOr(&mark[c >> 5], 1u << (c & 31u));
                    }
                    __syncthreads();
                    uint32_t mine = 0;  // the vertices of this thread that are marked
                    for (uint32_t todo = work; todo; todo &= todo - 1u) {
                        const uint32_t q = static_cast<uint32_t>(__builtin_ctz(todo));
                        if (marked(q * T + tid)) mine |= 1u << q;
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
                    if (!again) {  // list the cycles
                        for (uint32_t todo = mine; todo; todo &= todo - 1u) {
                            const uint32_t c = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                            uint32_t x = c, len = 0;
                            do {
                                x = arrow[x] & kIdMask;
                                ++len;
                            } while (!marked(x));
                            uint32_t at = atomicAdd(&s_cnt, len);
                            if (at + len > L.cap) continue;
                            x = c;
                            do {
                                list[at++] = static_cast<uint16_t>(x);
                                x = arrow[x] & kIdMask;
                            } while (--len);
                        }
                        __syncthreads();
                        total = uniform(s_cnt);
                        if (total > L.cap) {
                            // no room for all of them: each thread pops the stretches from
                            // its marks on as it walks (the marks stay until all are done)
                            for (uint32_t todo = mine; todo; todo &= todo - 1u) {
                                uint32_t x = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                                do {
                                    const uint32_t y = arrow[x] & kIdMask;
                                    uint32_t at[kD] = {x};
                                    redraw(at, 1u);
                                    x = y;
                                } while (!marked(x));
                            }
                        }
                    }
                    __syncthreads();
                    for (uint32_t i = tid; i < 2u * L.nb; i += T) mark[i] = 0u;  // and hit
                    if (tid == 0) s_flags[3] = 0;
                    if (!again) break;
                    least = kMoreJumps;
                    __syncthreads();
                }
                if (done) break;
                if (total == 0u) {  // cannot be: somebody is left, so is a cycle
                    err |= kErrStepCap;
                    return;
                }
                head = 0;
                ccur = total;
                if (total > L.cap) {
                    ccur = 0;
                    draws += total;
                }
                __syncthreads();
                grow();
                mark_time(ph_cycle);
                wide = false;
            }
            __syncthreads();
            if (!uniform(s_ext)) return;
            // the set was full: where the paths end that hang off those the last rounds settled
            for (uint32_t todo = open; todo; todo &= todo - 1u) {
                const uint32_t i = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                if (jump[i] & kDone) open &= ~(todo & (0u - todo));
                else jump[i] = static_cast<uint16_t>(arrow[i] & kIdMask);
            }
            __syncthreads();
            for (uint32_t p = 0;; ++p) {  // ends: every path leads to a known exit
                for (uint32_t todo = open; todo; todo &= todo - 1u) {
                    const uint32_t i = static_cast<uint32_t>(__builtin_ctz(todo)) * T + tid;
                    const uint32_t x = jump[jump[i]];
                    jump[i] = static_cast<uint16_t>(x);
                    if (x & kDone) open &= ~(todo & (0u - todo));
                }
                if (__ballot(open != 0u) && lane == 0) s_flags[p & 3u] = 1u;
                __syncthreads();
                const bool more = uniform(s_flags[p & 3u]) != 0u;
                if (tid == 0) s_flags[(p + 2u) & 3u] = 0;
                if (!more) break;
            }
            mark_time(ph_jump);
        };

        // Sets, and what goes on between them.  The settled bits are in LDS but while a
        // set is there.
        uint32_t b = hot, ucount = 0, rounds = 0, seeds = max(a.set >> 3, kLeastSeeds);
        bool hubs = true, peels = false;
        for (;;) {
            if (++epoch == kEpochs) {
                err |= kErrStepCap;
                break;
            }
            tag = static_cast<unsigned long long>(epoch) << 47;
            if (!hubs) {
                __syncthreads();
                for (uint32_t i = tid; i < lb; i += T) gbits[i] = s_dyn[i];
                for (uint32_t i = tid; i < b; i += T) {
                    const uint32_t v = lo32(U[i]);
                    vid[i] = v;
                    st[v] = tag | (static_cast<unsigned long long>(i) << 31) | draws_in(st[v]);
                }
                __syncthreads();
            }
            pop_set(b, !hubs, hubs ? kPhClaim : kPhRest, hubs ? kPhPop : kPhRest,
                    hubs ? kPhJump : kPhRest, hubs ? kPhCycle : kPhRest);
            if (err & kErrStepCap) break;
            const bool full = uniform(s_ext) != 0u;
            if (!hubs && !full && b == ucount) break;
            const uint32_t members = min(uniform(s_set), a.set);
            for (uint32_t i = tid; i < members; i += T) {
                const uint32_t v = hubs && i < hot ? i : vid[i];
                fin[i] = kNobody;
                if (v == kNobody) continue;
                if (hubs) {
                    uint32_t k = drawn[i];
                    if ((spill[i >> 5] >> (i & 31u)) & 1u) k |= (lo32(st[v]) & kDrawMask) << kLowBits;
                    st[v] = tag | (static_cast<unsigned long long>(i) << 31) | k;
                }
                if (!full || (jump[i] & kIdMask) == kRoot) fin[i] = v;
            }
            __syncthreads();
            for (uint32_t i = tid; i < lb; i += T) s_dyn[i] = hubs ? 0u : gbits[i];
            if (hubs)
                for (uint32_t i = lb + tid; i < nb; i += T) gbits[i] = 0u;
            if (tid == 0) s_u = 0;
            __syncthreads();
            for (uint32_t i = tid; i < members; i += T)
                if (fin[i] != kNobody) settle(fin[i]);
            __syncthreads();
            mark_time(hubs ? kPhCycle : kPhRest);
            bool stale = true;
            if (hubs) {
                // 2. the stream: outputs, and every vertex whose target is settled
                const bool want_k = job.visit_counts || job.tree_visits;
                uint64_t w_ahead[kS];  // (loaded one step ahead)
                uint32_t ov_ahead[kS];
#pragma unroll
                for (int q = 0; q < kS; ++q) {
                    const uint32_t v = wave_base + q * T + lane;
                    w_ahead[q] = v < nl ? cur[v] : 0ull;
                    ov_ahead[q] = v < nl ? job.orig[v] : 0u;
                }
                for (uint32_t base = wave_base; base < nl; base += kS * T) {
                    uint64_t w[kS];
                    uint32_t ov[kS], to[kS];
                    bool left[kS], ends[kS];
#pragma unroll
                    for (int q = 0; q < kS; ++q) {
                        const uint32_t v = base + (kS + q) * T + lane;
                        w[q] = w_ahead[q];
                        ov[q] = ov_ahead[q];
                        w_ahead[q] = v < nl ? cur[v] : 0ull;
                        ov_ahead[q] = v < nl ? job.orig[v] : 0u;
                    }
#pragma unroll
                    for (int q = 0; q < kS; ++q) to[q] = lo32(w[q]);
                    settled_all(to, ends);
#pragma unroll
                    for (int q = 0; q < kS; ++q) {
                        const uint32_t v0 = base + q * T, v = v0 + lane;
                        left[q] = false;
                        if (v < nl) {
                            left[q] = !ends[q] && !settled(v);
                            my_digest += mix64((static_cast<unsigned long long>(ov[q]) << 32) | hi32(w[q]));
                            if (to[q] == n) {
                                ++my_roots;
                                atomicAdd(&job.rint[v], 1u);
                            }
                            const size_t at = static_cast<size_t>(ti) * n + ov[q];
                            if (job.parents) job.parents[at] = static_cast<int32_t>(hi32(w[q]));
                            if (want_k) {
                                const uint32_t k = draws_in(st[v]);
                                if (job.visit_counts)
                                    atomicAdd(&job.visit_counts[ov[q]], static_cast<unsigned long long>(k));
                                if (job.tree_visits) job.tree_visits[at] = k;
                            }
                        }
                        // (the wave's own two words of the bitmap)
                        const uint64_t now = __ballot(v < nl && !left[q]);
                        if ((lane == 0u || lane == 32u) && v0 + lane < nl) {
                            const uint32_t x = (v0 + lane) >> 5, bits = static_cast<uint32_t>(now >> lane);
                            if (x < lb) s_dyn[x] = bits;
                            else gbits[x] = bits;
                        }
                        w[q] = pair(v, lo32(w[q]));
                    }
                    wave_append_many<kS>(U, &s_u, nl, &s_over, w, left);
                }
                __syncthreads();
                mark_time(kPhStream);
                ucount = min(uniform(s_u), nl);
                hubs = stale = false;
            } else if (full) {
                peels = b <= kLeastSeeds;
                seeds = max(min(seeds, b) >> 2, kLeastSeeds);
            }

            // 3. the list, until it fits LDS or a set is due
            b = 0;
            while (ucount > 0u && b == 0u) {
                if (ucount <= a.set && !stale) {
                    b = ucount;
                    break;
                }
                if (++rounds > a.max_rounds || draws > job.step_cap || s_over) {
                    err |= kErrStepCap;
                    break;
                }
                __syncthreads();
                if (tid == 0) s_u = 0;
                __syncthreads();
                for (uint32_t base = wave_base; base < ucount; base += kR * T) {
                    uint64_t e[kR];
                    bool left[kR];
#pragma unroll
                    for (int q = 0; q < kR; ++q) {
                        const uint32_t i = base + q * T + lane;
                        e[q] = i < ucount ? U[i] : 0ull;
                    }
#pragma unroll
                    for (int q = 0; q < kR; ++q)
                        if (stale && base + q * T + lane < ucount) e[q] = pair(lo32(e[q]), lo32(cur[lo32(e[q])]));
                    uint32_t to[kR];
                    bool ends[kR];
#pragma unroll
                    for (int q = 0; q < kR; ++q) to[q] = hi32(e[q]);
                    settled_all(to, ends);
#pragma unroll
                    for (int q = 0; q < kR; ++q) {
                        const bool in = base + q * T + lane < ucount &&
                                        !(stale && settled(lo32(e[q])));
                        left[q] = in && !ends[q];
                        if (in && ends[q]) settle(lo32(e[q]));
                    }
                    wave_append_many<kR>(Unext, &s_u, nl, &s_over, e, left);
                }
                __syncthreads();
                const uint32_t before = ucount;
                ucount = min(uniform(s_u), nl);
                uint64_t *const spent = U;
                U = Unext;
                Unext = spent;
                stale = false;
                if (ucount <= a.set || ucount <= before - (before >> 3)) continue;
                // too few settled: the others hang off cycles, many of them 2-cycles
                __syncthreads();
                if (tid == 0) {
                    s_u = 0;
                    s_c = 0;
                }
                __syncthreads();
                for (uint32_t base = wave_base; base < ucount; base += kR * T) {
                    uint64_t e[kR];
                    bool two[kR], left[kR];
#pragma unroll
                    for (int q = 0; q < kR; ++q) {
                        const uint32_t i = base + q * T + lane;
                        e[q] = i < ucount ? U[i] : 0ull;
                    }
#pragma unroll
                    for (int q = 0; q < kR; ++q) {
                        const bool ok = base + q * T + lane < ucount;
                        two[q] = ok && lo32(cur[hi32(e[q])]) == lo32(e[q]);
                        left[q] = ok && !two[q];
                    }
                    wave_append_many<kR>(peel, &s_c, nl, &s_over, e, two);
                    wave_append_many<kR>(Unext, &s_u, nl, &s_over, e, left);
                }
                __syncthreads();
                uint32_t pops = min(uniform(s_c), nl);
                if (pops < T && !peels) {  // too few: a set, unless none is small enough
                    b = min(ucount, seeds);
                } else if (pops == 0u) {
                    peels = false;
                    // none: peel what has no in-arrow, what is left stands on cycles
                    for (uint32_t i = tid; i < ucount; i += T) pc[lo32(U[i])] = 0u;
                    __syncthreads();
                    if (tid == 0) {
                        s_c = 0;
                        s_u = 0;
                    }
                    for (uint32_t i = tid; i < ucount; i += T) {
                        const uint32_t to = hi32(U[i]);
                        if (!settled(to)) atomicAdd(&pc[to], 1u);
                    }
                    __syncthreads();
                    for (uint32_t base = wave_base; base < ucount; base += T) {
                        uint64_t e[1] = {0ull};
                        bool leaf[1] = {false};
                        if (base + lane < ucount) {
                            e[0] = U[base + lane];
                            leaf[0] = pc[lo32(e[0])] == 0u;
                        }
                        wave_append_many<1>(peel, &s_c, nl, &s_over, e, leaf);
                    }
                    __syncthreads();
                    uint32_t lo = 0, hi = min(uniform(s_c), nl);
                    __syncthreads();  // s_c is read
                    while (lo < hi) {
                        for (uint32_t base = lo + wave_base; base < hi; base += T) {
                            uint64_t e[1] = {0ull};
                            bool push[1] = {false};
                            if (base + lane < hi) {
                                const uint32_t to = hi32(peel[base + lane]);
                                if (!settled(to) && atomicSub(&pc[to], 1u) == 1u) {
                                    e[0] = pair(to, lo32(cur[to]));
                                    push[0] = true;
                                }
                            }
                            wave_append_many<1>(peel, &s_c, nl, &s_over, e, push);
                        }
                        __syncthreads();
                        lo = hi;
                        hi = min(uniform(s_c), nl);
                        __syncthreads();
                    }
                    if (tid == 0) s_c = 0;
                    __syncthreads();
                    for (uint32_t base = wave_base; base < ucount; base += T) {
                        uint64_t e[1] = {0ull};
                        bool on[1] = {false}, left[1] = {false};
                        if (base + lane < ucount) {
                            e[0] = U[base + lane];
                            on[0] = pc[lo32(e[0])] != 0u;
                            left[0] = !on[0];
                        }
                        wave_append_many<1>(peel, &s_c, nl, &s_over, e, on);
                        wave_append_many<1>(Unext, &s_u, nl, &s_over, e, left);
                    }
                    __syncthreads();
                    pops = min(uniform(s_c), nl);
                }
                for (uint32_t base = wave_base; base < pops; base += kP * T) {
                    uint32_t v[kP], k[kP];
                    uint64_t was[kP], e[kP];
                    VRec r[kP];
                    bool ok[kP], left[kP];
#pragma unroll
                    for (int q = 0; q < kP; ++q) {
                        ok[q] = base + q * T + lane < pops;
                        v[q] = ok[q] ? lo32(peel[base + q * T + lane]) : 0u;
                    }
#pragma unroll
                    for (int q = 0; q < kP; ++q) {
                        r[q] = load_vrec(job.vrec, v[q]);
                        was[q] = cur[v[q]];
                        k[q] = draws_in(st[v[q]]);
                    }
#pragma unroll
                    for (int q = 0; q < kP; ++q) {
                        hold_vrec(r[q]);
                        e[q] = hub_draw<kWeighted>(job, r[q], a.key0, a.key1, k[q], t);
                    }
#pragma unroll
                    for (int q = 0; q < kP; ++q) {
                        left[q] = false;
                        if (!ok[q]) continue;
                        if (k[q] >= a.k_limit) {
                            err |= kErrVisitOverflow;
                            e[q] = pair(n, n);
                        }
                        correct(v[q], r[q].always_root & 0x7FFFFFFFu, was[q], e[q], k[q]);
                        cur[v[q]] = e[q];
                        st[v[q]] = tag | (k[q] + 1u);
                        e[q] = pair(v[q], lo32(e[q]));
                        left[q] = !settled(hi32(e[q]));
                        if (!left[q]) settle(v[q]);
                    }
                    wave_append_many<kP>(Unext, &s_u, nl, &s_over, e, left);
                }
                draws += pops;
                __syncthreads();
                ucount = min(uniform(s_u), nl);
                uint64_t *const was = U;
                U = Unext;
                Unext = was;
                if (b > 0u) b = ucount <= a.set ? ucount : min(b, ucount);
            }
            if (err & kErrStepCap) break;
            mark_time(kPhList);
            if (b == 0u) break;
        }
        if (err & kErrStepCap) break;
        if (draws > job.step_cap) {
            err |= kErrStepCap;
            break;
        }
        // isolated vertices: roots of every tree after one draw (counted for all
        // trees of the job by the workgroup of its first one)
        if (iso_job != job.first_item) {
            iso_job = job.first_item;
            iso_digest = 0;
            for (uint32_t v = nl + tid; v < n; v += T)
                iso_digest += mix64((static_cast<unsigned long long>(job.orig[v]) << 32) | n);
        }
        my_digest += iso_digest;
        if (tid == 0) my_roots += n - nl;
        if (ti == 0u)
            for (uint32_t v = nl + tid; v < n; v += T) {
                atomicAdd(&job.root_counts[job.orig[v]], job.tree_count);
                if (job.visit_counts)
                    atomicAdd(&job.visit_counts[job.orig[v]],
                              static_cast<unsigned long long>(job.tree_count));
            }
        if (job.parents || job.tree_visits)
            for (uint32_t v = nl + tid; v < n; v += T) {
                const size_t at = static_cast<size_t>(ti) * n + job.orig[v];
                if (job.parents) job.parents[at] = static_cast<int32_t>(n);
                if (job.tree_visits) job.tree_visits[at] = 1u;
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
        mark_time(kPhRest);
    }
    if (timing && tid == 0)
        for (int i = 0; i < kPhNum; ++i) atomicAdd(&a.phase_ticks[i], s_ph[i]);
    if (s_over) err |= kErrStepCap;
    if (err) atomicOr(&a.totals->error, err);
}

// First arrows of all trees ahead: each thread owns one vertex and draws in `trees`
// trees, so its record and row are read once for them.  Rows of up to kPreRow entries
// (without weights) wait in LDS, a column for each thread: drawn from memory, the 64
// lines of a wave's draw are as many requests to the L2, which held it to 165 G draws/s
// on R-MAT of 2^22 vertices (6.3 ms for 512 trees; with rows of 8 5.4, of 16 5.0, of 24
// 4.4, of 32, where too few waves fit, 4.6; with 256 trees instead of 64 after a row is
// there 3.8).
constexpr uint32_t kPreTrees = 256, kPreBlocks = 2048;  // trees at most; blocks wanted
constexpr uint32_t kPreThreads = 256;
constexpr uint32_t kPreRow = 24;

template <bool kWeighted>
__global__ __launch_bounds__(kPreThreads) void hub_predraw_kernel(CoopArgs a, uint32_t trees,
                                                                  uint32_t groups) {
    __shared__ unsigned long long s_row[kWeighted ? 1 : kPreRow][kPreThreads];
    const CoopJob &j = a.single;
    const uint32_t v = blockIdx.x * kPreThreads + threadIdx.x;
    if (v >= j.n3) return;
    const VRec r = load_vrec(j.vrec, v);
    const bool near = !kWeighted && r.deg <= kPreRow;
    if (near)
        for (uint32_t i = 0; i < r.deg; ++i) s_row[i][threadIdx.x] = j.adj[r.start + static_cast<int32_t>(i)];
    for (uint32_t g = blockIdx.y; g < groups; g += gridDim.y) {
#pragma unroll 4
        for (uint32_t q = 0; q < trees; ++q) {
            const uint32_t item = g * trees + q;
            if (item >= a.item_count) break;
            const uint32_t orig = r.always_root & 0x7FFFFFFFu;
            const Philox4 x = philox4x32_10(orig, 0u, j.tree_begin + item, j.stream_id, a.key0, a.key1);
            uint64_t w = pair(j.n, j.n);
            if (!(r.always_root >> 31) && x.x0 >= r.thr) {
                const uint32_t idx = neighbour_entry<kWeighted>(r, x.x1, j.wsum, j.wthr);
                w = near ? s_row[idx][threadIdx.x] : j.adj[r.start + static_cast<int32_t>(idx)];
            }
            a.pre[static_cast<size_t>(item) * a.n_max + v] = w;
        }
    }
}

// Root counts back on original ids.  The trees count them by internal id, where the
// stream's 64 lanes add to one or two lines of memory instead of up to 64 (R-MAT of
// 2^22 vertices, 512 trees: 27.3 ms with the counts on original ids, 25.4 so).
__global__ __launch_bounds__(256) void hub_counts_kernel(CoopArgs a) {
    const CoopJob job = a.jobs ? a.jobs[blockIdx.y] : a.single;
    for (uint32_t v = blockIdx.x * 256u + threadIdx.x; v < job.n3; v += gridDim.x * 256u) {
        const uint32_t c = job.rint[v];
        if (c) atomicAdd(&job.root_counts[job.orig[v]], c);
    }
}

const void *hub_kernel_of(bool weighted) {
    return weighted ? reinterpret_cast<const void *>(&wilson_hub_kernel<true>)
                    : reinterpret_cast<const void *>(&wilson_hub_kernel<false>);
}

}  // namespace

size_t hub_lds_bytes(uint32_t set) { return 4u * static_cast<size_t>(set_layout(set).words); }

hipError_t hub_set_limit(size_t bytes) {
    for (bool w : {false, true}) {
        const hipError_t e = hipFuncSetAttribute(hub_kernel_of(w), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(bytes));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int hub_max_active(uint32_t threads, size_t lds, bool weighted) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, hub_kernel_of(weighted),
                                                     static_cast<int>(threads), lds) != hipSuccess)
        return 0;
    return blocks;
}

hipError_t launch_hub_counts(const CoopArgs &a, uint32_t count, uint32_t n_max, hipStream_t stream) {
    if (count == 0 || n_max == 0) return hipSuccess;
    const uint32_t blocks = (n_max + 255u) / 256u;
    const uint32_t step = 65535u;
    for (uint32_t j = 0; j < count; j += step) {
        CoopArgs part = a;
        if (a.jobs) part.jobs = a.jobs + j;
        const dim3 grid(blocks < 2048u ? blocks : 2048u, count - j < step ? count - j : step);
        hub_counts_kernel<<<grid, 256, 0, stream>>>(part);
    }
    return hipGetLastError();
}

hipError_t launch_hub_predraw(const CoopArgs &a, hipStream_t stream) {
    if (!a.pre || a.single.n3 == 0 || a.item_count == 0) return hipSuccess;
    // vertex tiles a multiple of 8 wide: block b of every tree group then runs on
    // XCD b mod 8, whose L2 keeps that tile's records and adjacency rows
    uint32_t tiles = (a.single.n3 + kPreThreads - 1) / kPreThreads;
    tiles = (tiles + 7u) & ~7u;
    // as many trees a block as leave enough blocks (and 16 at least)
    uint32_t trees = static_cast<uint32_t>(static_cast<uint64_t>(a.item_count) * tiles / kPreBlocks);
    trees = trees < 16u ? 16u : trees > kPreTrees ? kPreTrees : trees;
    const uint32_t groups = (a.item_count - 1u) / trees + 1u;
    const dim3 grid(tiles, groups < 65535u ? groups : 65535u);
    if (a.single.wsum) hub_predraw_kernel<true><<<grid, kPreThreads, 0, stream>>>(a, trees, groups);
    else hub_predraw_kernel<false><<<grid, kPreThreads, 0, stream>>>(a, trees, groups);
    return hipGetLastError();
}

hipError_t launch_wilson_hub(const CoopArgs &a, uint32_t threads, size_t lds, bool weighted,
                             hipStream_t stream) {
    if (a.n_max == 0 || a.item_count == 0 || a.slots == 0) return hipSuccess;
    if (a.set == 0 || a.set % 64u || a.set > kHubOwn * threads || a.set > kHubMax ||
        a.lds_bits % 32u || a.hub_hot > 1000u || lds < hub_lds_bytes(a.set) || lds < a.lds_bits / 8u)
        return hipErrorInvalidValue;
    void *args[] = {const_cast<CoopArgs *>(&a)};
    return hipLaunchKernel(hub_kernel_of(weighted), dim3(a.slots), dim3(threads), args, lds, stream);
}

}  // namespace fc
