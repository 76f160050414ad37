// Workgroup-per-tree sampler for graphs whose vertex ids are local (road
// networks, grids: most edges join ids that are close), by tile-local cycle
// popping.
//
// Wilson's cycle-popping theorem (the tree and every per-vertex arrow count
// are the same whatever order the cycles of the top arrows are popped in)
// lets one workgroup pop a tree's cycles in any grouping.  Here:
//
// 1. Tiles.  The ids are cut into tiles of B consecutive vertices, handled
//    one after another, whole in LDS: draws, 2-cycles, pointer jumping and cycle
//    pops as in the small-graph sampler (wilson_jump.hip says how, and why it
//    finds every cycle), where an arrow out of the tile ends a path as one to u*
//    does.  Every vertex of the tile then has an exit: the last tile vertex on
//    its path (whose arrow leaves the tile), or "settled" when the path reaches
//    u* inside the tile.  The tile's part of the outputs is written at once;
//    what the residual changes later, it corrects.
// 2. Exit graph.  On the exit vertices the map u -> ex[target(u)] is a
//    functional graph whose cycles are exactly the arrows' cycles that cross
//    tiles.  A Kahn peel over the exits (global counters; only exits take
//    part) and a reverse sweep find which exits reach u*.
// 3. Residual.  A vertex is settled exactly when its exit is.  The few
//    vertices that are not (on a crossing cycle or hanging off one) finish
//    as one more LDS set like a tile (numbered in list order, a target
//    settled before counting as u*) once they fit the tile arrays; until
//    then, with the ordinary round-synchronous popping: a settled bitmap (LDS
//    when it fits), global in-arrow counters and lists, only for them.
// No global atomic touches a vertex outside the exit graph and the residual.
//
// What bounds it (grid of 1000 x 1000, 12% of the edges removed, alpha 1, 1024 trees
// on 256 CUs, 40 tiles a tree; 32.1 ms when the tiles were peeled level by level and
// the first arrows drawn ahead by a kernel of their own, 19.6 ms now): first arrows
// 3.5 ms, all of it Philox and so the arithmetic units; redraws 5.0 ms, a chain of 13
// passes a tile that each wait for the loads of one draw (record, then neighbour);
// jumps 3.9 ms and cycles 1.4 ms, LDS; outputs 2.7 ms, the digest's products and the
// root counts' atomics (0.8 ms); exit graph 0.7 ms, residual 2.4 ms.  One workgroup a
// CU with the widest tile: two with tiles half as wide wait as long on each, and cut
// twice as many paths (29.1 ms).
//
// LDS during the tiles (6.4 bytes a vertex):
//   mark, hit, spill  bitmaps: marks (or the vertices of the 2-cycle check under
//             way), marks that a walk ended at, draw counts that left 8 bits
//   T      u16 tile-local target, or kRoot (u*) / kExt (a vertex of another
//              tile), | drawn again << 15
//   J      u16 open: jump; else kDone | the tile-local id of the exit, or kRoot
//   list   u16 vertices that draw again, for half of the tile's vertices (pairs
//              and cycles without room there are popped without it)
//   K      u8  low byte of the draw count (the rest in kk, where spill says so)
// and, once the tiles are done, the exit bitmap and then the settled bitmap,
// when n/8 bytes fit.  A thread owns the set's vertices tid, tid + T, ...: at most
// 32, with a bit each in a register for "open".
// Global, per tree slot:
//   tw[v]  u32  the top arrow's target (u* = n), where it leaves its tile and for
//               the residual
//   tl[v]  u16  its tile-local form (T), ex[v] u16 tile-local id of v's exit, or
//               kRoot: of every vertex once its tile is done
//   kk[v]  u32  arrows drawn, of the vertices not settled within their tile
//   exl    u32  each tile's exit vertices, at offset tile * B; ecnt[tile]
//   pc, sc u32  in-counts (exit graph, residual) and exit successors
//   bl     u32  lists: exits / residual, next residual, peel order
//   lv     u32  peel level bounds
//   xb          exits whose chain reaches u* (LDS when n/8 bytes fit)
//   bits        settled bitmap of the residual rounds (copied into LDS when it
//               fits)
#include "fc_kernels.hpp"
#include "fc_rows.hpp"
#include "fc_wave.hpp"

namespace fc {

namespace {

constexpr uint32_t kRoot = 0x7FFFu;   // T: the arrow goes to u*; ex: the path ends there
constexpr uint32_t kExt = 0x7FFEu;    // T: the arrow leaves the tile
constexpr uint32_t kAgain = 0x8000u;  // T: drawn more than once
constexpr uint32_t kDone = 0x8000u;   // J: the exit is known
constexpr uint32_t kIdMask = 0x7FFFu;
constexpr uint32_t kMinJumps = 4;   // passes before marks are tried
constexpr uint32_t kMoreJumps = 3;  // and after some were not on a cycle
constexpr uint32_t kU = 4, kD = 2;  // vertices a thread keeps in flight: jumping, drawing
constexpr uint32_t kWalk = 96;      // arrows a walk to the next vertex that drew again may take
constexpr uint32_t kFewPairs = 64;  // 2-cycles of the first arrows: fewer vertices wait for the cycles
constexpr uint32_t kLowBits = 8;

// LDS of a set of up to Bp vertices (Bp a multiple of 64), in words from the start.
struct TileLayout {
    uint32_t nb;                       // words of a bitmap
    uint32_t arrow, jump, list, cap;   // cap: entries of the list
    uint32_t drawn, words;
};
__host__ __device__ inline TileLayout tile_layout(uint32_t Bp) {
    TileLayout L{};
    L.nb = Bp >> 5;
    L.arrow = 3u * L.nb;
    L.jump = L.arrow + (Bp >> 1);
    L.list = L.jump + (Bp >> 1);
    L.cap = Bp >> 1;
    L.drawn = L.list + (Bp >> 2);
    L.words = L.drawn + (Bp >> 2);
    return L;
}

// Per-phase clock sums (tid 0 of each workgroup): first arrows, 2-cycles and all
// redraws, jumps, cycle marks and walks, the tiles' exits and outputs, the exit
// graph, the residual, the tree's totals.
enum Phase : int { kPhDraw = 0, kPhPop, kPhJump, kPhCycle, kPhExits, kPhExit, kPhResidual,
                   kPhOutput, kPhNum };

// One arrow of v in tree t with draw index k (original ids; kWeighted: the
// graph may carry running weight sums).
template <bool kWeighted>
__device__ __forceinline__ uint32_t tile_draw(const TileArgs &a, uint32_t v, uint32_t k,
                                              uint32_t t) {
    VRec r = load_vrec(a.vrec, v);
    hold_vrec(r);
    if (r.always_root) return a.n;
    const Philox4 x = philox4x32_10(v, k, t, a.stream_id, a.key0, a.key1);
    return arrow_target<kWeighted>(r, x.x0, x.x1, a.col_idx, a.wsum, a.wthr, a.n);
}

// Appends `item` to a list whose tail counter is in LDS when `pred` holds (one
// LDS atomic per wave); items at or past `cap` are dropped and reported through
// *over.  The position is relative to `base` (list[base + tail]).  Every lane
// of the wave must reach the call.
template <typename T>
__device__ __forceinline__ void wave_push(T *__restrict__ list, uint32_t base, uint32_t *tail,
                                          uint32_t cap, uint32_t *over, T item, bool pred) {
    const uint64_t mask = __ballot(pred);
    if (mask == 0) return;
    const uint32_t lane = __lane_id();
    const uint32_t cnt = static_cast<uint32_t>(__popcll(mask));
    const uint32_t leader = static_cast<uint32_t>(__ffsll(static_cast<unsigned long long>(mask))) - 1u;
    uint32_t off = 0;
    if (lane == leader) {
        off = atomicAdd(tail, cnt);
        if (base + off + cnt > cap) atomicOr(over, 1u);
    }
    off = __shfl(off, static_cast<int>(leader), 64);
    if (pred) {
        const uint32_t at = base + off + static_cast<uint32_t>(__popcll(mask & ((1ull << lane) - 1ull)));
        if (at < cap) list[at] = item;
    }
}

template <bool kWeighted>
__global__ __launch_bounds__(1024) void wilson_tile_kernel(TileArgs a) {
    extern __shared__ uint32_t s_dyn[];
    // s_lc: three rotating tail counters, so that one barrier per peel level
    // suffices (level k appends with counter (k + 1) % 3 while thread 0 clears
    // counter (k + 2) % 3, which everyone read a level ago)
    __shared__ uint32_t s_item, s_u, s_c, s_cnt, s_over, s_lc[3], s_flags[4];
    __shared__ unsigned long long s_digest, s_roots;
    __shared__ unsigned long long s_ph[kPhNum + 1];

    const uint32_t T = blockDim.x;
    const uint32_t tid = threadIdx.x;
    const uint32_t wave_base = tid & ~63u;
    const uint32_t lane = tid & 63u;
    const size_t slot = blockIdx.x;
    const uint32_t n = a.n;
    const uint32_t B = a.B;
    const uint32_t ntiles = a.ntiles;
    const size_t nn = n;
    const uint32_t nw = (n + 31u) >> 5;

    const TileLayout L = tile_layout(a.Bp);
    uint32_t *__restrict__ mark = s_dyn;
    uint32_t *__restrict__ hit = s_dyn + L.nb;
    uint32_t *__restrict__ spill = s_dyn + 2u * L.nb;
    uint16_t *arrow = reinterpret_cast<uint16_t *>(s_dyn + L.arrow);
    uint16_t *jump = reinterpret_cast<uint16_t *>(s_dyn + L.jump);
    uint16_t *__restrict__ list = reinterpret_cast<uint16_t *>(s_dyn + L.list);
    uint8_t *__restrict__ drawn = reinterpret_cast<uint8_t *>(s_dyn + L.drawn);
    uint32_t *const gbits = a.bits + slot * static_cast<size_t>(nw);
    uint32_t *__restrict__ bits = a.bits_lds ? s_dyn : gbits;
    uint32_t *__restrict__ xb = a.xb ? a.xb + slot * static_cast<size_t>(nw) : s_dyn;

    uint32_t *__restrict__ tw = a.tw + slot * nn;
    uint32_t *__restrict__ kk = a.kk + slot * nn;
    uint16_t *__restrict__ tl = a.tl + slot * nn;
    uint16_t *__restrict__ ex = a.ex + slot * ((nn + 7u) & ~static_cast<size_t>(7u));
    uint32_t *__restrict__ exl = a.exl + slot * nn;
    uint32_t *__restrict__ ecnt = a.ecnt + slot * static_cast<size_t>(ntiles);
    uint32_t *__restrict__ pc = a.pc + slot * nn;
    uint32_t *__restrict__ sc = a.sc + slot * nn;
    uint32_t *__restrict__ bU = a.bl + slot * (3ull * nn);
    uint32_t *__restrict__ bN = bU + nn;
    uint32_t *__restrict__ bP = bN + nn;
    uint32_t *__restrict__ lvg = a.lv + slot * (nn + 2u);

    unsigned int err = 0;
    const bool timing = a.phase_ticks != nullptr;
    if (tid == 0) {
        s_over = 0;
        s_lc[0] = s_lc[1] = s_lc[2] = 0;
    }
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
    auto is_settled = [&](uint32_t v) -> bool {
        return v >= n || ((bits[v >> 5] >> (v & 31u)) & 1u);
    };
    auto set_settled = [&](uint32_t v) { atomicOr(&bits[v >> 5], 1u << (v & 31u)); };

    for (;;) {
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(a.queue, 1u);
        __syncthreads();
        const uint32_t item = uniform(s_item);
        if (item >= a.tree_count) break;
        const uint32_t t = a.tree_begin + item;
        unsigned long long draws = n;  // arrows drawn in this tree
        unsigned long long my_digest = 0, my_roots = 0;
        if (tid == 0) {
            s_digest = 0;
            s_roots = 0;
        }
        // A vertex of the residual draws its arrow with index k: the outputs had
        // the one before.
        auto redrawn = [&](uint32_t v, uint32_t was, uint32_t tg, uint32_t k) {
            const unsigned long long hi = static_cast<unsigned long long>(v) << 32;
            my_digest += mix64(hi | tg) - mix64(hi | was);
            if (tg == n) {
                ++my_roots;
                atomicAdd(&a.root_counts[v], 1u);
            }
            if (a.parents) a.parents[static_cast<size_t>(item) * nn + v] = static_cast<int32_t>(tg);
            if (a.visit_counts) atomicAdd(&a.visit_counts[v], 1ull);
            if (a.tree_visits) a.tree_visits[static_cast<size_t>(item) * nn + v] = k + 1u;
            kk[v] = k + 1u;
            tw[v] = tg;
        };
        auto pop_global = [&](uint32_t v) -> uint32_t {  // the residual's global rounds
            const uint32_t k = kk[v], was = tw[v];
            if (k >= a.k_limit) err |= kErrVisitOverflow;
            const uint32_t tg = tile_draw<kWeighted>(a, v, k, t);
            redrawn(v, was, tg, k);
            return tg;
        };

        // Cycle popping inside a vertex set held in LDS: the tile of the b ids from
        // lo on, which draw their first arrows, or (res) the residual, b ids in
        // res_list.  Ends with every vertex's exit in J (a tile), or with nobody
        // left to pop (the residual).
        uint32_t *res_list = bU;
        auto pop_set = [&](uint32_t b, uint32_t lo, bool res, int ph_pop, int ph_jump, int ph_cycle) {
            auto marked = [&](uint32_t i) { return (mark[i >> 5] >> (i & 31u)) & 1u; };
            auto code_of = [&](uint32_t tg) -> uint32_t {
                if (tg == n) return kRoot;
                if (res) {
                    const uint32_t at = sc[tg];  // (both loads at once)
                    return ((gbits[tg >> 5] >> (tg & 31u)) & 1u) ? kRoot : at;
                }
                return tg - lo < b ? tg - lo : kExt;
            };
            // Arrows of set vertices at[0..m) from their next draws; the draw counts go
            // up by one.  The loads of kD draws are in flight together.
            auto redraw = [&](const uint32_t (&at)[kD], uint32_t m) {
                uint32_t k[kD], was[kD], tg[kD];
                VRec r[kD];
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q) {
                    k[q] = was[q] = 0;
                    r[q] = {};
                    if (q >= m) continue;
                    const uint32_t i = at[q], v = res ? res_list[i] : lo + i;
                    if (res) {
                        k[q] = kk[v];
                        was[q] = tw[v];
                    } else {
                        k[q] = drawn[i];
                        if ((spill[i >> 5] >> (i & 31u)) & 1u) k[q] |= kk[v] << kLowBits;
                    }
                    r[q] = load_vrec(a.vrec, v);  // on its way during the Philox rounds
                }
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q) {
                    tg[q] = n;
                    if (q >= m) continue;
                    const uint32_t v = res ? res_list[at[q]] : lo + at[q];
                    const Philox4 x = philox4x32_10(v, k[q], t, a.stream_id, a.key0, a.key1);
                    hold_vrec(r[q]);
                    tg[q] = arrow_target<kWeighted>(r[q], x.x0, x.x1, a.col_idx, a.wsum, a.wthr, n);
                }
#pragma unroll
                for (uint32_t q = 0; q < kD; ++q) {
                    if (q >= m) continue;
                    const uint32_t i = at[q], v = res ? res_list[i] : lo + i;
                    if (k[q] >= a.k_limit) {  // the error ends the tree here: as if v were a root
                        err |= kErrVisitOverflow;
                        arrow[i] = static_cast<uint16_t>(kRoot | kAgain);
                        jump[i] = static_cast<uint16_t>(kDone | kRoot);
                        continue;
                    }
                    if (res) redrawn(v, was[q], tg[q], k[q]);
                    const uint32_t code = code_of(tg[q]);
                    arrow[i] = static_cast<uint16_t>(code | kAgain);
                    if (code == kRoot) {
                        jump[i] = static_cast<uint16_t>(kDone | kRoot);
                    } else if (code == kExt) {
                        jump[i] = static_cast<uint16_t>(kDone | i);
                        tw[v] = tg[q];
                    } else {  // a target whose exit is known: its path is final
                        const uint32_t j = jump[code];
                        if (j & kDone) jump[i] = static_cast<uint16_t>(j);
                    }
                    if (!res) {
                        drawn[i] = static_cast<uint8_t>(k[q] + 1u);
                        if (((k[q] + 1u) & ((1u << kLowBits) - 1u)) == 0u) {
                            kk[v] = (k[q] + 1u) >> kLowBits;
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

            for (uint32_t i = tid; i < 3u * L.nb; i += T) s_dyn[i] = 0u;
            if (tid == 0) s_cnt = 0;
            if (tid < 4u) s_flags[tid] = 0;
            uint32_t open = 0;  // bit q: the exit of vertex q T + tid is not known
            if (res) {
                for (uint32_t q = 0; q * T + tid < b; ++q) {
                    const uint32_t i = q * T + tid;
                    const uint32_t code = code_of(tw[res_list[i]]);
                    arrow[i] = static_cast<uint16_t>(code);
                    jump[i] = static_cast<uint16_t>(code == kRoot ? kDone | kRoot : 0u);
                    if (code != kRoot) open |= 1u << q;
                }
            } else {
                for (uint32_t i0 = 0; i0 * T < b; i0 += kD) {
                    VRec r[kD] = {};
                    uint32_t tg[kD];
#pragma unroll
                    for (uint32_t q = 0; q < kD; ++q) {
                        const uint32_t i = (i0 + q) * T + tid;
                        if (i < b) r[q] = load_vrec(a.vrec, lo + i);
                    }
#pragma unroll
                    for (uint32_t q = 0; q < kD; ++q) {
                        const uint32_t i = (i0 + q) * T + tid;
                        tg[q] = n;
                        if (i < b) {
                            const Philox4 x = philox4x32_10(lo + i, 0u, t, a.stream_id, a.key0, a.key1);
                            tg[q] = arrow_target<kWeighted>(r[q], x.x0, x.x1, a.col_idx, a.wsum, a.wthr, n);
                        }
                    }
#pragma unroll
                    for (uint32_t q = 0; q < kD; ++q) {
                        const uint32_t i = (i0 + q) * T + tid;
                        if (i >= b) continue;
                        const uint32_t code = code_of(tg[q]);
                        arrow[i] = static_cast<uint16_t>(code);
                        drawn[i] = 1;
                        jump[i] = static_cast<uint16_t>(code == kRoot ? kDone | kRoot
                                                        : code == kExt ? kDone | i : 0u);
                        if (code == kExt) tw[lo + i] = tg[q];
                        if (code < kExt) open |= 1u << (i0 + q);
                    }
                }
            }
            __syncthreads();
            if (!res) mark_time(kPhDraw);
            // 2-cycles of the first arrows, each listed by its smaller end
            {
                uint32_t pop = 0;
                for (uint32_t todo = open; todo; todo &= todo - 1u) {
                    const uint32_t q = static_cast<uint32_t>(__builtin_ctz(todo));
                    const uint32_t i = q * T + tid, w = arrow[i];
                    if (i < w && arrow[w] == i) pop |= 1u << q;
                }
                while (__ballot(pop != 0u)) {
                    const bool have = pop != 0u;
                    const uint32_t u = have ? static_cast<uint32_t>(__builtin_ctz(pop)) * T + tid : 0u;
                    append_pair(0u, L.cap, u, have ? arrow[u] : 0u, have);
                    pop &= pop - 1u;
                }
            }
            __syncthreads();
            uint32_t rounds = 0;
            bool wide = true;  // this round's jumps go over all open vertices
            uint32_t cur = 0, ccur = min(uniform(s_cnt), L.cap);  // list entries that draw
            bool done = false;
            __syncthreads();
            for (;;) {
                // pop what is listed, then the 2-cycles that the new arrows close.  A
                // pass takes 2 us, nearly all of it the loads of one draw after the
                // other: the few pairs that are left of the first arrows' are as well
                // popped with the first cycles (grid of 1e6 vertices, alpha 1, 1024
                // trees: 20.8 ms with every pass, 20.4 without those below kFewPairs).
                while (ccur > (wide ? kFewPairs : 0u)) {
                    for (uint32_t j = tid; j < ccur; j += kD * T) {
                        uint32_t at[kD], m = 0;
#pragma unroll
                        for (uint32_t q = 0; q < kD; ++q) {
                            at[q] = 0;
                            if (j + q * T < ccur) {
                                at[q] = list[cur + j + q * T];
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
                    if (draws > a.step_cap) break;
                    // pairs go to the larger part of the list that is free; pairs that
                    // find no room there wait for the cycle search
                    const uint32_t after = L.cap - (cur + ccur);
                    const uint32_t nxt = after >= cur ? cur + ccur : 0u;
                    const uint32_t room = a.repop ? (after >= cur ? after : cur) & ~1u : 0u;
                    for (uint32_t j0 = wave_base; j0 < ccur; j0 += T) {
                        uint32_t u = 0, w = 0;
                        bool pair = false;
                        if (j0 + lane < ccur) {
                            u = list[cur + j0 + lane];
                            w = arrow[u] & kIdMask;
                            // the pair belongs to its smaller end if both drew
                            if (w < kExt)
                                pair = (arrow[w] & kIdMask) == u && (!marked(w) || u < w);
                        }
                        append_pair(nxt, room, u, w, pair);
                    }
                    __syncthreads();
                    for (uint32_t j = tid; j < ccur; j += T) {
                        const uint32_t i = list[cur + j];
                        atomicAnd(&mark[i >> 5], ~(1u << (i & 31u)));
                    }
                    ccur = min(uniform(s_cnt), room);
                    cur = nxt;
                    __syncthreads();  // s_cnt is read, the marks are gone
                }
                mark_time(ph_pop);
                if (++rounds > a.max_rounds || draws > a.step_cap) {
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
                cur = 0;
                ccur = total;
                if (total > L.cap) {
                    ccur = 0;
                    draws += total;
                }
                __syncthreads();
                mark_time(ph_cycle);
                wide = false;
            }
            __syncthreads();
            if (res) return;
            // the exits of the vertices that hang off those the last rounds settled
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

        // -------------------------------------------------------------------
        // 1. tiles: their own cycles, then every vertex's exit
        // -------------------------------------------------------------------
        for (uint32_t tile = 0; tile < ntiles && !(err & kErrStepCap); ++tile) {
            const uint32_t lo = tile * B;
            const uint32_t b = min(B, n - lo);
            __syncthreads();
            pop_set(b, lo, false, kPhPop, kPhJump, kPhCycle);
            if (err & kErrStepCap) break;
            // the tile's exits, and its part of the outputs
            if (tid == 0) s_c = 0;
            __syncthreads();
            for (uint32_t i0 = wave_base; i0 < b; i0 += T) {
                const uint32_t i = i0 + lane, v = lo + i;
                bool isx = false;
                if (i < b) {
                    const uint32_t c = arrow[i] & kIdMask, e = jump[i] & kIdMask;
                    isx = c == kExt;
                    ex[v] = static_cast<uint16_t>(e);
                    uint32_t k = drawn[i];
                    if ((spill[i >> 5] >> (i & 31u)) & 1u) k |= kk[v] << kLowBits;
                    if (e != kRoot) {
                        tl[v] = static_cast<uint16_t>(c);
                        kk[v] = k;
                    }
                    uint32_t tg = lo + c;
                    if (c == kRoot) {
                        tg = n;
                        ++my_roots;
                        atomicAdd(&a.root_counts[v], 1u);
                    } else if (isx) {
                        tg = tw[v];
                        pc[v] = 0u;
                    }
                    my_digest += mix64((static_cast<unsigned long long>(v) << 32) | tg);
                    const size_t at = static_cast<size_t>(item) * nn + v;
                    if (a.parents) a.parents[at] = static_cast<int32_t>(tg);
                    if (a.visit_counts)
                        atomicAdd(&a.visit_counts[v], static_cast<unsigned long long>(k));
                    if (a.tree_visits) a.tree_visits[at] = k;
                }
                wave_push<uint32_t>(exl, lo, &s_c, lo + b, &s_over, v, isx);
            }
            __syncthreads();
            if (tid == 0) ecnt[tile] = min(s_c, b);
            mark_time(kPhExits);
        }
        __syncthreads();
        if (err & kErrStepCap) break;

        // -------------------------------------------------------------------
        // 2. the exit graph: u -> ex[target(u)] over the exit vertices
        // -------------------------------------------------------------------
        if (tid == 0) {
            s_u = 0;
            s_lc[0] = s_lc[1] = s_lc[2] = 0;
        }
        for (uint32_t i = tid; i < nw; i += T) xb[i] = 0u;
        __syncthreads();
        for (uint32_t tile = wave_base >> 6; tile < ntiles; tile += T >> 6) {
            const uint32_t c = ecnt[tile];
            const uint32_t *seg = exl + static_cast<size_t>(tile) * B;
            for (uint32_t i = 0; i < c; i += 64) {
                const bool ok = i + lane < c;
                wave_push<uint32_t>(bU, 0u, &s_u, n, &s_over, ok ? seg[i + lane] : 0u, ok);
            }
        }
        __syncthreads();
        const uint32_t m = min(uniform(s_u), n);
        bool residual = false;
        if (m > 0) {
            for (uint32_t i = tid; i < m; i += T) {
                const uint32_t u = bU[i];
                const uint32_t x = tw[u];
                const uint32_t e = ex[x];
                const uint32_t s = e == kRoot ? n : x - x % B + e;
                sc[u] = s;
                if (s < n) atomicAdd(&pc[s], 1u);
            }
            __syncthreads();
            if (tid == 0) s_u = 0;  // everybody has read it; the residual counts with it
            for (uint32_t i = wave_base; i < m; i += T) {
                const uint32_t li = i + lane;
                uint32_t u = 0;
                bool leaf = false;
                if (li < m) {
                    u = bU[li];
                    leaf = pc[u] == 0u;
                }
                wave_push<uint32_t>(bP, 0u, &s_lc[0], n, &s_over, u, leaf);
            }
            __syncthreads();
            uint32_t plo = 0, phi = min(uniform(s_lc[0]), n), nlev = 0;
            if (tid == 0) lvg[0] = 0;
            while (phi > plo) {
                const uint32_t cn = (nlev + 1u) % 3u, cz = (nlev + 2u) % 3u;
                if (tid == 0) {
                    lvg[nlev + 1] = phi;
                    s_lc[cz] = 0;
                }
                for (uint32_t i = plo + wave_base; i < phi; i += T) {
                    const uint32_t li = i + lane;
                    uint32_t s = 0;
                    bool push = false;
                    if (li < phi) {
                        s = sc[bP[li]];
                        if (s < n) push = atomicSub(&pc[s], 1u) == 1u;
                    }
                    wave_push<uint32_t>(bP, phi, &s_lc[cn], n, &s_over, s, push);
                }
                __syncthreads();
                ++nlev;
                plo = phi;
                phi = min(phi + uniform(s_lc[cn]), n);
            }
            // reverse sweep: an exit reaches u* when its successor does (bit in xb)
            for (uint32_t L = nlev; L > 0; --L) {
                const uint32_t a0 = lvg[L - 1], a1 = lvg[L];
                for (uint32_t i = a0 + tid; i < a1; i += T) {
                    const uint32_t u = bP[i];
                    const uint32_t s = sc[u];
                    if (s >= n || ((xb[s >> 5] >> (s & 31u)) & 1u)) atomicOr(&xb[u >> 5], 1u << (u & 31u));
                }
                __syncthreads();
            }
            residual = plo < m;  // exits left unpeeled lie on crossing cycles
        }
        mark_time(kPhExit);

        // -------------------------------------------------------------------
        // 3. the residual: vertices whose exit does not reach u*
        // -------------------------------------------------------------------
        if (residual) {
            // exits on crossing cycles keep one in-arrow count: clear it
            for (uint32_t i = tid; i < m; i += T) pc[bU[i]] = 0u;
            __syncthreads();
            // settled bitmap (global first) and the residual list: v is settled iff
            // its path reaches u* inside its tile or its exit's chain does.  The
            // residual works on global targets and counters of its own.
            // Eight vertices a lane: one 16-byte load of exits (kS in flight), one byte
            // of the bitmap.
            constexpr uint32_t kS = 4;
            for (uint32_t base0 = wave_base * 8u; base0 < n; base0 += kS * 8u * T) {
                uint4 e4[kS];
#pragma unroll
                for (uint32_t p = 0; p < kS; ++p) {
                    const uint32_t v0 = base0 + (p * T + lane) * 8u;
                    e4[p] = v0 < n ? *reinterpret_cast<const uint4 *>(ex + v0) : uint4{};
                }
                uint32_t left[kS], mine = 0;  // bit q: v0 + q is not settled
#pragma unroll
                for (uint32_t p = 0; p < kS; ++p) {
                    left[p] = 0;
                    const uint32_t v0 = base0 + (p * T + lane) * 8u;
                    if (v0 >= n) continue;
                    const uint32_t e2[4] = {e4[p].x, e4[p].y, e4[p].z, e4[p].w};
                    const uint32_t lo = v0 - v0 % B;  // (tiles are multiples of 64 ids)
#pragma unroll
                    for (uint32_t q = 0; q < 8u; ++q) {
                        const uint32_t e = (e2[q >> 1] >> ((q & 1u) << 4)) & 0xFFFFu;
                        if (v0 + q < n && e != kRoot) {
                            const uint32_t x = lo + e;
                            if (!((xb[x >> 5] >> (x & 31u)) & 1u)) left[p] |= 1u << q;
                        }
                    }
                    reinterpret_cast<uint8_t *>(gbits)[v0 >> 3] = static_cast<uint8_t>(~left[p]);
                    mine += static_cast<uint32_t>(__popc(left[p]));
                }
                if (!__ballot(mine != 0u)) continue;
                uint32_t at = mine;  // running sum over the wave
                for (uint32_t off = 1; off < 64u; off <<= 1) {
                    const uint32_t y = __shfl_up(at, off, 64);
                    if (lane >= off) at += y;
                }
                uint32_t first = 0;
                if (lane == 63u) first = atomicAdd(&s_u, at);
                at += __shfl(first, 63, 64) - mine;
#pragma unroll
                for (uint32_t p = 0; p < kS; ++p)
                    for (uint32_t todo = left[p]; todo; todo &= todo - 1u)
                        bU[at++] = base0 + (p * T + lane) * 8u + static_cast<uint32_t>(__builtin_ctz(todo));
            }
            __syncthreads();
            uint32_t ucount = min(uniform(s_u), n);
            for (uint32_t i = tid; i < ucount; i += T) {
                const uint32_t v = bU[i], c = tl[v];
                if (c != kExt) tw[v] = v - v % B + c;
                pc[v] = 0u;
            }
            __syncthreads();
            if (ucount > B && a.bits_lds) {  // the global rounds test the bitmap in LDS
                for (uint32_t i = tid; i < nw; i += T) s_dyn[i] = gbits[i];
                __syncthreads();
            }
            uint32_t *U = bU, *Un = bN;
            uint32_t rounds = 0;
            while (ucount > 0) {
                if (ucount <= B) {
                    // What is left fits the tiles' LDS arrays: pop it as one more
                    // set, its vertices numbered in list order (sc, spent since the
                    // exit graph, maps an id to that number); targets settled
                    // before count as u*.
                    if (rounds > 0 && a.bits_lds) {  // the settled bitmap back to global
                        for (uint32_t i = tid; i < nw; i += T) gbits[i] = s_dyn[i];
                        __syncthreads();
                    }
                    for (uint32_t i = tid; i < ucount; i += T) sc[U[i]] = i;
                    __syncthreads();
                    res_list = U;
                    pop_set(ucount, 0u, true, kPhResidual, kPhResidual, kPhResidual);
                    break;
                }
                if (++rounds > a.max_rounds || s_over) {
                    err |= kErrStepCap;
                    break;
                }
                if (tid == 0) s_lc[0] = s_lc[1] = s_lc[2] = 0;
                for (uint32_t i = tid; i < ucount; i += T) {
                    const uint32_t tg = tw[U[i]];
                    if (!is_settled(tg)) atomicAdd(&pc[tg], 1u);
                }
                __syncthreads();
                if (tid == 0) {  // the last round's are read, the next barrier is before this one's
                    s_u = 0;
                    s_c = 0;
                }
                for (uint32_t i = wave_base; i < ucount; i += T) {
                    const uint32_t li = i + lane;
                    uint32_t x = 0;
                    bool leaf = false;
                    if (li < ucount) {
                        x = U[li];
                        leaf = pc[x] == 0u;
                    }
                    wave_push<uint32_t>(bP, 0u, &s_lc[0], n, &s_over, x, leaf);
                }
                __syncthreads();
                uint32_t plo = 0, phi = min(uniform(s_lc[0]), n), nlev = 0;
                if (tid == 0) lvg[0] = 0;
                while (phi > plo) {
                    const uint32_t cn = (nlev + 1u) % 3u, cz = (nlev + 2u) % 3u;
                    if (tid == 0) {
                        lvg[nlev + 1] = phi;
                        s_lc[cz] = 0;
                    }
                    for (uint32_t i = plo + wave_base; i < phi; i += T) {
                        const uint32_t li = i + lane;
                        uint32_t tg = 0;
                        bool push = false;
                        if (li < phi) {
                            tg = tw[bP[li]];
                            if (!is_settled(tg)) push = atomicSub(&pc[tg], 1u) == 1u;
                        }
                        wave_push<uint32_t>(bP, phi, &s_lc[cn], n, &s_over, tg, push);
                    }
                    __syncthreads();
                    ++nlev;
                    plo = phi;
                    phi = min(phi + uniform(s_lc[cn]), n);
                }
                const uint32_t peeled = phi;
                // reverse sweep: settled when the target is; the others hang off a
                // cycle and stay listed
                for (uint32_t L = nlev; L > 0; --L) {
                    const uint32_t a0 = lvg[L - 1], a1 = lvg[L];
                    for (uint32_t i = a0 + wave_base; i < a1; i += T) {
                        const uint32_t li = i + lane;
                        uint32_t x = 0;
                        bool hang = false;
                        if (li < a1) {
                            x = bP[li];
                            if (is_settled(tw[x])) set_settled(x);
                            else hang = true;
                        }
                        wave_push<uint32_t>(Un, 0u, &s_u, n, &s_over, x, hang);
                    }
                    __syncthreads();
                }
                if (peeled == ucount) break;  // no cycle left
                // pop the cycles: listed vertices never peeled (one in-arrow left)
                uint32_t pops = 0;
                for (uint32_t i = wave_base; i < ucount; i += T) {
                    const uint32_t li = i + lane;
                    uint32_t x = 0;
                    bool live = false;
                    if (li < ucount) {
                        x = U[li];
                        if (!is_settled(x) && pc[x] != 0u) {
                            pc[x] = 0u;
                            const uint32_t tg = pop_global(x);
                            if (tg == n) set_settled(x);
                            else live = true;
                            ++pops;
                        }
                    }
                    wave_push<uint32_t>(Un, 0u, &s_u, n, &s_over, x, live);
                }
                wave_count(&s_c, pops);
                __syncthreads();
                draws += uniform(s_c);
                ucount = min(uniform(s_u), n);
                uint32_t *tmp = U;
                U = Un;
                Un = tmp;
            }
            __syncthreads();
            if (err & kErrStepCap) break;
        }
        mark_time(kPhResidual);
        if (draws > a.step_cap) {
            err |= kErrStepCap;
            break;
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
            if (a.tree_digests) a.tree_digests[item] = s_digest;
            if (a.tree_steps) a.tree_steps[item] = draws;
            atomicAdd(&a.totals->walk_steps, draws);
            atomicAdd(&a.totals->roots, s_roots);
            atomicAdd(&a.totals->digest_sum, s_digest);
        }
        mark_time(kPhOutput);
    }
    if (timing && tid == 0)
        for (int i = 0; i < kPhNum; ++i) atomicAdd(&a.phase_ticks[i], s_ph[i]);
    if (s_over) err |= kErrStepCap;
    if (err) atomicOr(&a.totals->error, err);
}

// Entries that join ids of different tiles, one CSR entry per lane and step.
// (One row per thread left the hub rows to one lane each: 10.8 ms on R-MAT
// with 2^22 vertices, 65 M entries; now 0.19 ms.)
constexpr uint32_t kCrossThreads = 1024, kCrossBlocks = 512;

__global__ __launch_bounds__(kCrossThreads) void count_cross_kernel(const int32_t *__restrict__ row_ptr,
                                                          const int32_t *__restrict__ col_idx,
                                                          int32_t n, int64_t nnz, uint32_t B,
                                                          uint32_t steps, unsigned long long *out) {
    __shared__ uint32_t s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    RowFinder rows;
    uint32_t c = 0;
    const int64_t first =
        (static_cast<int64_t>(blockIdx.x) * (kCrossThreads / 64u) + (threadIdx.x >> 6)) * 64 * steps;
    for (uint32_t t = 0; t < steps; ++t) {
        const int64_t j0 = first + static_cast<int64_t>(t) * 64;
        if (j0 >= nnz) break;
        const int64_t j = j0 + (threadIdx.x & 63u);
        int32_t v = 0, b = 0, e = 0;
        rows.find(row_ptr, n, j0, nnz, &v, &b, &e);
        if (j < nnz && static_cast<uint32_t>(col_idx[j]) / B != static_cast<uint32_t>(v) / B) ++c;
    }
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
    if ((threadIdx.x & 63u) == 0 && c) atomicAdd(&s_sum, c);
    __syncthreads();
    if (threadIdx.x == 0 && s_sum) atomicAdd(out, static_cast<unsigned long long>(s_sum));
}

}  // namespace

hipError_t launch_count_cross(const int32_t *row_ptr, const int32_t *col_idx, uint32_t n,
                              int64_t nnz, uint32_t B, unsigned long long *out,
                              hipStream_t stream) {
    if (n == 0 || nnz == 0) return hipSuccess;
    const int64_t per_step = static_cast<int64_t>(kCrossThreads) * kCrossBlocks;
    const uint32_t steps = static_cast<uint32_t>((nnz + per_step - 1) / per_step);
    const int64_t per = static_cast<int64_t>(kCrossThreads) * steps;
    count_cross_kernel<<<static_cast<unsigned int>((nnz + per - 1) / per), kCrossThreads, 0,
                         stream>>>(row_ptr, col_idx, static_cast<int32_t>(n), nnz, B, steps, out);
    return hipGetLastError();
}

size_t tile_lds_bytes(uint32_t B) {
    return 4u * static_cast<size_t>(tile_layout((B + 63u) & ~63u).words);
}

hipError_t tile_set_limit(size_t bytes) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wilson_tile_kernel<false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(bytes));
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&wilson_tile_kernel<true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
}

int tile_max_active(uint32_t threads, size_t lds, bool weighted) {
    int blocks = 0;
    const void *f = weighted ? reinterpret_cast<const void *>(&wilson_tile_kernel<true>)
                             : reinterpret_cast<const void *>(&wilson_tile_kernel<false>);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, static_cast<int>(threads), lds) !=
        hipSuccess)
        return 0;
    return blocks;
}

hipError_t launch_wilson_tile(const TileArgs &a, uint32_t threads, size_t lds, hipStream_t stream) {
    if (a.n == 0 || a.tree_count == 0 || a.slots == 0) return hipSuccess;
    if (a.B == 0 || a.B > kTileMax || a.Bp % 64u || a.Bp < a.B) return hipErrorInvalidValue;
    if (a.B > kTileOwn * threads || lds < tile_lds_bytes(a.Bp)) return hipErrorInvalidValue;
    const size_t bw = 4u * static_cast<size_t>((a.n + 31u) >> 5);
    if ((a.bits_lds || !a.xb) && bw > lds) return hipErrorInvalidValue;
    if (a.wsum) wilson_tile_kernel<true><<<a.slots, threads, lds, stream>>>(a);
    else wilson_tile_kernel<false><<<a.slots, threads, lds, stream>>>(a);
    return hipGetLastError();
}

}  // namespace fc
