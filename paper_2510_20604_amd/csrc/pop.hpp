// Cycle popping in rounds: Wilson's algorithm for graphs of up to kPopMaxNodes nodes, one
// work-group per tree, the tree in LDS.  Included by sampler.hip.
//
// Wilson's algorithm is cycle popping (Propp and Wilson, "How to get a perfectly random sample from
// a generic Markov chain and generate a random spanning tree of a directed graph", J. Algorithms
// 27, 1998): every node holds the current entry of its stack of arrows, cycles of the arrow
// configuration are popped in any order, and whatever the order, the same stack entries are
// popped and the same tree is left.  A node's departure count in Algorithm 3 is the number of
// its entries read: the popped ones and the one that stays.  So instead of walking, every node
// draws its first arrow at once, and then each round pops every cycle there is.  On small-world
// graphs a few rounds are enough (nine on average for BA(20 000, 5), nineteen for ER(1000, 8)),
// each of them work for many lanes without waiting or claims, where a team of walkers on the
// same tree spends most of its time waiting on each other's paths (ER(1000, 8): 61 % of its
// lanes; 370 dependent iterations per tree).
//
// Finding the cycles.  A round follows every arrow path at once by pointer doubling: with f the
// arrow map, f^2, f^4, ... of every active node, each level one LDS read per node and all threads
// in step.  Once 2^L is at least the number of active nodes, f^(2^L) of a node either has run into
// a node known to lead to the root (then so does the node, for good: no arrow on that path can
// be on a cycle again, and the node leaves the active ones) or is a cycle node, and the
// images are exactly the cycle nodes.  (Lanes that each follow their own path instead, with
// Brent's algorithm, need fewer reads but one after the other: a round of ER(1000, 8) took 35 us.)
//
// The arrows are 16-bit internal indices in LDS with the "leads to the root" flag in bit 15, so
// that one LDS read per step answers both questions.  Departure counts (32 bits) are in LDS for
// small graphs, else in a slot of the workspace per work-group (read together with the node's
// record, whose latency it shares).
//
// Meshes take thousands of rounds of few cycles each (a 20 000-node mesh: 3 000) and have a kernel of
// their own (tokens.hpp).
//
// What bounds it: the latency of a round (levels of two barriers and two LDS accesses, then a draw) while
// the device is not full, and the issue of the levels' instructions once it is.  On large graphs a round
// costs too much that way (100 us for 20 000 nodes) when only few arrows changed: a cycle runs through a
// node whose arrow changed in the round before, so such a round follows only those nodes' paths
// (pop_walk).  So it does on graphs with hubs, whose paths are short, and where heavy edges make many
// rounds of few cycles (the rules: follows_changes in sampler.hip).
//
// A work-group adds its trees' visits up in the workspace and pop_reduce adds the work-groups' sums
// (single graphs: an atomic per node and tree bounded large calls, 29 G/s: BA(2000, 4) x 20 000
// trees 2.88 -> 1.27 ms, BA(20 000, 5) x 2000 2.40 -> 1.81 ms).
#pragma once

#include "common.hpp"
#include "device.hpp"
#include "select.hpp"
#include "walk.hpp"

namespace rwc {
namespace {

constexpr uint32_t kPopDone = 0x8000u;
constexpr int32_t kPopMaxNodes = 30000;      // 15-bit indices, 5 bytes of LDS per node
constexpr int32_t kPopLdsCounts = 8192;      // largest graph with its counts in LDS
constexpr int kPopMaxThreads = 1024;

// LDS of one work-group, in 4-byte words: the arrows, the doubled arrows (after the last level: the
// list of cycle nodes), two lists of active nodes, a bitmap of cycle nodes, and the counts
// of graphs that keep them here.  A list of active nodes holds a quarter of the nodes; while
// more are active, a round looks at every node.
struct PopLayout {
    int32_t arrows, cap, list_words, bit_words, counts;
    __host__ __device__ explicit PopLayout(int32_t n)
        : arrows((n + 1) / 2), cap(n / 4), list_words((cap + 1) / 2), bit_words((n + 31) / 32),
          counts(n <= kPopLdsCounts ? n : 0) {}
    __host__ __device__ int32_t words() const { return 2 * arrows + 2 * list_words + bit_words + counts; }
};

struct PopArgs {
    const GraphArgs* graphs;
    const Item* items;        // one per graph, in the order they are worked through; slot0 1: rounds of cycle_pop that
                              // changed few arrows follow those nodes only
    int32_t ngraphs;
    uint32_t* queue;
    int64_t sample_begin, l;
    uint64_t seed;
    const int64_t* node_off;
    uint32_t* slots;          // [work-groups][slot_stride] words of the trees in the workspace
    int64_t slot_stride;
    uint64_t* sums;           // [work-groups][2][sum_stride] visits and squared visits of the work-group's trees,
    int64_t sum_stride;       // reduced by pop_reduce; null: every tree is added to the totals
    uint64_t *counts, *counts_sq;
    int32_t* parents;
    uint64_t *tree_hash, *total_steps;
    uint32_t* status;
};

__device__ __forceinline__ uint32_t lds_or(RWC_LDS uint32_t* p, uint32_t v) {
    return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_and(RWC_LDS uint32_t* p, uint32_t v) {
    __hip_atomic_fetch_and(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t lds_add(RWC_LDS uint32_t* p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The arrow at entry k of node v's stack (an internal index).
template <bool kStrat>
__device__ __forceinline__ uint32_t pop_draw(const GraphArgs& G, uint32_t v, uint32_t k, uint32_t sw, uint32_t k0,
                                             uint32_t k1) {
    const auto col = global_ptr(G.col);
    const auto cdf = global_ptr(G.cdf);
    const auto q = global_ptr(G.rec) + (kRecWords / 4) * static_cast<int64_t>(v);
    const uint4 a = load_u4(q);
    uint64_t r;
    auto word = [&]() {
        r = philox_x64(k, a.z, sw, G.graph_word, k0, k1);   // word kRecId: the node's input id
        if constexpr (kStrat) r = stratified_word(r, k, a.z, sw, G.graph_word, k0, k1, G.strata);
    };
    static_assert(kRecId == 2 && kRecFirst == 3, "record words read below");
    if (cdf == nullptr) {
        word();
        const uint32_t pos = static_cast<uint32_t>(select_unweighted(r, static_cast<int32_t>(a.x)));
        if (pos == 0) return a.w;
        if (pos < static_cast<uint32_t>(kRecInline))
            return reinterpret_cast<const RWC_GLOBAL uint32_t*>(q)[kRecFirst + pos];
        return static_cast<uint32_t>(col[static_cast<int32_t>(a.y) + static_cast<int32_t>(pos)]);
    }
    const uint4 b = load_u4(q + 1), c = load_u4(q + 2), d = load_u4(q + 3);
    word();
    return choose_neighbor(r, [&](uint32_t i) { return rec_word(a, b, c, d, i); }, col, cdf);
}

// Counts of the current tree, in LDS or in this work-group's slot of the workspace.
template <bool kLds>
struct PopCounts;
template <>
struct PopCounts<true> {
    RWC_LDS uint32_t* p;
    __device__ uint32_t get(uint32_t v) const { return p[v]; }
    __device__ void set(uint32_t v, uint32_t c) const { p[v] = c; }
};
template <>
struct PopCounts<false> {
    RWC_GLOBAL uint32_t* p;
    __device__ uint32_t get(uint32_t v) const { return p[v]; }
    __device__ void set(uint32_t v, uint32_t c) const { p[v] = c; }
};

// A round that walks: each changed node follows its path, four steps between two looks, until it is
// back, meets a node known to lead to the root, or has gone round a cycle it is not on (Brent's
// algorithm); a lane back at its node lists the cycle's nodes.  A call of its own: inlined, its registers and
// place in the loop cost the rounds that double (ER(1000, 8), 2000 trees 664 and 679 us; BA(20 000, 5) 1966
// and 1994).
__device__ __attribute__((noinline)) void pop_walk(uint32_t changed, const RWC_LDS uint16_t* old_list, RWC_LDS uint16_t* nx,
                                         RWC_LDS uint32_t* bits, RWC_LDS uint16_t* new_list, uint32_t cap,
                                         RWC_LDS uint32_t* found) {
    constexpr uint32_t kNode = kPopDone - 1u;
    for (uint32_t i = threadIdx.x; i < changed; i += blockDim.x) {
        const uint32_t c = old_list[i];
        const uint32_t first = nx[c];
        if (first & kPopDone) continue;   // a root
        uint32_t p = first, mark = kPopDone, power = 2, lam = 0;   // (no node is kPopDone)
        bool on_cycle, done;
        while (true) {
            const uint32_t a1 = nx[p], a2 = nx[a1 & kNode], a3 = nx[a2 & kNode], a4 = nx[a3 & kNode];
            done = ((a1 | a2 | a3 | a4) & kPopDone) != 0;
            on_cycle = !done && (p == c || a1 == c || a2 == c || a3 == c);
            if (done || on_cycle || a1 == mark || a2 == mark || a3 == mark || a4 == mark) break;
            if (++lam == power) {
                mark = a4;
                power <<= 1;
                lam = 0;
            }
            p = a4;
        }
        if (done) nx[c] = static_cast<uint16_t>(first | kPopDone);
        if (!on_cycle || (bits[c >> 5] >> (c & 31)) & 1u) continue;   // listed: by a lane that lists all of it
        p = c;
        do {
            const uint32_t bit = 1u << (p & 31);
            if (!(lds_or(&bits[p >> 5], bit) & bit)) {
                const uint32_t slot = lds_add(found, 1u);
                if (slot < cap) new_list[slot] = static_cast<uint16_t>(p);
            }
            p = nx[p];
        } while (p != c);
    }
}

// A round after at most kWalkShare / 64 of the nodes changed walks (on graphs that the plan says so of).  The
// space of the doubled arrows then holds the list of changed nodes and the one the round makes in
// its two halves, so a list that is walked must fit one: at most half of the nodes.
constexpr int32_t kWalkShare = 16;
static_assert(kWalkShare <= 32, "the changed nodes must fit half of the doubled arrows' space");

// Grows one tree; returns with the arrows and counts final.  Every thread of the work-group
// calls; kPerThread * blockDim.x >= n.  counters: two sets of (cycle nodes, active nodes).
template <bool kStrat, bool kLdsCounts, int kPerThread>
__device__ __forceinline__ void pop_tree(const GraphArgs& G, uint64_t sample, uint64_t seed, int32_t walk_share,
                                         const PopLayout& P, RWC_LDS uint32_t* lds, PopCounts<kLdsCounts> cnt, RWC_LDS uint32_t* counters,
                                         RWC_LDS uint32_t* err) {
    RWC_LDS uint16_t* const nx = (RWC_LDS uint16_t*)lds;
    RWC_LDS uint16_t* const jump = (RWC_LDS uint16_t*)(lds + P.arrows);
    RWC_LDS uint16_t* const lists = (RWC_LDS uint16_t*)(lds + 2 * P.arrows);
    RWC_LDS uint32_t* const bits = lds + 2 * P.arrows + 2 * P.list_words;
    const uint32_t n = static_cast<uint32_t>(G.n), cap = static_cast<uint32_t>(P.cap);
    const uint32_t t = threadIdx.x, T = blockDim.x, lane = t & (kWave - 1);
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    const uint32_t sw = static_cast<uint32_t>(sample);
    for (uint32_t i = t; i < static_cast<uint32_t>(P.bit_words); i += T) bits[i] = 0;
    if (t < 4) counters[t] = 0;
    for (uint32_t v = t; v < n; v += T) {
        const bool root = G.rootmask ? ((G.rootmask[v >> 5] >> (v & 31)) & 1u) != 0 : static_cast<int32_t>(v) == G.root;
        nx[v] = static_cast<uint16_t>(root ? kPopDone | v : pop_draw<kStrat>(G, v, 0, sw, k0, k1));
        cnt.set(v, root ? 0u : 1u);
    }
    __syncthreads();
    bool listed = false;         // the active nodes are in a list; otherwise all nodes are looked at
    uint32_t count = n, active = n;
    uint32_t popped = n;         // nodes whose arrow the round before changed
    const uint32_t half = n / 2;   // the doubled arrows' space holds two lists of them in turn
    uint32_t at_list = 0;
    int cur = 0, lcur = 0;
    uint64_t rounds = 0, departures = n;
    while (true) {
        RWC_LDS uint32_t* const found = counters + 2 * cur;
        bool scan = false;   // the cycle nodes do not fit their list: read the bitmap
        if (static_cast<uint64_t>(popped) * 64u <= static_cast<uint64_t>(walk_share) * n) {
            const uint32_t from = at_list;
            at_list = half - at_list;
            pop_walk(popped, jump + from, nx, bits, jump + at_list, half, &found[0]);
            __syncthreads();
            popped = found[0];
            scan = popped > half;
        } else {
        at_list = 0;
        RWC_LDS uint16_t* const old_list = lists + lcur * (2 * P.list_words);
        RWC_LDS uint16_t* const new_list = lists + (lcur ^ 1) * (2 * P.list_words);
        // g[i]: f^(2^level) of this thread's i-th node, or kPopDone
        uint32_t g[kPerThread];
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const uint32_t at = t + i * T;
            g[i] = kPopDone;
            if (i * T >= count) break;
            if (at < count) {
                const uint32_t a = nx[listed ? old_list[at] : at];
                if (!(a & kPopDone)) {
                    const uint32_t b = nx[a];   // f^2, and whether f leads to the root
                    if (!(b & kPopDone)) g[i] = (nx[b] & kPopDone) ? kPopDone : b;
                }
            }
        }
        for (uint32_t reach = 2; reach < active; reach <<= 1) {
#pragma unroll
            for (int i = 0; i < kPerThread; ++i) {
                const uint32_t at = t + i * T;
                if (i * T >= count) break;
                if (at < count) jump[listed ? old_list[at] : at] = static_cast<uint16_t>(g[i]);
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kPerThread; ++i) {
                if (i * T >= count) break;
                if (!(g[i] & kPopDone)) g[i] = jump[g[i]];
            }
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const uint32_t at = t + i * T;
            if (i * T >= count) break;
            uint32_t v = 0;
            bool stays = false;
            if (at < count) {
                v = listed ? old_list[at] : at;
                stays = !(g[i] & kPopDone);
                if (stays) {
                    const uint32_t bit = 1u << (g[i] & 31);
                    if (!(lds_or(&bits[g[i] >> 5], bit) & bit)) jump[lds_add(&found[0], 1u)] = static_cast<uint16_t>(g[i]);
                } else {
                    nx[v] |= static_cast<uint16_t>(kPopDone);
                }
            }
            const uint64_t m = __ballot(stays);
            uint32_t slot = 0;
            if (lane == 0 && m) slot = lds_add(&found[1], static_cast<uint32_t>(__popcll(m)));
            slot = __shfl(slot, 0, kWave) + __popcll(m & ((1ull << lane) - 1ull));
            if (stays && slot < cap) new_list[slot] = static_cast<uint16_t>(v);
        }
        __syncthreads();
        popped = found[0];
        active = found[1];
        lcur ^= 1;
        listed = active <= cap;
        count = listed ? active : n;
        }
        if (popped == 0) break;
        const uint32_t redo = scan ? n : popped;
        for (uint32_t i = t; i < redo; i += T) {
            if (scan && !((bits[i >> 5] >> (i & 31)) & 1u)) continue;
            const uint32_t v = scan ? i : jump[at_list + i];
            const uint32_t k = cnt.get(v);
            nx[v] = static_cast<uint16_t>(pop_draw<kStrat>(G, v, k, sw, k0, k1));
            cnt.set(v, k + 1);
            if (k + 1 >= kCntMax) lds_or(err, static_cast<uint32_t>(kErrCountOverflow));
            lds_and(&bits[v >> 5], ~(1u << (v & 31)));
        }
        cur ^= 1;
        if (t < 2) counters[2 * cur + t] = 0;   // the next round's
        if (t == 0) {
            // the walker teams' guard on iterations, which bounds the rounds and, times 64 walkers,
            // the departures
            departures += popped;
            if (rounds + 1 > G.guard || departures / kWave > G.guard)
                lds_or(err, static_cast<uint32_t>(kErrStepLimit));
        }
        ++rounds;
        __syncthreads();
        if (*err) break;
    }
}

// Totals, checksum and parents of a grown tree (outputs are indexed by input id): count(x) is the
// node's departures (0: a root), next(x) its parent.
template <class Count, class Next>
__device__ __forceinline__ void finish_tree(const PopArgs& A, const DumpArgs& dumps, const GraphArgs& G, int32_t graph,
                                            int64_t rel, bool first, Count count, Next next,
                                            RWC_LDS uint32_t* err, RWC_LDS uint64_t* red) {
    const int t = threadIdx.x, T = blockDim.x, lane = t & (kWave - 1);
    int32_t dump_out = -1;
    for (int d = 0; d < dumps.count; ++d)
        if (dumps.slot[d] == rel) dump_out = dumps.out[d];
    const int64_t off = A.node_off[graph];
    uint64_t steps = 0, h = 0;
    for (int32_t x = t; x < G.n; x += T) {
        const uint32_t c = count(x);
        const int64_t id = G.node_id[x];
        if (A.sums) {
            uint64_t* const s = A.sums + static_cast<int64_t>(blockIdx.x) * 2 * A.sum_stride + x;
            s[0] = (first ? 0ull : s[0]) + c;
            s[A.sum_stride] = (first ? 0ull : s[A.sum_stride]) + square_count(c);
        }
        if (c) {
            steps += c;
            if (!A.sums) {
                atomicAdd(reinterpret_cast<unsigned long long*>(&A.counts[off + id]), static_cast<unsigned long long>(c));
                if (A.counts_sq)
                    atomicAdd(reinterpret_cast<unsigned long long*>(&A.counts_sq[off + id]),
                              static_cast<unsigned long long>(square_count(c)));
            }
            if (A.tree_hash)
                h += splitmix64((static_cast<uint64_t>(id) << 32) | static_cast<uint32_t>(G.node_id[next(x)]));
        }
        if (dump_out >= 0) A.parents[static_cast<int64_t>(dump_out) * G.n + id] = c ? G.node_id[next(x)] : -1;
    }
    steps = wave_sum(steps);
    h = wave_sum(h);
    if (lane == 0) {
        red[t / kWave] = steps;
        red[kPopMaxThreads / kWave + t / kWave] = h;
    }
    __syncthreads();
    if (t == 0) {
        steps = h = 0;
        for (int w = 0; w < T / kWave; ++w) {
            steps += red[w];
            h += red[kPopMaxThreads / kWave + w];
        }
        if (A.total_steps)
            atomicAdd(reinterpret_cast<unsigned long long*>(&A.total_steps[graph]), static_cast<unsigned long long>(steps));
        if (A.tree_hash) A.tree_hash[static_cast<int64_t>(graph) * A.l + rel] = h;
        if (*err) atomicOr(A.status, *err);
    }
    __syncthreads();   // the next tree must not overtake this one's reads
}

template <bool kStrat, bool kLdsCounts, int kPerThread>
__device__ __forceinline__ void pop_item(const PopArgs& A, const DumpArgs& dumps, const GraphArgs& G, int32_t graph,
                                         int64_t rel, int32_t walk_share, bool first, RWC_LDS uint32_t* lds,
                                         RWC_LDS uint32_t* counters, RWC_LDS uint32_t* err, RWC_LDS uint64_t* red) {
    const PopLayout P(G.n);
    RWC_LDS uint16_t* const nx = (RWC_LDS uint16_t*)lds;
    PopCounts<kLdsCounts> cnt;
    if constexpr (kLdsCounts)
        cnt.p = lds + (P.words() - P.counts);
    else
        cnt.p = global_ptr(A.slots + static_cast<int64_t>(blockIdx.x) * A.slot_stride);
    if (threadIdx.x == 0) *err = 0;
    pop_tree<kStrat, kLdsCounts, kPerThread>(G, static_cast<uint64_t>(A.sample_begin + rel), A.seed, walk_share, P, lds,
                                             cnt, counters, err);
    finish_tree(
        A, dumps, G, graph, rel, first, [&](int32_t x) { return cnt.get(x); },
        [&](int32_t x) { return nx[x] & (kPopDone - 1u); }, err, red);
}

// Persistent: work-groups pop trees, graph by graph, from `queue`, and hand them to
// grow(item, arguments, sample, first of this work-group, error word, scratch).
template <class Grow>
__device__ __forceinline__ void pop_items(const PopArgs& A, Grow grow) {
    __shared__ uint32_t err, next_item, bad;
    __shared__ uint64_t red[2 * (kPopMaxThreads / kWave)];
    // a root set found faulty leaves trees without a root: the outputs are discarded anyway
    if (threadIdx.x == 0) bad = *A.status;
    __syncthreads();
    if (bad) return;
    const int64_t total = static_cast<int64_t>(A.ngraphs) * A.l;
    bool first = true;
    while (true) {
        if (threadIdx.x == 0) next_item = atomicAdd(A.queue, 1u);
        __syncthreads();
        const int64_t idx = next_item;
        __syncthreads();
        if (idx >= total) break;
        const Item it = A.items[idx / A.l];
        const GraphArgs G = A.graphs[it.graph];
        grow(it, G, idx % A.l, first, (RWC_LDS uint32_t*)&err, (RWC_LDS uint64_t*)red);
        first = false;
    }
    if (A.sums && first)   // no tree for this work-group
        for (int64_t i = threadIdx.x; i < 2 * A.sum_stride; i += blockDim.x)
            A.sums[static_cast<int64_t>(blockIdx.x) * 2 * A.sum_stride + i] = 0;
}

template <bool kStrat, int kPerThread>
__device__ __forceinline__ void pop_graphs(const PopArgs& A, const DumpArgs& dumps, RWC_LDS uint32_t* lds) {
    __shared__ uint32_t counters[4];
    pop_items(A, [&](const Item& it, const GraphArgs& G, int64_t rel, bool first, RWC_LDS uint32_t* err,
                     RWC_LDS uint64_t* red) {
        const int32_t walk_share = __builtin_amdgcn_readfirstlane(it.slot0) ? kWalkShare : 0;
        if (G.n <= kPopLdsCounts)
            pop_item<kStrat, true, kPerThread>(A, dumps, G, it.graph, rel, walk_share, first, lds,
                                               (RWC_LDS uint32_t*)counters, err, red);
        else
            pop_item<kStrat, false, kPerThread>(A, dumps, G, it.graph, rel, walk_share, first, lds,
                                                (RWC_LDS uint32_t*)counters, err, red);
    });
}

// Adds the work-groups' sums to the totals of a single graph: 256 nodes and kPopSlots work-groups
// per block.
constexpr int kPopSlots = 64;

__global__ void __launch_bounds__(256) pop_reduce(const uint64_t* __restrict__ sums, int64_t stride, int32_t groups, int32_t n,
                           const int32_t* __restrict__ node_id, uint64_t* __restrict__ counts,
                           uint64_t* __restrict__ counts_sq) {
    const int32_t x = blockIdx.x * 256 + threadIdx.x;
    if (x >= n) return;
    const int32_t end = min(groups, (static_cast<int32_t>(blockIdx.y) + 1) * kPopSlots);
    uint64_t a = 0, b = 0;
#pragma unroll 8
    for (int32_t g = blockIdx.y * kPopSlots; g < end; ++g) {
        const uint64_t* const s = sums + static_cast<int64_t>(g) * 2 * stride + x;
        a += s[0];
        b += s[stride];
    }
    const int32_t id = node_id[x];
    if (a) atomicAdd(reinterpret_cast<unsigned long long*>(&counts[id]), static_cast<unsigned long long>(a));
    if (b && counts_sq) atomicAdd(reinterpret_cast<unsigned long long*>(&counts_sq[id]), static_cast<unsigned long long>(b));
}

// kPerThread nodes per thread.  Up to 8192 nodes: eight waves per SIMD (64 registers), so that two
// work-groups of kPopMaxThreads fill a compute unit; above, the LDS holds one work-group.
template <int kPerThread>
__global__ void __launch_bounds__(kPopMaxThreads, kPerThread <= 8 ? 8 : 4) cycle_pop(PopArgs A, DumpArgs dumps) {
    extern __shared__ uint32_t pop_lds[];
    pop_graphs<false, kPerThread>(A, dumps, (RWC_LDS uint32_t*)pop_lds);
}

template <int kPerThread>
__global__ void __launch_bounds__(kPopMaxThreads, kPerThread <= 8 ? 8 : 4) cycle_pop_strata(PopArgs A, DumpArgs dumps) {
    extern __shared__ uint32_t pop_lds[];
    pop_graphs<true, kPerThread>(A, dumps, (RWC_LDS uint32_t*)pop_lds);
}

}  // namespace
}  // namespace rwc
