// Cycle popping in rounds (pop.hpp) on meshes, where a round has few cycles and a tree thousands of
// rounds: what counts is the time of a round.  Included by sampler.hip.
//
// Tokens.  Each node has the round its arrow last changed in, and nodes are ordered by (that round,
// index).  A token starts at every node whose arrow changed and follows the arrows, kTokenSteps
// per round.  A token from c that meets
//  * a node later in the order is dropped: a cycle through c would run through that node too;
//  * a node known to lead to the root: so does c; the nodes from c on are marked as known;
//  * c itself: a cycle, whose nodes are listed and take their next arrows.
// Of a cycle's nodes the last in the order changed when the cycle closed or before, nothing on
// the cycle changed since, and its token meets no later node, so it comes back: every cycle is
// found, and when no token is left there is none.  A token under way for several rounds may have
// passed nodes that changed behind it, so what it finds after its first round counts only if
// following the arrows from c again, as many steps, leads there too (for a cycle: over nodes
// before c only, so that c alone lists it).
//
// One word per node holds all a step asks: the round, the "leads to the root" mark and the arrow.
// Up to kTokenLdsNodes nodes the words are in LDS (16, 1 and 15 bits); above, in the workspace
// (the arrow as wide as the node indices, the round in the rest).
//
// Sweeps.  Nodes whose token has no room in the list (the first rounds change thousands of arrows) are
// marked in a bitmap, and in the next round every marked node follows its path to the end at
// once.  A path that goes round a cycle without its node (Brent's algorithm) needs no token: the
// node is on no cycle, and one that it comes to lie on later runs through a node changed later.  The
// first round is a sweep over all nodes, and so is the one after the rounds have run out of bits.
//
// A draw (its count, its generator and its record are a chain of 1.5 us and more) is not on the
// round's path: every node's next arrow lies ready, and while three quarters of the threads follow
// tokens the last quarter draws the arrows after those that the round before took (half of
// them: 97 013-node mesh, 300 trees 294 instead of 248 ms).
//
// What bounds it: the latency of a round, that is its longest chain of dependent reads (25 to 50),
// times the rounds, of the slowest trees twice the average.  Against walker teams (weighted meshes,
// 300 trees, walk and reduction): 1000 nodes 15.7 -> 3.5 ms, 5000 50 -> 15, 20 000 241 -> 44,
// 97 013 941 -> 248.  Steps per round: 8 or 32 instead of 16 are 0 to 10 % slower.
#pragma once

#include "pop.hpp"

namespace rwc {
namespace {

constexpr int kTokenSteps = 16;             // a multiple of 4
constexpr int32_t kTokenSmallNodes = 2048;   // five work-groups and more on a compute unit
constexpr int32_t kTokenMidNodes = 8000;     // two and more
constexpr int32_t kTokenLdsNodes = 20500;    // one
constexpr int32_t kTokenMaxNodes = 200000;   // three bitmaps of n bits in LDS

// The words of a tree.  Arrow in the low `bits` bits, mark above them, round in the rest.
template <bool kWide>
struct TokenTree;

template <>
struct TokenTree<false> {
    RWC_LDS uint32_t* node;
    RWC_LDS uint16_t* ready;   // each node's next arrow
    static constexpr uint32_t kBits = 15;
    __device__ uint32_t bits() const { return kBits; }
    __device__ uint32_t get(uint32_t v) const { return node[v]; }
    __device__ void set(uint32_t v, uint32_t w) const { node[v] = w; }
    __device__ uint32_t get_ready(uint32_t v) const { return ready[v]; }
    __device__ void set_ready(uint32_t v, uint32_t a) const { ready[v] = static_cast<uint16_t>(a); }
};

template <>
struct TokenTree<true> {
    RWC_GLOBAL uint32_t* node;
    RWC_GLOBAL uint32_t* ready;
    uint32_t width;
    __device__ uint32_t bits() const { return width; }
    __device__ uint32_t get(uint32_t v) const {
        return __hip_atomic_load(node + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ void set(uint32_t v, uint32_t w) const {
        __hip_atomic_store(node + v, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ uint32_t get_ready(uint32_t v) const {
        return __hip_atomic_load(ready + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ void set_ready(uint32_t v, uint32_t a) const {
        __hip_atomic_store(ready + v, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

// LDS of one work-group, in 4-byte words: the nodes' words and next arrows (unless wide), two
// token lists (origin, next node, round it started in), two lists of popped nodes (of this round
// and the last), the bitmaps of popped nodes past the list and (two) of nodes to sweep.
struct TokenLayout {
    int32_t nodes, ready_words, cap, bit_words;
    __host__ __device__ explicit TokenLayout(int32_t n)
        : nodes(n <= kTokenLdsNodes ? n : 0), ready_words((nodes + 1) / 2), cap(n <= kTokenMidNodes ? 512 : 1024),
          bit_words((n + 31) / 32) {}
    // origin and next node 2 words, start 1/2 word (two lists each); popped nodes 1 word (two lists)
    __host__ __device__ int32_t words() const { return nodes + ready_words + 7 * cap + 3 * bit_words; }
};

// Grows one tree; returns with the arrows and counts final.  Every thread of the work-group calls.
// cnt: the departure counts, in the workspace.  ctl: two sets of (tokens kept, nodes popped), and the
// errors found while tokens walk.  Every thread decides by itself whether a round is the last, so no
// word it looks at may change under another thread of a round further: *err is written between the
// two barriers of a round and read after the second, ctl written before the first and read after it.
template <bool kStrat, bool kWide>
__device__ __forceinline__ void token_tree(const GraphArgs& G, uint64_t sample, uint64_t seed, const TokenLayout& P,
                                           RWC_LDS uint32_t* lists, const TokenTree<kWide>& W, RWC_GLOBAL uint32_t* cnt,
                                           RWC_LDS uint32_t* ctl, RWC_LDS uint32_t* err) {
    const uint32_t n = static_cast<uint32_t>(G.n), cap = static_cast<uint32_t>(P.cap);
    const uint32_t words = static_cast<uint32_t>(P.bit_words);
    const uint32_t kDone = 1u << W.bits(), kArrow = kDone - 1u, kShift = W.bits() + 1u;
    const uint32_t kRound = ~0u << kShift, max_round = kRound >> kShift;
    RWC_LDS uint32_t* const origin = lists;              // [2][cap]
    RWC_LDS uint32_t* const ahead = origin + 2 * cap;    // [2][cap]
    RWC_LDS uint32_t* const popped = ahead + 2 * cap;    // [2][cap]
    RWC_LDS uint16_t* const starts = (RWC_LDS uint16_t*)(popped + 2 * cap);   // [2][cap]
    RWC_LDS uint32_t* const bits = popped + 3 * cap;
    RWC_LDS uint32_t* const marks = bits + words;        // [2][words]
    const uint32_t t = threadIdx.x, T = blockDim.x, walkers = T - T / 4;   // threads from `walkers` on draw
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    const uint32_t sw = static_cast<uint32_t>(sample);
    for (uint32_t i = t; i < words; i += T) {
        bits[i] = marks[words + i] = 0;
        marks[i] = ~0u;   // (bits past n are never looked at)
    }
    if (t < 5) ctl[t] = 0;
    for (uint32_t v = t; v < n; v += T) {
        const bool root = G.rootmask ? ((G.rootmask[v >> 5] >> (v & 31)) & 1u) != 0 : static_cast<int32_t>(v) == G.root;
        W.set(v, root ? kDone | v : pop_draw<kStrat>(G, v, 0, sw, k0, k1));
        if (!root) W.set_ready(v, pop_draw<kStrat>(G, v, 1, sw, k0, k1));
        cnt[v] = root ? 0u : 1u;
    }
    __syncthreads();
    // the nodes from c to one known to lead to the root do so too
    auto mark_path = [&](uint32_t c) {
        for (uint32_t x = c;;) {
            const uint32_t w = W.get(x);
            if (w & kDone) break;
            W.set(x, w | kDone);
            x = w & kArrow;
        }
    };
    // the `len` nodes of c's cycle, to the list or past its end to the bitmap
    auto list_cycle = [&](uint32_t c, uint32_t len, RWC_LDS uint32_t* found, RWC_LDS uint32_t* list) {
        const uint32_t base = lds_add(found, len);
        uint32_t x = c;
        for (uint32_t i = base; i < base + len; ++i) {
            if (i < cap)
                list[i] = x;
            else
                lds_or(&bits[x >> 5], 1u << (x & 31));
            x = W.get(x) & kArrow;
        }
    };
    // the arrow after the one that v has just taken
    auto draw_ahead = [&](uint32_t v, RWC_LDS uint32_t* error) {
        const uint32_t k = cnt[v] + 1u;
        cnt[v] = k;
        if (k >= kCntMax) lds_or(error, static_cast<uint32_t>(kErrCountOverflow));
        W.set_ready(v, pop_draw<kStrat>(G, v, k, sw, k0, k1));
    };
    bool sweep = true;
    uint32_t ntok = 0, round = 0, taken = 0;   // taken: listed nodes popped in the last round
    int cur = 0;
    uint64_t rounds = 0, departures = n;
    while (true) {
        const uint32_t a = cur * cap, b = (cur ^ 1) * cap;   // this round's and the next one's lists
        if (t >= walkers) {
            for (uint32_t i = t - walkers; i < taken; i += T - walkers) draw_ahead(popped[b + i], &ctl[4]);
        } else {
            for (uint32_t i = t; i < ntok; i += walkers) {
                const uint32_t c = origin[a + i], start = starts[a + i];
                uint32_t p = ahead[a + i];
                const uint32_t wc = W.get(c);
                // known to lead to the root, or changed since (and with a newer token)
                if ((wc & kDone) || (wc >> kShift) > start) continue;
                const uint32_t key = (wc & kRound) | c;
                uint32_t s = kTokenSteps * (round - start);   // steps before this round
                enum { kOn, kDrop, kLeads, kCycle } end = kOn;
                for (int j = 0; j < kTokenSteps / 4; ++j) {
                    const uint32_t w0 = W.get(p), p1 = w0 & kArrow, w1 = W.get(p1), p2 = w1 & kArrow, w2 = W.get(p2),
                                   p3 = w2 & kArrow, w3 = W.get(p3);
                    const bool e0 = p == c || (w0 & kDone) || ((w0 & kRound) | p) > key;
                    const bool e1 = p1 == c || (w1 & kDone) || ((w1 & kRound) | p1) > key;
                    const bool e2 = p2 == c || (w2 & kDone) || ((w2 & kRound) | p2) > key;
                    const bool e3 = p3 == c || (w3 & kDone) || ((w3 & kRound) | p3) > key;
                    if (!(e0 || e1 || e2 || e3)) {
                        p = w3 & kArrow;
                        s += 4;
                        continue;
                    }
                    const uint32_t at = e0 ? p : e1 ? p1 : e2 ? p2 : p3, w = e0 ? w0 : e1 ? w1 : e2 ? w2 : w3;
                    s += e0 ? 0 : e1 ? 1 : e2 ? 2 : 3;
                    end = at == c ? kCycle : (w & kDone) ? kLeads : kDrop;
                    break;
                }
                if (end == kDrop) continue;
                if (end == kOn) {
                    if (s > n) continue;   // further than a cycle is long: c is not on one
                    const uint32_t slot = b + lds_add(&ctl[2 * cur], 1u);
                    origin[slot] = c;
                    ahead[slot] = p;
                    starts[slot] = static_cast<uint16_t>(start);
                    continue;
                }
                if (start != round) {   // the way there, again
                    uint32_t x = wc & kArrow, w = W.get(x);
                    uint32_t j = 0;
                    for (; j < s && x != c && !(w & kDone) && ((w & kRound) | x) < key; ++j) {
                        x = w & kArrow;
                        w = W.get(x);
                    }
                    if (end == kCycle ? (x != c || j != s) : !(w & kDone)) continue;
                }
                if (end == kLeads)
                    mark_path(c);
                else
                    list_cycle(c, s + 1, &ctl[2 * cur + 1], popped + a);
            }
        }
        RWC_LDS uint32_t* const old_marks = marks + cur * words;
        RWC_LDS uint32_t* const new_marks = marks + (cur ^ 1) * words;
        if (sweep)
            for (uint32_t c = t; c < n; c += T) {
                if (!((old_marks[c >> 5] >> (c & 31)) & 1u)) continue;
                const uint32_t wc = W.get(c);
                if (wc & kDone) continue;
                const uint32_t key = (wc & kRound) | c;
                uint32_t p = wc & kArrow, mark = kDone, power = 4, lam = 0, len = 1;   // (no node is kDone)
                while (true) {
                    if (p == c) {
                        list_cycle(c, len, &ctl[2 * cur + 1], popped + a);
                        break;
                    }
                    const uint32_t w = W.get(p);
                    if (w & kDone) {
                        mark_path(c);
                        break;
                    }
                    if (((w & kRound) | p) > key || p == mark) break;
                    if (++lam == power) {
                        mark = p;
                        power <<= 1;
                        lam = 0;
                    }
                    p = w & kArrow;
                    ++len;
                }
            }
        __syncthreads();
        const uint32_t kept = ctl[2 * cur], npop = ctl[2 * cur + 1], late = ctl[4];
        ++round;
        // the popped nodes take their next arrows; their tokens follow the kept ones
        auto take = [&](uint32_t v, uint32_t slot) {
            const uint32_t next = W.get_ready(v);
            W.set(v, (round << kShift) | next);
            if (slot < cap) {
                origin[b + slot] = v;
                ahead[b + slot] = next;
                starts[b + slot] = static_cast<uint16_t>(round);
            } else {
                lds_or(&new_marks[v >> 5], 1u << (v & 31));
            }
        };
        taken = npop < cap ? npop : cap;
        for (uint32_t i = t; i < taken; i += T) take(popped[a + i], kept + i);
        if (npop > cap)   // the rest, with the draws in place
            for (uint32_t i = t; i < words; i += T) {
                for (uint32_t w = bits[i]; w != 0; w &= w - 1) {
                    const uint32_t v = 32 * i + static_cast<uint32_t>(__builtin_ctz(w));
                    take(v, cap);
                    draw_ahead(v, err);
                }
                bits[i] = 0;
            }
        if (sweep)
            for (uint32_t i = t; i < words; i += T) old_marks[i] = 0;   // the next round's new ones
        sweep = kept + npop > cap;
        ntok = kept + taken < cap ? kept + taken : cap;
        cur ^= 1;
        if (t < 2) ctl[2 * cur + t] = 0;   // the next round's
        if (t == 0) {
            // the walker teams' guard on iterations, which bounds the rounds and, times 64 walkers, the
            // departures
            departures += npop;
            if (++rounds > G.guard || departures / kWave > G.guard) lds_or(err, static_cast<uint32_t>(kErrStepLimit));
            if (late) lds_or(err, late);
        }
        __syncthreads();
        if (*err || (ntok == 0 && !sweep)) break;   // (no token: nothing was taken either)
        if (round == max_round || round == 0xFFFFu) {   // out of bits: all are equal again
            for (uint32_t v = t; v < n; v += T) W.set(v, W.get(v) & ~kRound);
            for (uint32_t i = t; i < words; i += T) marks[cur * words + i] = ~0u;
            ntok = round = 0;
            sweep = true;
            __syncthreads();
        }
    }
}

template <bool kStrat, bool kWide>
__device__ __forceinline__ void token_item(const PopArgs& A, const DumpArgs& dumps, const GraphArgs& G, int32_t graph,
                                           int64_t rel, bool first, RWC_LDS uint32_t* lds, RWC_LDS uint32_t* ctl,
                                           RWC_LDS uint32_t* err, RWC_LDS uint64_t* red) {
    const TokenLayout P(G.n);
    RWC_GLOBAL uint32_t* const slot = global_ptr(A.slots + static_cast<int64_t>(blockIdx.x) * A.slot_stride);
    TokenTree<kWide> W;
    if constexpr (kWide) {
        W.node = slot + G.stride;
        W.ready = slot + 2 * G.stride;
        W.width = 32u - static_cast<uint32_t>(__builtin_clz(static_cast<uint32_t>(G.n - 1)));
    } else {
        W.node = lds;
        W.ready = (RWC_LDS uint16_t*)(lds + P.nodes);
    }
    if (threadIdx.x == 0) *err = 0;
    token_tree<kStrat, kWide>(G, static_cast<uint64_t>(A.sample_begin + rel), A.seed, P, lds + P.nodes + P.ready_words, W,
                              slot, ctl, err);
    const uint32_t arrow = (1u << W.bits()) - 1u;
    finish_tree(
        A, dumps, G, graph, rel, first, [&](int32_t x) { return slot[x]; },
        [&](int32_t x) { return W.get(x) & arrow; }, err, red);
}

template <bool kStrat>
__device__ __forceinline__ void token_graphs(const PopArgs& A, const DumpArgs& dumps, RWC_LDS uint32_t* lds) {
    __shared__ uint32_t ctl[5];
    pop_items(A, [&](const Item& it, const GraphArgs& G, int64_t rel, bool first, RWC_LDS uint32_t* err,
                     RWC_LDS uint64_t* red) {
        if (G.n <= kTokenLdsNodes)
            token_item<kStrat, false>(A, dumps, G, it.graph, rel, first, lds, (RWC_LDS uint32_t*)ctl, err, red);
        else
            token_item<kStrat, true>(A, dumps, G, it.graph, rel, first, lds, (RWC_LDS uint32_t*)ctl, err, red);
    });
}

constexpr int kTokenThreads = 768;

__global__ void __launch_bounds__(kTokenThreads, 4) mesh_pop(PopArgs A, DumpArgs dumps) {
    extern __shared__ uint32_t pop_lds[];
    token_graphs<false>(A, dumps, (RWC_LDS uint32_t*)pop_lds);
}

__global__ void __launch_bounds__(kTokenThreads, 4) mesh_pop_strata(PopArgs A, DumpArgs dumps) {
    extern __shared__ uint32_t pop_lds[];
    token_graphs<true>(A, dumps, (RWC_LDS uint32_t*)pop_lds);
}

}  // namespace
}  // namespace rwc
