// rwc_build_csr: edge list -> symmetric CSR with sorted rows, integer CDF rows, weighted
// degrees, vol, pivot and a connectivity check, all on the GPU.
//
// Internal order.  On a graph with a heavy degree tail (largest degree above four times the
// mean) nodes are stored by descending weighted degree, ties by ascending input id, so the
// pivot is internal index 0 and the nodes a random walk visits most share cache lines: their
// per-tree state words, records and rows (R-MAT scale 23: the walk 20 % faster).  Otherwise
// the internal order is the input order.  Only memory placement changes: the records carry
// each node's input id, rows list neighbours by ascending input id, and everything the caller
// sees is indexed by input id, so every result is the same in either order.
//
// The 2m directed entries are sorted once, by (input id of the row, input id of the neighbour),
// with an LSD radix sort, which makes the CSR a deterministic function of the edge set.  Degrees
// and weighted degrees are then sums over contiguous rows (no atomics on hub counters: those
// took 1.6 ms of a 5.3 ms build of BA(10^6, 5), weighted); the internal order is a sort of the n
// nodes, and whole rows are copied to their internal place.
//
// Connectivity comes from the breadth-first search that orders the start nodes: when it reaches
// every node there is one component.  Only otherwise does a lock-free union-find over the input
// edges label the components: roots are always hooked from the larger id to the smaller one
// with a compare-and-swap, so every parent pointer decreases and every find terminates.
#include <utility>

#include "common.hpp"
#include "device.hpp"

namespace rwc {
namespace {

constexpr int kBlock = 256;
constexpr int kItems = 8;
constexpr int kTile = kBlock * kItems;

struct BuildScalars {
    uint32_t status;
    int32_t max_deg;
    uint64_t max_s;       // largest weighted degree (fixed point)
    uint64_t vol_fixed;
    int32_t pivot_id;     // input id of the pivot: the largest weighted degree, smallest id
    int32_t nroots;       // components (union-find, only when the search missed a node)
    uint32_t bfs_tail;    // nodes the breadth-first search reached
    int32_t bfs_done;
    int32_t bfs_depth;
    float min_w, max_w;   // smallest and largest edge weight
};

// ------------------------------------------------------------------ exclusive scan -----
__device__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wave_tot, uint32_t* total) {
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, kWave);
        if (lane >= off) x += y;
    }
    if (lane == kWave - 1) wave_tot[wid] = x;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) {
        const uint32_t s = wave_tot[w];
        if (w < wid) pre += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return pre + x - v;
}

// Blocked arrangement: thread t owns elements [t*kItems, (t+1)*kItems) of its tile.
__global__ void scan_tile_sums(const uint32_t* __restrict__ in, int64_t len, uint32_t* __restrict__ sums) {
    __shared__ uint32_t wave_tot[kBlock / kWave];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kTile + threadIdx.x * kItems;
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i)
        if (base + i < len) s += in[base + i];
    uint32_t tot;
    block_exclusive_scan(s, wave_tot, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Exclusive scan of `count` tile sums in place by one block, chunk by chunk with a carry.
__global__ void scan_sums_single(uint32_t* __restrict__ sums, int64_t count) {
    __shared__ uint32_t wave_tot[kBlock / kWave];
    uint32_t carry = 0;
    for (int64_t c = 0; c < count; c += kTile) {
        const int64_t base = c + threadIdx.x * kItems;
        uint32_t v[kItems];
        uint32_t s = 0;
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            v[i] = (base + i < count) ? sums[base + i] : 0u;
            s += v[i];
        }
        uint32_t tot;
        uint32_t pre = block_exclusive_scan(s, wave_tot, &tot) + carry;
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            if (base + i < count) sums[base + i] = pre;
            pre += v[i];
        }
        carry += tot;
    }
}

__global__ void scan_tile_apply(const uint32_t* in, uint32_t* out, int64_t len, const uint32_t* __restrict__ sums) {
    __shared__ uint32_t wave_tot[kBlock / kWave];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kTile + threadIdx.x * kItems;
    uint32_t v[kItems];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        v[i] = (base + i < len) ? in[base + i] : 0u;
        s += v[i];
    }
    uint32_t tot;
    uint32_t pre = block_exclusive_scan(s, wave_tot, &tot) + sums[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        if (base + i < len) out[base + i] = pre;
        pre += v[i];
    }
}

// Exclusive scan of len uint32 values (in may equal out).  `sums` needs
// ceil(len / kTile) entries.  Up to kScanSingle values one block scans alone: three launches of
// a few microseconds each cost more than its 16 chunks.
constexpr int64_t kScanSingle = 16 * kTile;

int exclusive_scan(uint32_t* v, int64_t len, uint32_t* sums, hipStream_t s) {
    if (len <= 0) return RWC_OK;
    if (len <= kScanSingle) {
        hipLaunchKernelGGL(scan_sums_single, dim3(1), dim3(kBlock), 0, s, v, len);
    } else {
        const unsigned nb = blocks_for(len, kTile);
        hipLaunchKernelGGL(scan_tile_sums, dim3(nb), dim3(kBlock), 0, s, v, len, sums);
        hipLaunchKernelGGL(scan_sums_single, dim3(1), dim3(kBlock), 0, s, sums, static_cast<int64_t>(nb));
        hipLaunchKernelGGL(scan_tile_apply, dim3(nb), dim3(kBlock), 0, s, v, v, len, sums);
    }
    RWC_HIP(hipGetLastError());
    return RWC_OK;
}

// --------------------------------------------------------------- LSD radix sort -------
// A tile's elements are taken by its waves in order (wave w the w-th quarter) and by each wave
// 64 at a time, so (wave, round, lane) is the input order and ranks counted in it are stable.
template <class K>
__global__ void radix_hist(const K* __restrict__ keys, int64_t len, int shift, uint32_t* __restrict__ ghist, int nb) {
    __shared__ uint32_t hist[256];
    hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kTile;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t i = tile0 + r * kBlock + threadIdx.x;
        if (i < len) atomicAdd(&hist[static_cast<uint32_t>(keys[i] >> shift) & 0xFFu], 1u);
    }
    __syncthreads();
    ghist[static_cast<int64_t>(threadIdx.x) * nb + blockIdx.x] = hist[threadIdx.x];
}

// Ranks come from per-wave digit counters (no barrier between rounds); the tile is then put in
// digit order in LDS, so that each digit's run leaves as consecutive stores.
template <class K>
__global__ void __launch_bounds__(kBlock)
    radix_scatter(const K* __restrict__ kin, const int32_t* __restrict__ vin, K* __restrict__ kout,
                  int32_t* __restrict__ vout, int64_t len, int shift, const uint32_t* __restrict__ goff, int nb) {
    constexpr int kWaves = kBlock / kWave;
    __shared__ uint32_t wcnt[kWaves][256];   // digit counts of each wave, then its first rank
    __shared__ uint32_t first[256];          // the digit's first place in the tile
    __shared__ uint32_t base[256];           // its first place in the output, minus `first`
    __shared__ uint32_t wave_tot[kWaves];
    __shared__ K lk[kTile];
    __shared__ int32_t lv[kTile];
    const int t = threadIdx.x, lane = t & (kWave - 1), wid = t / kWave;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) wcnt[w][t] = 0;
    __syncthreads();
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const int64_t mine = tile0 + wid * (kTile / kWaves) + lane;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    K k[kItems];
    int32_t v[kItems];
    uint32_t rank[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t i = mine + r * kWave;
        k[r] = i < len ? kin[i] : K{0};
        v[r] = i < len ? vin[i] : 0;
    }
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const bool valid = mine + r * kWave < len;
        const uint32_t d = static_cast<uint32_t>(k[r] >> shift) & 0xFFu;
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            same &= bit ? bb : ~bb;
        }
        const uint32_t below = __popcll(same & lt_mask);
        uint32_t before = 0;   // this wave's earlier elements of the digit
        if (valid && below == 0) before = atomicAdd(&wcnt[wid][d], static_cast<uint32_t>(__popcll(same)));
        before = __shfl(before, valid ? __builtin_ctzll(same) : lane, kWave);
        rank[r] = before + below;
    }
    __syncthreads();
    uint32_t tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = wcnt[w][t];
        wcnt[w][t] = tot;
        tot += c;
    }
    uint32_t all;
    const uint32_t f = block_exclusive_scan(tot, wave_tot, &all);
    first[t] = f;
    base[t] = goff[static_cast<int64_t>(t) * nb + blockIdx.x] - f;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        if (mine + r * kWave < len) {
            const uint32_t d = static_cast<uint32_t>(k[r] >> shift) & 0xFFu;
            const uint32_t at = first[d] + wcnt[wid][d] + rank[r];
            lk[at] = k[r];
            lv[at] = v[r];
        }
    }
    __syncthreads();
    for (uint32_t i = t; i < all; i += kBlock) {
        const K x = lk[i];
        const uint32_t pos = base[static_cast<uint32_t>(x >> shift) & 0xFFu] + i;
        kout[pos] = x;
        vout[pos] = lv[i];
    }
}

// Sorts keys[0 .. len) by their low `bits` bits with their values; the sorted pair of arrays is
// left in *keys / *vals (the other pair is scratch).
template <class K>
int radix_sort(K** keys, K** keys_tmp, int32_t** vals, int32_t** vals_tmp, int64_t len, int bits, uint32_t* hist,
               uint32_t* sums, hipStream_t s) {
    const int nb = static_cast<int>(blocks_for(len, kTile));
    for (int sh = 0; sh < bits; sh += 8) {
        hipLaunchKernelGGL(radix_hist<K>, dim3(nb), dim3(kBlock), 0, s, *keys, len, sh, hist, nb);
        RWC_CHECK(exclusive_scan(hist, 256ll * nb, sums, s));
        hipLaunchKernelGGL(radix_scatter<K>, dim3(nb), dim3(kBlock), 0, s, *keys, *vals, *keys_tmp, *vals_tmp, len, sh,
                           hist, nb);
        RWC_HIP(hipGetLastError());
        std::swap(*keys, *keys_tmp);
        std::swap(*vals, *vals_tmp);
    }
    return RWC_OK;
}

// ----------------------------------------------------------------- build kernels ------
__global__ void init_scalars(BuildScalars* sc) { *sc = BuildScalars{}; }

// Checks every edge and writes its two directed entries' keys, (row << bits | neighbour) by
// input id.  A faulty edge gets the key 0, so that no later index derived from a key is out of
// range whatever the input held.
template <class K>
__global__ void entry_keys(int64_t m, const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                           const float* __restrict__ w, int32_t n, int bits, K* __restrict__ keys,
                           int32_t* __restrict__ vals, BuildScalars* sc) {
    uint32_t err = 0;
    for (int64_t e = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; e < m;
         e += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int32_t a = src[e], b = dst[e];
        if (a < 0 || a >= n || b < 0 || b >= n) {
            err |= kErrNodeRange;
            a = b = 0;
        } else if (a == b) {
            err |= kErrSelfLoop;
        }
        if (w) {
            const float x = w[e];
            // NaN fails both comparisons
            if (!(x >= 0.5f && x < 65536.0f)) err |= kErrWeight;
        }
        keys[2 * e] = (static_cast<K>(a) << bits) | static_cast<K>(b);
        keys[2 * e + 1] = (static_cast<K>(b) << bits) | static_cast<K>(a);
        vals[2 * e] = static_cast<int32_t>(2 * e);
        vals[2 * e + 1] = static_cast<int32_t>(2 * e + 1);
    }
    if (err) atomicOr(&sc->status, err);
}

// rows[u] = first entry of input node u's row (a binary search over the sorted keys), u = 0 .. n.
template <class K>
__global__ void row_bounds(int32_t n, int64_t nnz, int bits, const K* __restrict__ keys, int32_t* __restrict__ rows) {
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u <= n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int64_t lo = 0, hi = nnz;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (static_cast<int64_t>(keys[mid] >> bits) < u)
                lo = mid + 1;
            else
                hi = mid;
        }
        rows[u] = static_cast<int32_t>(lo);
    }
}

// Weight in fixed point: w is a float32 in [0.5, 65536), so w 2^24 is an exact integer below 2^40.
__device__ __forceinline__ uint64_t fixed_weight(float w) {
    return static_cast<uint64_t>(static_cast<double>(w) * 16777216.0);
}

// Sum that stops at 2^63: a row of 2^53 or more is rejected, and a long row of large weights must
// not wrap back under that bound first.
__device__ __forceinline__ uint64_t sat_add(uint64_t a, uint64_t b) {
    const uint64_t s = a + b;
    return (s < a || s > (1ull << 63)) ? (1ull << 63) : s;
}

// The row kernels.  kRowLanes lanes share a row; a row's loads form a chain (its bounds, its
// entries, what those point at), so a group of lanes works on kRowsAhead rows at once, each
// stage's loads for all of them before the next stage's.  Four neighbouring rows lie in one
// wave (they share cache lines), and consecutive fours go to different blocks, since hubs
// cluster at small indices (sixteen neighbouring rows per wave: 312 -> 446 us for the rows).  A block collects its rows of more than kLongRow entries in LDS
// and takes them with all its threads at the end; those past the list's end stay with their
// group.  (BA(10^6, 5), weighted: one row per group at a time took 276 us for the sums and
// 474 us for the rows.)
constexpr int kRowLanes = 16;
constexpr int kRowsAhead = 4;
constexpr int kLongRow = 256;
constexpr int kLongList = 256;
constexpr int kRowBlocks = 2048;   // largest grid of the row kernels (their partials are kept per block)

// Calls body(u[]) for every kRowsAhead rows of this thread's group.
template <class Body>
__device__ __forceinline__ void for_rows(int32_t n, Body body) {
    constexpr int kGroupsPerWave = kWave / kRowLanes;
    const int64_t nb = gridDim.x;
    const int64_t waves = nb * (kBlock / kWave);
    const int64_t first = (threadIdx.x / kWave) * nb + blockIdx.x;
    const int g = (threadIdx.x & (kWave - 1)) / kRowLanes;
    for (int64_t c = first; c * kGroupsPerWave < n; c += kRowsAhead * waves) {
        int64_t u[kRowsAhead];
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) u[q] = (c + q * waves) * kGroupsPerWave + g;
        body(u);
    }
}

struct RowPartial {
    uint64_t max_s, vol;
    int32_t arg, max_deg;   // input id of the largest row (smallest id on ties)
    float min_w, max_w;     // of the entries' weights
    uint32_t err, reserved;
};

__device__ __forceinline__ RowPartial no_rows() { return RowPartial{0, 0, 0x7FFFFFFF, 0, 65536.0f, 0.5f, 0, 0}; }

__device__ __forceinline__ void take_weight(RowPartial& p, float w) {
    p.min_w = fminf(p.min_w, w);
    p.max_w = fmaxf(p.max_w, w);
}

__device__ __forceinline__ void take_row(RowPartial& p, uint64_t S, int32_t u, int32_t deg) {
    if (S >= (1ull << 53)) p.err |= kErrStrength;
    // vol must stay an exact uint64: a wrap of the running sum is seen as a result smaller than
    // the row added
    if (p.vol + S < p.vol) p.err |= kErrVolume;
    p.vol += S;
    if (S > p.max_s || (S == p.max_s && u < p.arg)) {
        p.max_s = S;
        p.arg = u;
    }
    p.max_deg = deg > p.max_deg ? deg : p.max_deg;
}

__device__ __forceinline__ void merge_partial(RowPartial& p, const RowPartial& q) {
    if (p.vol + q.vol < p.vol) p.err |= kErrVolume;
    p.vol += q.vol;
    if (q.max_s > p.max_s || (q.max_s == p.max_s && q.arg < p.arg)) {
        p.max_s = q.max_s;
        p.arg = q.arg;
    }
    p.max_deg = q.max_deg > p.max_deg ? q.max_deg : p.max_deg;
    p.min_w = fminf(p.min_w, q.min_w);
    p.max_w = fmaxf(p.max_w, q.max_w);
    p.err |= q.err;
}

// Block-wide merge of the threads' partials; valid in thread 0.
__device__ __forceinline__ RowPartial block_merge(RowPartial p, RowPartial* lds) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        RowPartial q;
        q.max_s = __shfl_xor(p.max_s, off, kWave);
        q.vol = __shfl_xor(p.vol, off, kWave);
        q.arg = __shfl_xor(p.arg, off, kWave);
        q.max_deg = __shfl_xor(p.max_deg, off, kWave);
        q.min_w = __shfl_xor(p.min_w, off, kWave);
        q.max_w = __shfl_xor(p.max_w, off, kWave);
        q.err = __shfl_xor(p.err, off, kWave);
        merge_partial(p, q);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave] = p;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < static_cast<int>(blockDim.x) / kWave; ++w) merge_partial(p, lds[w]);
    return p;
}

// Weighted degree (fixed point) of every input row, the entries' weights in row order (fill_rows
// would gather them again: half of them are random lines), the repeated-edge check (equal
// neighbours in the sorted keys), and per-block partials of vol, the largest row, the largest degree and
// the range of the weights.
template <class K>
__global__ void __launch_bounds__(kBlock)
    row_sums(int32_t n, const K* __restrict__ keys, const int32_t* __restrict__ vals, const float* __restrict__ w,
             const int32_t* __restrict__ rows, float* __restrict__ wrow, uint64_t* __restrict__ sfix,
             RowPartial* __restrict__ parts) {
    __shared__ RowPartial lds[kBlock / kWave];
    __shared__ uint64_t lsum[kBlock / kWave];
    __shared__ int32_t long_rows[kLongList];
    __shared__ uint32_t nlong;
    if (threadIdx.x == 0) nlong = 0;
    __syncthreads();
    const int sub = threadIdx.x & (kRowLanes - 1);
    RowPartial p = no_rows();
    auto entry = [&](uint32_t i) -> uint64_t {
        if (i > 0 && keys[i - 1] == keys[i]) p.err |= kErrDupEdge;
        if (!w) return 1ull << 24;
        const float x = w[vals[i] >> 1];
        wrow[i] = x;
        take_weight(p, x);
        return fixed_weight(x);
    };
    for_rows(n, [&](const int64_t (&u)[kRowsAhead]) {
        int32_t beg[kRowsAhead], end[kRowsAhead];
        uint64_t S[kRowsAhead];
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            beg[q] = u[q] < n ? rows[u[q]] : 0;
            end[q] = u[q] < n ? rows[u[q] + 1] : 0;
        }
        // the first kRowLanes entries of every row, stage by stage
        K key[kRowsAhead], prev[kRowsAhead];
        int32_t e[kRowsAhead];
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            const uint32_t i = static_cast<uint32_t>(beg[q] + sub);
            const bool have = sub < end[q] - beg[q];
            key[q] = have ? keys[i] : K{1};
            prev[q] = have && i > 0 ? keys[i - 1] : K{0};
            e[q] = have && w ? vals[i] >> 1 : 0;
            if (have && i > 0 && prev[q] == key[q]) p.err |= kErrDupEdge;
        }
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            const bool have = sub < end[q] - beg[q];
            const float x = have && w ? w[e[q]] : 1.0f;
            if (have && w) {
                wrow[beg[q] + sub] = x;
                take_weight(p, x);
            }
            S[q] = have ? fixed_weight(x) : 0ull;
        }
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            const int32_t deg = end[q] - beg[q];
            if (deg > kLongRow) {
                uint32_t slot = 0;
                if (sub == 0) {
                    slot = atomicAdd(&nlong, 1u);
                    if (slot < kLongList) long_rows[slot] = static_cast<int32_t>(u[q]);
                }
                if (__shfl(slot, 0, kRowLanes) < kLongList) continue;
            }
            for (uint32_t i = position(beg[q], sub + kRowLanes); i < position(end[q]); i += kRowLanes)
                S[q] = sat_add(S[q], entry(i));
#pragma unroll
            for (int off = kRowLanes / 2; off > 0; off >>= 1) S[q] = sat_add(S[q], __shfl_xor(S[q], off, kWave));
            if (sub == 0 && u[q] < n) {
                sfix[u[q]] = S[q];
                take_row(p, S[q], static_cast<int32_t>(u[q]), deg);
            }
        }
    });
    __syncthreads();
    const uint32_t nl = nlong < kLongList ? nlong : kLongList;
    for (uint32_t j = 0; j < nl; ++j) {
        const int32_t u = long_rows[j];
        const int32_t beg = rows[u], end = rows[u + 1];
        uint64_t S = 0;
        for (uint32_t i = position(beg, threadIdx.x); i < position(end); i += kBlock) S = sat_add(S, entry(i));
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) S = sat_add(S, __shfl_xor(S, off, kWave));
        __syncthreads();
        if ((threadIdx.x & (kWave - 1)) == 0) lsum[threadIdx.x / kWave] = S;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int v = 1; v < kBlock / kWave; ++v) S = sat_add(S, lsum[v]);
            sfix[u] = S;
            take_row(p, S, u, end - beg);
        }
    }
    __syncthreads();
    p = block_merge(p, lds);
    if (threadIdx.x == 0) parts[blockIdx.x] = p;
}

__global__ void __launch_bounds__(kBlock) row_stats(int nparts, const RowPartial* __restrict__ parts, BuildScalars* sc) {
    __shared__ RowPartial lds[kBlock / kWave];
    RowPartial p = no_rows();
    for (int i = threadIdx.x; i < nparts; i += kBlock) merge_partial(p, parts[i]);
    p = block_merge(p, lds);
    if (threadIdx.x == 0) {
        sc->max_s = p.max_s;
        sc->vol_fixed = p.vol;
        sc->max_deg = p.max_deg;
        sc->pivot_id = p.arg;
        sc->min_w = p.min_w;
        sc->max_w = p.max_w;
        sc->status |= p.err;
    }
}

// Sort keys of the internal order: the strength below the largest (ascending key = descending
// strength), the input id as value; the stable sort keeps ties in ascending id.
__global__ void order_keys(int32_t n, const uint64_t* __restrict__ sfix, const BuildScalars* __restrict__ sc,
                           uint64_t* __restrict__ keys, int32_t* __restrict__ vals) {
    const uint64_t top = sc->max_s;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        keys[u] = top - sfix[u];
        vals[u] = static_cast<int32_t>(u);
    }
}

// node_id (from the sorted values, or the identity), its inverse, and the degrees in internal
// order (the scan input for row_ptr; entry n is zero).
__global__ void invert_order(int32_t n, const int32_t* __restrict__ sorted, int32_t* __restrict__ node_id,
                             int32_t* __restrict__ node_index, const int32_t* __restrict__ rows,
                             uint32_t* __restrict__ deg) {
    for (int64_t x = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; x <= n;
         x += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        if (x == n) {
            deg[x] = 0;
            continue;
        }
        const int32_t id = sorted ? sorted[x] : static_cast<int32_t>(x);
        node_id[x] = id;
        node_index[id] = static_cast<int32_t>(x);
        deg[x] = static_cast<uint32_t>(rows[id + 1] - rows[id]);
    }
}

template <int kLanes>
__device__ __forceinline__ uint64_t lanes_incl_scan_u64(uint64_t x, int sub) {
#pragma unroll
    for (int off = 1; off < kLanes; off <<= 1) {
        const uint64_t y = __shfl_up(x, off, kLanes);
        if (sub >= off) x += y;
    }
    return x;
}

struct RowOut {
    int32_t* col;
    int32_t* edge_id;
    float* weight;
    uint64_t* cdf;   // null for unweighted graphs
};

// Copies every row to its internal place (column, edge, weight), with the integer CDF, the
// weighted degree and the 64-byte node record (layout in device.hpp): the record gives a walker
// the degree, the row offset and the row's first neighbours (with their CDF values and the row's
// total when weighted) in one aligned load.  A row's sixteen lanes hold one word of its record
// each, so it leaves as one 64-byte store.
template <class K>
__global__ void __launch_bounds__(kBlock)
    fill_rows(int32_t n, int bits, const K* __restrict__ keys, const int32_t* __restrict__ vals,
              const float* __restrict__ wrow, const int32_t* __restrict__ rows, const uint64_t* __restrict__ sfix,
              const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ node_id,
              const int32_t* __restrict__ node_index, RowOut out, double* __restrict__ strength,
              uint32_t* __restrict__ rec) {
    static_assert(kRowLanes == kRecWords, "one record word per lane of a row");
    __shared__ uint64_t lsum[kBlock / kWave];
    __shared__ int32_t long_rows[kLongList];
    __shared__ uint32_t nlong;
    if (threadIdx.x == 0) nlong = 0;
    __syncthreads();
    const int sub = threadIdx.x & (kRowLanes - 1);
    const K mask = (static_cast<K>(1) << bits) - 1;
    // entry i of the sorted list -> entry o of the CSR; returns its fixed-point weight
    auto copy = [&](int64_t i, int64_t o, int32_t& c) -> uint64_t {
        c = node_index[static_cast<uint32_t>(keys[i] & mask)];
        const int32_t e = vals[i] >> 1;
        const float x = wrow ? wrow[i] : 1.0f;
        out.col[o] = c;
        out.edge_id[o] = e;
        out.weight[o] = x;
        return out.cdf ? fixed_weight(x) : 0ull;
    };
    // record words of the lanes of one row: c / W hold entry `sub` of the row (the first chunk)
    auto put_record = [&](int64_t x, int32_t beg, int32_t deg, int32_t id, int32_t c, uint64_t cd, uint64_t S) {
        const uint32_t cfirst =
            static_cast<uint32_t>(__shfl(c, sub >= kRecFirst ? sub - kRecFirst : 0, kRowLanes));
        const uint64_t cc = __shfl(cd, sub >= 8 ? (sub - 8) >> 1 : 0, kRowLanes);
        uint32_t word = 0;
        if (sub == 0)
            word = static_cast<uint32_t>(deg);
        else if (sub == 1)
            word = static_cast<uint32_t>(beg);
        else if (sub == kRecId)
            word = static_cast<uint32_t>(id);
        else if (out.cdf == nullptr)
            word = (sub - kRecFirst < deg) ? cfirst : 0u;   // kRecInline words 3 .. 15
        else if (sub < kRecFirst + kRecInlineWeighted)
            word = (sub - kRecFirst < deg) ? cfirst : 0u;
        else if (sub < 8)
            word = deg > 0 ? static_cast<uint32_t>(sub == 6 ? S : S >> 32) : 0u;
        else if (sub < 8 + 2 * kRecInlineWeighted && (sub - 8) / 2 < deg)
            word = static_cast<uint32_t>((sub & 1) ? cc >> 32 : cc);
        rec[static_cast<int64_t>(kRecWords) * x + sub] = word;
        if (sub == 0) strength[x] = static_cast<double>(S) * (1.0 / 16777216.0);
    };
    for_rows(n, [&](const int64_t (&x)[kRowsAhead]) {
        int32_t id[kRowsAhead], from[kRowsAhead], beg[kRowsAhead], deg[kRowsAhead];
        uint64_t S[kRowsAhead];
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            id[q] = x[q] < n ? node_id[x[q]] : 0;
            beg[q] = x[q] < n ? row_ptr[x[q]] : 0;
            deg[q] = x[q] < n ? row_ptr[x[q] + 1] - beg[q] : 0;
        }
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            from[q] = rows[id[q]];
            S[q] = sfix[id[q]];
        }
        // the first kRowLanes entries of every row, stage by stage
        int32_t c[kRowsAhead], e[kRowsAhead];
        float wt[kRowsAhead];
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            const bool have = sub < deg[q];
            const int64_t i = static_cast<int64_t>(from[q]) + sub;
            c[q] = have ? static_cast<int32_t>(keys[i] & mask) : 0;
            e[q] = have ? vals[i] >> 1 : 0;
            wt[q] = have && wrow ? wrow[i] : 1.0f;
        }
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) c[q] = node_index[c[q]];
#pragma unroll
        for (int q = 0; q < kRowsAhead; ++q) {
            if (x[q] >= n) continue;
            if (deg[q] > kLongRow) {
                uint32_t slot = 0;
                if (sub == 0) {
                    slot = atomicAdd(&nlong, 1u);
                    if (slot < kLongList) long_rows[slot] = static_cast<int32_t>(x[q]);
                }
                if (__shfl(slot, 0, kRowLanes) < kLongList) continue;
            }
            const bool have = sub < deg[q];
            const int64_t o = static_cast<int64_t>(beg[q]) + sub;
            if (have) {
                out.col[o] = c[q];
                out.edge_id[o] = e[q];
                out.weight[o] = wt[q];
            }
            uint64_t cd = 0, carry = 0;
            if (out.cdf) {
                cd = lanes_incl_scan_u64<kRowLanes>(have ? fixed_weight(wt[q]) : 0ull, sub);
                if (have) out.cdf[o] = cd;
                carry = __shfl(cd, kRowLanes - 1, kRowLanes);
            }
            put_record(x[q], beg[q], deg[q], id[q], c[q], cd, S[q]);
            for (int32_t b0 = kRowLanes; b0 < deg[q]; b0 += kRowLanes) {
                const int32_t i = b0 + sub;
                int32_t cc = 0;
                const uint64_t W = i < deg[q] ? copy(static_cast<int64_t>(from[q]) + i, static_cast<int64_t>(beg[q]) + i, cc)
                                              : 0ull;
                if (out.cdf) {
                    const uint64_t y = carry + lanes_incl_scan_u64<kRowLanes>(W, sub);
                    if (i < deg[q]) out.cdf[beg[q] + i] = y;
                    carry = __shfl(y, kRowLanes - 1, kRowLanes);
                }
            }
        }
    });
    __syncthreads();
    const uint32_t nl = nlong < kLongList ? nlong : kLongList;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    for (uint32_t j = 0; j < nl; ++j) {
        const int32_t x = long_rows[j];
        const int32_t beg = row_ptr[x], deg = row_ptr[x + 1] - beg;
        const int32_t id = node_id[x];
        const int32_t from = rows[id];
        uint64_t carry = 0;
        for (int32_t b0 = 0; b0 < deg; b0 += kBlock) {
            const int32_t i = b0 + static_cast<int32_t>(threadIdx.x);
            int32_t c = 0;
            const uint64_t W = i < deg ? copy(static_cast<int64_t>(from) + i, static_cast<int64_t>(beg) + i, c) : 0ull;
            uint64_t cd = 0;
            if (out.cdf) {
                const uint64_t s = lanes_incl_scan_u64<kWave>(W, lane);
                __syncthreads();
                if (lane == kWave - 1) lsum[wid] = s;
                __syncthreads();
                uint64_t pre = carry;
#pragma unroll
                for (int v = 0; v < kBlock / kWave; ++v) {
                    const uint64_t y = lsum[v];
                    if (v < wid) pre += y;
                    carry += y;
                }
                cd = pre + s;
                if (i < deg) out.cdf[beg + i] = cd;
            }
            if (b0 == 0 && threadIdx.x < kRowLanes) put_record(x, beg, deg, id, c, cd, sfix[id]);
        }
    }
}

// Breadth-first order from the pivot, built in place: order[0..tail) is the queue; each level
// expands order[lo, hi) and appends newly reached nodes.  The order within a level follows
// the atomics and is not reproducible; nothing that depends on it is observable except speed
// (any start order yields the same forest).

// The frontier bounds live on the device, so that levels are launched without a host round trip
// each.  A level of few nodes and entries costs its latency, not its work, so one block runs such
// levels back to back inside one launch (bfs_narrow: 480 levels of a 97 013-node mesh took 4.1 ms
// of device time and as much again between the launches as three launches each; small graphs
// need no other kernel).  It stops at a wide level, which bfs_level and bfs_long expand over the
// whole device; the next bfs_narrow launch moves to the nodes they appended.
constexpr int32_t kBfsLongRow = 4096;   // frontier rows longer than this are shared by every wave
constexpr int kBfsLongRows = 256;       // such rows one level defers (any more expand in place)

struct BfsState {
    uint32_t tail;    // nodes in the queue so far
    uint32_t lo, hi;  // the frontier of the level that the wide kernels expand
    int32_t level;    // its distance from the pivot
    int32_t done;     // no frontier left: further launches return at once
    int32_t up;       // the level is expanded from the unreached nodes (bfs_up)
    uint32_t nlong;   // long frontier rows deferred to bfs_long this level
    int32_t long_rows[kBfsLongRows];
};

// Newly reached nodes collect in a per-wave LDS buffer of kBfsBuf entries, which goes to the
// queue with one atomic on its tail when it cannot take another 64 (and when the wave ends).
constexpr int kBfsBuf = 512;

struct BfsBuffer {
    int32_t* buf;   // this wave's kBfsBuf entries in LDS
    int32_t count;  // entries held (wave-uniform)
};

__device__ __forceinline__ void bfs_flush(BfsBuffer& b, int lane, int32_t* __restrict__ order, BfsState* st) {
    if (b.count == 0) return;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&st->tail, static_cast<uint32_t>(b.count));
    base = __shfl(base, 0, kWave);
    for (int32_t i = lane; i < b.count; i += kWave) order[base + i] = b.buf[i];
    b.count = 0;
}

// The last entries of a block's waves, with one atomic for the block (an atomic per wave on the one
// tail took 150 us a level at 16384 waves).
__device__ __forceinline__ void bfs_finish(const BfsBuffer& b, int lane, int32_t* __restrict__ order, BfsState* st) {
    __shared__ uint32_t count[kBlock / kWave];
    __shared__ uint32_t base;
    const int wid = threadIdx.x / kWave;
    if (lane == 0) count[wid] = static_cast<uint32_t>(b.count);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int w = 0; w < kBlock / kWave; ++w) {
            const uint32_t c = count[w];
            count[w] = total;
            total += c;
        }
        base = total ? atomicAdd(&st->tail, total) : 0u;
    }
    __syncthreads();
    const uint32_t at = base + count[wid];
    for (int32_t i = lane; i < b.count; i += kWave) order[at + i] = b.buf[i];
}

// Visits entry k of a row (lanes with `have`; the whole wave calls): a neighbour still unreached
// is claimed for the next level and buffered for the queue.
__device__ __forceinline__ void bfs_expand(bool have, uint32_t k, int lane, int32_t level,
                                           const int32_t* __restrict__ col, int32_t* __restrict__ dist,
                                           int32_t* __restrict__ order, BfsState* st, BfsBuffer& b) {
    int32_t w = 0;
    bool found = false;
    if (have) {
        w = col[k];
        found = dist[w] == -1 && atomicCAS(&dist[w], -1, level + 1) == -1;
    }
    const uint64_t m = __ballot(found);
    if (m == 0) return;
    if (b.count > kBfsBuf - kWave) bfs_flush(b, lane, order, st);
    if (found) b.buf[b.count + __popcll(m & ((1ull << lane) - 1))] = w;
    b.count += __popcll(m);
}

// A wave takes four frontier nodes at a time, sixteen lanes over the neighbours of each (most rows
// are short: with a wave per node BA(10^6, 5)'s levels took 683 us); rows past
// kBfsGroupRow are then taken by the whole wave, and rows longer than kBfsLongRow go to bfs_long
// (up to kBfsLongRows of them), so a hub's row does not hold the level on one wave.
constexpr int kBfsLanes = 16;
constexpr int kBfsGroupRow = 128;

// Once the frontier outweighs the unreached nodes (Beamer, Asanovic, Patterson, "Direction-
// optimizing breadth-first search", SC 2012; their factor 14, on node counts), each unreached
// node looks for a neighbour on the frontier instead: few probes per node and no
// compare-and-swap per entry (a stale line of another XCD's L2 sends most of those out in vain).
constexpr int64_t kBfsUpFactor = 14;
constexpr int kBfsUpLanes = 8;

__device__ __forceinline__ void bfs_up(int32_t n, int64_t wave, int64_t nw, int lane, int32_t level,
                                       const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                       int32_t* __restrict__ dist, int32_t* __restrict__ order, BfsState* st,
                                       BfsBuffer& b) {
    constexpr int kRows = kWave / kBfsUpLanes;
    const int sub = lane & (kBfsUpLanes - 1);
    for (int64_t u0 = kRows * wave; u0 < n; u0 += kRows * nw) {
        const int64_t u = u0 + lane / kBfsUpLanes;
        int32_t beg = 0, end = 0;
        if (u < n && dist[u] == -1) {
            beg = row_ptr[u];
            end = row_ptr[u + 1];
        }
        const bool short_row = end - beg <= kBfsGroupRow;
        bool found = false;
        uint32_t k = position(beg), stop = short_row ? position(end) : k;
        while (__any(k < stop)) {
            const bool hit = k + sub < stop && dist[col[k + sub]] == level;
            const uint64_t m = __ballot(hit);
            if ((m >> (lane & ~(kBfsUpLanes - 1))) & ((1u << kBfsUpLanes) - 1u)) {
                found = true;
                stop = 0;
            }
            k += kBfsUpLanes;
        }
        uint64_t rest = __ballot(!short_row && sub == 0);
        while (rest) {   // longer rows: the whole wave, or every wave (bfs_long)
            const int src = __builtin_ctzll(rest);
            rest &= rest - 1;
            const uint32_t rb = __shfl(position(beg), src, kWave), re = __shfl(position(end), src, kWave);
            if (re - rb > kBfsLongRow) {
                uint32_t slot = 0;
                if (lane == src) {
                    slot = atomicAdd(&st->nlong, 1u);
                    if (slot < kBfsLongRows) st->long_rows[slot] = static_cast<int32_t>(u);
                }
                if (__shfl(slot, src, kWave) < kBfsLongRows) continue;
            }
            for (uint32_t k0 = rb; k0 < re; k0 += kWave)
                if (__any(k0 + lane < re && dist[col[k0 + lane]] == level)) {
                    found = found || lane == src;
                    break;
                }
        }
        found = found && sub == 0;
        if (found) dist[u] = level + 1;
        const uint64_t m = __ballot(found);
        if (m == 0) continue;
        if (b.count > kBfsBuf - kWave) bfs_flush(b, lane, order, st);
        if (found) b.buf[b.count + __popcll(m & ((1ull << lane) - 1))] = static_cast<int32_t>(u);
        b.count += __popcll(m);
    }
}

__global__ void bfs_level(int32_t n, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                          int32_t* __restrict__ dist, int32_t* __restrict__ order, BfsState* st) {
    if (st->done) return;
    const uint32_t lo = st->lo, hi = st->hi;
    const int32_t level = st->level;
    const int lane = threadIdx.x & (kWave - 1);
    constexpr int kRows = kWave / kBfsLanes;
    const int64_t wave = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) +
                         __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t nw = static_cast<int64_t>(gridDim.x) * blockDim.x / kWave;
    __shared__ int32_t lds[kBlock / kWave][kBfsBuf];
    BfsBuffer b{lds[threadIdx.x / kWave], 0};
    if (st->up) {
        bfs_up(n, wave, nw, lane, level, row_ptr, col, dist, order, st, b);
        bfs_finish(b, lane, order, st);
        return;
    }
    for (int64_t i0 = lo + kRows * wave; i0 < hi; i0 += kRows * nw) {
        const int64_t i = i0 + lane / kBfsLanes;
        int32_t u = 0, beg = 0, end = 0;
        if (i < hi) {
            u = order[i];
            beg = row_ptr[u];
            end = row_ptr[u + 1];
        }
        const bool short_row = end - beg <= kBfsGroupRow;
        const uint32_t stop = position(short_row ? end : beg);
        for (uint32_t k = position(beg, lane & (kBfsLanes - 1)); __any(k < stop); k += kBfsLanes)
            bfs_expand(k < stop, k, lane, level, col, dist, order, st, b);
        uint64_t rest = __ballot(!short_row && (lane & (kBfsLanes - 1)) == 0);
        while (rest) {
            const int src = __builtin_ctzll(rest);
            rest &= rest - 1;
            const uint32_t rb = __shfl(position(beg), src, kWave), re = __shfl(position(end), src, kWave);
            if (re - rb > kBfsLongRow) {
                uint32_t slot = 0;
                if (lane == src) {
                    slot = atomicAdd(&st->nlong, 1u);
                    if (slot < kBfsLongRows) st->long_rows[slot] = u;
                }
                if (__shfl(slot, src, kWave) < kBfsLongRows) continue;
            }
            for (uint32_t k0 = rb; k0 < re; k0 += kWave)
                bfs_expand(k0 + lane < re, k0 + lane, lane, level, col, dist, order, st, b);
        }
    }
    bfs_finish(b, lane, order, st);
}

// The level's long rows, every wave taking every nw-th 64-entry chunk of each.
__global__ void bfs_long(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                         int32_t* __restrict__ dist, int32_t* __restrict__ order, BfsState* st) {
    if (st->done) return;
    const uint32_t nl = st->nlong < kBfsLongRows ? st->nlong : kBfsLongRows;
    const int32_t level = st->level;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) +
                         __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t nw = static_cast<int64_t>(gridDim.x) * blockDim.x / kWave;
    __shared__ int32_t lds[kBlock / kWave][kBfsBuf];
    BfsBuffer b{lds[threadIdx.x / kWave], 0};
    for (uint32_t j = 0; j < nl; ++j) {
        const int32_t u = st->long_rows[j];
        const int32_t beg = row_ptr[u], end = row_ptr[u + 1];
        if (st->up) {
            // u is unreached: one neighbour on the frontier is enough
            bool hit = false;
            for (int64_t k0 = beg + wave * kWave; !hit && k0 < end; k0 += nw * kWave)
                hit = __any(k0 + lane < end && dist[col[k0 + lane]] == level);
            const bool found = hit && lane == 0 && atomicCAS(&dist[u], -1, level + 1) == -1;
            const uint64_t m = __ballot(found);
            if (m == 0) continue;
            if (b.count > kBfsBuf - kWave) bfs_flush(b, lane, order, st);
            if (found) b.buf[b.count] = u;
            b.count += 1;
            continue;
        }
        for (int64_t k0 = beg + wave * kWave; k0 < end; k0 += nw * kWave)
            bfs_expand(k0 + lane < end, static_cast<uint32_t>(k0) + lane, lane, level, col, dist, order, st, b);
    }
    bfs_finish(b, lane, order, st);
}

// Levels of up to kNarrowNodes nodes and kNarrowEdges entries in one block: eight lanes per row
// of up to kNarrowRow entries, one wave per row of up to kNarrowThreads, and all threads for a
// longer one.  `first`: the search starts here;
// otherwise the wide kernels have just expanded [lo, hi).
constexpr int kNarrowThreads = 1024;
constexpr int kNarrowNodes = 2048;
constexpr int kNarrowEdges = 16384;
constexpr int kNarrowRow = 64;

__global__ void __launch_bounds__(kNarrowThreads)
    bfs_narrow(int32_t n, bool first, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
               int32_t* __restrict__ dist, int32_t* __restrict__ order, BfsState* st, BuildScalars* sc) {
    __shared__ int32_t list[2][kNarrowNodes];
    __shared__ int2 row[kNarrowNodes];
    __shared__ uint32_t wsum[kNarrowThreads / kWave];
    __shared__ uint32_t found_count;
    if (st->done) return;
    const int t = threadIdx.x, lane = t & (kWave - 1), wid = t / kWave;
    uint32_t lo = first ? 0u : st->hi, hi = first ? 1u : st->tail;
    int32_t level = first ? 0 : st->level + 1;
    int cur = 0;
    bool listed = false;   // list[cur] holds the frontier
    __syncthreads();       // every thread has read the state before it is written below
    while (hi > lo) {
        const uint32_t size = hi - lo;
        if (size > kNarrowNodes) break;
        uint32_t edges = 0;
        bool wide = false;
        for (uint32_t i = t; i < size; i += kNarrowThreads) {
            const int32_t u = listed ? list[cur][i] : order[lo + i];
            const int2 r = make_int2(row_ptr[u], row_ptr[u + 1]);
            row[i] = r;
            // each term at most 2 kNarrowEdges, so that the sum cannot wrap
            const uint32_t d = static_cast<uint32_t>(r.y - r.x);
            edges += d < 2u * kNarrowEdges ? d : 2u * kNarrowEdges;
            wide = wide || d > kNarrowThreads;
        }
        edges = wave_sum(edges);
        if (lane == 0) wsum[wid] = edges;
        if (t == 0) found_count = 0;
        const bool any_wide = __syncthreads_or(wide) != 0;
        edges = 0;
        for (int w = 0; w < kNarrowThreads / kWave; ++w) edges += wsum[w];
        if (edges > kNarrowEdges) break;
        auto visit = [&](uint32_t k) {
            const int32_t w = col[k];
            if (dist[w] == -1 && atomicCAS(&dist[w], -1, level + 1) == -1) {
                const uint32_t slot = atomicAdd(&found_count, 1u);
                order[hi + slot] = w;
                if (slot < kNarrowNodes) list[cur ^ 1][slot] = w;
            }
        };
        for (uint32_t i = t / 8; i < size; i += kNarrowThreads / 8) {
            const int2 r = row[i];
            if (r.y - r.x <= kNarrowRow)
                for (uint32_t k = position(r.x, t & 7); k < position(r.y); k += 8) visit(k);
        }
        for (uint32_t i = wid; i < size; i += kNarrowThreads / kWave) {
            const int2 r = row[i];
            if (r.y - r.x > kNarrowRow && r.y - r.x <= kNarrowThreads)
                for (uint32_t k = position(r.x, lane); k < position(r.y); k += kWave) visit(k);
        }
        if (any_wide)   // at most kNarrowEdges / kNarrowThreads such rows
            for (uint32_t i = 0; i < size; ++i) {
                const int2 r = row[i];
                if (r.y - r.x > kNarrowThreads)
                    for (uint32_t k = position(r.x, t); k < position(r.y); k += kNarrowThreads) visit(k);
            }
        __syncthreads();
        const uint32_t found = found_count;
        __syncthreads();   // found_count and wsum are rewritten by the next level
        lo = hi;
        hi += found;
        ++level;
        cur ^= 1;
        listed = found <= kNarrowNodes;
    }
    if (t == 0) {
        const bool done = hi == lo;
        st->lo = lo;
        st->hi = hi;
        st->tail = hi;
        st->level = level;
        st->nlong = 0;
        st->up = kBfsUpFactor * (hi - lo) > n - static_cast<int64_t>(hi) ? 1 : 0;
        st->done = done ? 1 : 0;
        sc->bfs_tail = hi;
        sc->bfs_done = done ? 1 : 0;
        sc->bfs_depth = done ? level - 1 : level;
    }
}

__global__ void bfs_init(int32_t n, int32_t pivot, int32_t* __restrict__ dist, int32_t* __restrict__ order,
                         int32_t* __restrict__ component, BfsState* st) {
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        dist[u] = (u == pivot) ? 0 : -1;
        component[u] = 0;   // one component, unless the search misses a node
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        order[0] = pivot;
        st->tail = 1u;
        st->lo = 0u;
        st->hi = 1u;
        st->level = 0;
        st->done = 0;
        st->nlong = 0u;
    }
}

// Union-find with parent[x] <= x: find walks down to a root with path halving.
__device__ __forceinline__ int32_t uf_find(int32_t* parent, int32_t x) {
    int32_t p = parent[x];
    while (p != x) {
        const int32_t gp = parent[p];
        if (gp != p) parent[x] = gp;   // halving; any value written is an ancestor of x
        x = p;
        p = gp;
    }
    return x;
}

__global__ void uf_init(int32_t n, int32_t* parent) {
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x)
        parent[u] = static_cast<int32_t>(u);
}

__global__ void uf_hook(int64_t m, const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int32_t* parent) {
    for (int64_t e = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; e < m;
         e += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int32_t ra = uf_find(parent, src[e]);
        int32_t rb = uf_find(parent, dst[e]);
        // max(ra, rb) strictly decreases on every failed attempt, so this terminates.
        while (ra != rb) {
            const int32_t hi = ra > rb ? ra : rb, lo = ra > rb ? rb : ra;
            const int32_t old = atomicCAS(&parent[hi], hi, lo);
            if (old == hi) break;
            ra = uf_find(parent, old);
            rb = uf_find(parent, lo);
        }
    }
}

// component[u] = the smallest input id of u's component (the union-find root).
__global__ void uf_flatten(int32_t n, int32_t* parent, int32_t* __restrict__ component) {
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x)
        component[u] = uf_find(parent, static_cast<int32_t>(u));
}

// The nodes a breadth-first search from the pivot did not reach (other components), appended
// to its order in internal order: flags, their exclusive scan, then the scatter.
__global__ void unreached_flags(int32_t n, const int32_t* __restrict__ dist, uint32_t* __restrict__ flags) {
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u <= n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x)
        flags[u] = (u < n && dist[u] < 0) ? 1u : 0u;
}

__global__ void append_unreached(int32_t n, uint32_t tail, const int32_t* __restrict__ dist,
                                 const uint32_t* __restrict__ pos, int32_t* __restrict__ order) {
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x)
        if (dist[u] < 0) order[tail + pos[u]] = static_cast<int32_t>(u);
}

__global__ void uf_count_roots(int32_t n, const int32_t* __restrict__ parent, BuildScalars* sc) {
    int32_t c = 0;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x)
        c += (parent[u] == u);
    c = wave_sum(c);
    if ((threadIdx.x & (kWave - 1)) == 0 && c) atomicAdd(&sc->nroots, c);
}

int key_bits(int32_t n) {
    int b = 1;
    while (b < 31 && (static_cast<int64_t>(1) << b) < n) ++b;
    return b;
}

struct BuildLayout {
    int32_t* row_ptr;
    int32_t* col;
    float* weight;
    int32_t* edge_id;
    uint64_t* cdf;
    double* strength;
    uint32_t* rec;
    int32_t* bfs_order;
    int32_t* node_id;
    int32_t* node_index;
    int32_t* component;
    BuildScalars* scalars;
    size_t persistent;
    // scratch
    int32_t* rows;       // [n + 1] first sorted entry of each input node
    uint64_t* sfix;      // [n] weighted degree by input id, fixed point
    uint64_t* nkeys_a;   // node sort
    uint64_t* nkeys_b;
    int32_t* nvals_a;
    int32_t* nvals_b;
    uint64_t* keys_a;    // entry sort
    uint64_t* keys_b;
    int32_t* vals_a;
    int32_t* vals_b;
    uint32_t* hist;
    uint32_t* sums;
    RowPartial* parts;
    BfsState* bfs;
    size_t total;
};

BuildLayout carve_build(void* ws, int32_t n, int64_t m, bool weighted) {
    Carver c(ws);
    BuildLayout L{};
    const int64_t nnz = 2 * m;
    L.row_ptr = c.take<int32_t>(static_cast<size_t>(n) + 1);
    L.col = c.take<int32_t>(nnz);
    L.weight = c.take<float>(nnz);
    L.edge_id = c.take<int32_t>(nnz);
    L.cdf = weighted ? c.take<uint64_t>(nnz) : nullptr;
    L.strength = c.take<double>(n);
    L.rec = c.take<uint32_t>(static_cast<size_t>(kRecWords) * n);
    L.bfs_order = c.take<int32_t>(n);
    L.node_id = c.take<int32_t>(n);
    L.node_index = c.take<int32_t>(n);
    L.component = c.take<int32_t>(n);
    L.scalars = c.take<BuildScalars>(1);
    L.persistent = c.used();
    L.rows = c.take<int32_t>(static_cast<size_t>(n) + 1);
    L.sfix = c.take<uint64_t>(n);
    L.nkeys_a = c.take<uint64_t>(n);
    L.nkeys_b = c.take<uint64_t>(n);
    L.nvals_a = c.take<int32_t>(n);
    L.nvals_b = c.take<int32_t>(n);
    L.keys_a = c.take<uint64_t>(nnz);
    L.keys_b = c.take<uint64_t>(nnz);
    L.vals_a = c.take<int32_t>(nnz);
    L.vals_b = c.take<int32_t>(nnz);
    // the sorts run over the 2m entries and over the n nodes
    const int64_t nb = blocks_for(nnz > n ? nnz : n, kTile);
    L.hist = c.take<uint32_t>(256 * nb);
    const int64_t scan_len = (256 * nb > n + 1) ? 256 * nb : static_cast<int64_t>(n) + 1;
    L.sums = c.take<uint32_t>(blocks_for(scan_len, kTile) + 1);
    L.parts = c.take<RowPartial>(kRowBlocks);
    L.bfs = c.take<BfsState>(1);
    L.total = c.used();
    return L;
}

int check_sizes(int32_t n, int64_t m) {
    if (n < 2) return fail(RWC_ERR_INVALID_ARG, "n = %d: a graph needs at least two nodes", n);
    if (m < 1) return fail(RWC_ERR_INVALID_ARG, "m = %lld: a graph needs at least one edge", (long long)m);
    if (n >= 0x7FFFFFFF) return fail(RWC_ERR_TOO_LARGE, "n = %d is too large", n);
    if (2 * m >= 0x7FFFFFFFll) return fail(RWC_ERR_TOO_LARGE, "2m = %lld entries exceed int32 offsets", (long long)(2 * m));
    return RWC_OK;
}

// Internal order by descending weighted degree on heavy-tailed graphs: max degree > 4 x mean.
bool ordered_by_strength(const BuildScalars& host, int32_t n, int64_t m) {
    return static_cast<int64_t>(host.max_deg) * n > 8 * m;
}

// Everything up to the finished rows, for sort keys of type K: validation, the entry sort, the
// row sums (one host look: input errors, and the largest strength, which decides the internal
// order and the passes of its sort), the internal order, and the rows.
template <class K, class Grid, class Read>
int build_rows(int32_t n, int64_t m, const int32_t* src, const int32_t* dst, const float* w, int bits,
               const BuildLayout& L, BuildScalars* host, hipStream_t s, Grid grid, Read read_scalars) {
    const int64_t nnz = 2 * m;
    K *keys = reinterpret_cast<K*>(L.keys_a), *keys_tmp = reinterpret_cast<K*>(L.keys_b);
    int32_t *vals = L.vals_a, *vals_tmp = L.vals_b;
    hipLaunchKernelGGL(entry_keys<K>, grid(m), dim3(kBlock), 0, s, m, src, dst, w, n, bits, keys, vals, L.scalars);
    RWC_CHECK(radix_sort(&keys, &keys_tmp, &vals, &vals_tmp, nnz, 2 * bits, L.hist, L.sums, s));
    hipLaunchKernelGGL(row_bounds<K>, grid(static_cast<int64_t>(n) + 1), dim3(kBlock), 0, s, n, nnz, bits, keys, L.rows);
    float* wrow = w ? reinterpret_cast<float*>(keys_tmp) : nullptr;   // the sort's spare array
    const unsigned want = blocks_for(n, kBlock / kRowLanes);
    const unsigned gr = want < kRowBlocks ? want : kRowBlocks;
    hipLaunchKernelGGL(row_sums<K>, dim3(gr), dim3(kBlock), 0, s, n, keys, vals, w, L.rows, wrow, L.sfix,
                       L.parts);
    hipLaunchKernelGGL(row_stats, dim3(1), dim3(kBlock), 0, s, static_cast<int>(gr), L.parts, L.scalars);
    RWC_CHECK(read_scalars(host));
    // faults of single edges are reported before those of rows
    const uint32_t edge_bits = host->status & (kErrNodeRange | kErrSelfLoop | kErrWeight);
    RWC_CHECK(device_error_to_status(edge_bits ? edge_bits : host->status));
    int32_t* sorted = nullptr;
    if (ordered_by_strength(*host, n, m)) {
        int sbits = 1;
        while (sbits < 64 && (host->max_s >> sbits) != 0) ++sbits;
        uint64_t *nk = L.nkeys_a, *nk_tmp = L.nkeys_b;
        int32_t* nv_tmp = L.nvals_b;
        sorted = L.nvals_a;
        hipLaunchKernelGGL(order_keys, grid(n), dim3(kBlock), 0, s, n, L.sfix, L.scalars, nk, sorted);
        RWC_CHECK(radix_sort(&nk, &nk_tmp, &sorted, &nv_tmp, n, sbits, L.hist, L.sums, s));
    }
    uint32_t* deg = reinterpret_cast<uint32_t*>(L.row_ptr);
    hipLaunchKernelGGL(invert_order, grid(static_cast<int64_t>(n) + 1), dim3(kBlock), 0, s, n, sorted, L.node_id,
                       L.node_index, L.rows, deg);
    RWC_CHECK(exclusive_scan(deg, static_cast<int64_t>(n) + 1, L.sums, s));
    const RowOut out{L.col, L.edge_id, L.weight, L.cdf};
    hipLaunchKernelGGL(fill_rows<K>, dim3(gr), dim3(kBlock), 0, s, n, bits, keys, vals, wrow, L.rows, L.sfix, L.row_ptr,
                       L.node_id, L.node_index, out, L.strength, L.rec);
    RWC_HIP(hipGetLastError());
    return RWC_OK;
}

}  // namespace
}  // namespace rwc

using namespace rwc;

extern "C" int rwc_build_csr_workspace(int32_t n, int64_t m, int32_t weighted, size_t* bytes) {
    clear_error();
    if (!bytes) return fail(RWC_ERR_INVALID_ARG, "bytes is null");
    RWC_CHECK(check_sizes(n, m));
    *bytes = carve_build(nullptr, n, m, weighted != 0).total;
    return RWC_OK;
}

extern "C" int rwc_csr_persistent_bytes(int32_t n, int64_t m, int32_t weighted, size_t* bytes) {
    clear_error();
    if (!bytes) return fail(RWC_ERR_INVALID_ARG, "bytes is null");
    RWC_CHECK(check_sizes(n, m));
    *bytes = carve_build(nullptr, n, m, weighted != 0).persistent;
    return RWC_OK;
}

extern "C" int rwc_build_csr(int32_t n, int64_t m, const int32_t* src, const int32_t* dst, const float* w,
                             void* ws, size_t ws_bytes, rwc_csr* out, void* stream) {
    return rwc_build_csr_ex(n, m, src, dst, w, 0u, ws, ws_bytes, out, stream);
}

extern "C" int rwc_build_csr_ex(int32_t n, int64_t m, const int32_t* src, const int32_t* dst, const float* w,
                                uint32_t flags, void* ws, size_t ws_bytes, rwc_csr* out, void* stream) {
    clear_error();
    if (!src || !dst || !out) return fail(RWC_ERR_INVALID_ARG, "src, dst and out must not be null");
    if (flags & ~static_cast<uint32_t>(RWC_BUILD_ALLOW_DISCONNECTED))
        return fail(RWC_ERR_INVALID_ARG, "unknown build flags 0x%x", flags);
    const bool allow_disconnected = (flags & RWC_BUILD_ALLOW_DISCONNECTED) != 0;
    RWC_CHECK(check_sizes(n, m));
    const bool weighted = (w != nullptr);
    const size_t need = carve_build(nullptr, n, m, weighted).total;
    RWC_CHECK(check_workspace(ws, ws_bytes, need));
    hipStream_t s = static_cast<hipStream_t>(stream);
    BuildLayout L = carve_build(ws, n, m, weighted);
    const int64_t nnz = 2 * m;
    const unsigned gs = 4096;  // grid-stride launches
    auto grid = [&](int64_t work) { return dim3(blocks_for(work, kBlock) < gs ? blocks_for(work, kBlock) : gs); };
    auto read_scalars = [&](BuildScalars* host) -> int {
        RWC_HIP(hipGetLastError());
        RWC_HIP(hipMemcpyAsync(host, L.scalars, sizeof(*host), hipMemcpyDeviceToHost, s));
        RWC_HIP(hipStreamSynchronize(s));
        return RWC_OK;
    };
    BuildScalars host{};
    hipLaunchKernelGGL(init_scalars, dim3(1), dim3(1), 0, s, L.scalars);
    // 32-bit keys while a (row, neighbour) pair fits them: half the sort's key traffic
    const int bits = key_bits(n);
    if (2 * bits <= 32)
        RWC_CHECK(build_rows<uint32_t>(n, m, src, dst, w, bits, L, &host, s, grid, read_scalars));
    else
        RWC_CHECK(build_rows<uint64_t>(n, m, src, dst, w, bits, L, &host, s, grid, read_scalars));
    const bool by_strength = ordered_by_strength(host, n, m);
    // descending strength with ties by id puts the pivot first
    const int32_t pivot_index = by_strength ? 0 : host.pivot_id;

    // breadth-first start order from the pivot; the host looks once per batch of launches, and
    // levels past the last return at once
    int32_t* dist = L.nvals_a;
    hipLaunchKernelGGL(bfs_init, grid(n), dim3(kBlock), 0, s, n, pivot_index, dist, L.bfs_order, L.component, L.bfs);
    hipLaunchKernelGGL(bfs_narrow, dim3(1), dim3(kNarrowThreads), 0, s, n, true, L.row_ptr, L.col, dist, L.bfs_order,
                       L.bfs, L.scalars);
    // every level of a graph within the narrow limits is narrow
    const bool all_narrow = n <= kNarrowNodes && nnz <= kNarrowEdges;
    // 16 nodes per wave and more, and no more blocks than the device holds at once
    const unsigned gw = blocks_for(n, 64) < 2048u ? blocks_for(n, 64) : 2048u;
    // small-world graphs have two to four wide levels; deep graphs with wide levels double the
    // number launched between two looks, up to 32
    int64_t launched = 0;
    for (int32_t steps = all_narrow ? 0 : 4;; steps = steps < 32 ? 2 * steps : 32) {
        for (int32_t c = 0; c < steps; ++c) {
            hipLaunchKernelGGL(bfs_level, dim3(gw), dim3(kBlock), 0, s, n, L.row_ptr, L.col, dist, L.bfs_order, L.bfs);
            hipLaunchKernelGGL(bfs_long, dim3(gw), dim3(kBlock), 0, s, L.row_ptr, L.col, dist, L.bfs_order, L.bfs);
            hipLaunchKernelGGL(bfs_narrow, dim3(1), dim3(kNarrowThreads), 0, s, n, false, L.row_ptr, L.col, dist,
                               L.bfs_order, L.bfs, L.scalars);
        }
        RWC_CHECK(read_scalars(&host));
        if (host.bfs_done) break;
        launched += steps;
        if (launched > n || all_narrow)
            return fail(RWC_ERR_HIP, "breadth-first search did not finish in %d levels", n);
    }
    host.nroots = 1;
    if (host.bfs_tail != static_cast<uint32_t>(n)) {
        // several components: label them (an array of the node sort, n words: the entry sort's hold 2m,
        // which isolated nodes make fewer)
        int32_t* parent = L.nvals_b;
        hipLaunchKernelGGL(uf_init, grid(n), dim3(kBlock), 0, s, n, parent);
        hipLaunchKernelGGL(uf_hook, grid(m), dim3(kBlock), 0, s, m, src, dst, parent);
        hipLaunchKernelGGL(uf_count_roots, grid(n), dim3(kBlock), 0, s, n, parent, L.scalars);
        hipLaunchKernelGGL(uf_flatten, grid(n), dim3(kBlock), 0, s, n, parent, L.component);
        const uint32_t reached = host.bfs_tail;
        RWC_CHECK(read_scalars(&host));
        if (!allow_disconnected)
            return fail(RWC_ERR_DISCONNECTED, "the graph has %d connected components", host.nroots);
        // the other components' nodes follow the pivot's component, in internal order
        uint32_t* pos = reinterpret_cast<uint32_t*>(L.nkeys_a);   // n + 1 counters; the sorts are done
        hipLaunchKernelGGL(unreached_flags, grid(static_cast<int64_t>(n) + 1), dim3(kBlock), 0, s, n, dist, pos);
        RWC_CHECK(exclusive_scan(pos, static_cast<int64_t>(n) + 1, L.sums, s));
        hipLaunchKernelGGL(append_unreached, grid(n), dim3(kBlock), 0, s, n, reached, dist, pos, L.bfs_order);
        RWC_HIP(hipGetLastError());
    }
    const int32_t depth = host.bfs_depth;

    rwc_csr g{};
    g.n = n;
    g.pivot = host.pivot_id;
    g.m = m;
    g.nnz = nnz;
    g.weighted = weighted ? 1 : 0;
    g.max_degree = host.max_deg;
    g.vol_fixed = host.vol_fixed;
    g.vol = static_cast<double>(host.vol_fixed) * (1.0 / 16777216.0);
    g.row_ptr = L.row_ptr;
    g.col = L.col;
    g.weight = L.weight;
    g.edge_id = L.edge_id;
    g.cdf = L.cdf;
    g.strength = L.strength;
    g.rec = L.rec;
    g.bfs_order = L.bfs_order;
    g.bfs_depth = depth;
    g.node_id = L.node_id;
    g.node_index = L.node_index;
    g.pivot_index = pivot_index;
    g.internal_order = by_strength ? 1 : 0;
    g.weight_ratio = weighted ? static_cast<double>(host.max_w) / static_cast<double>(host.min_w) : 1.0;
    g.components = host.nroots;
    g.component = L.component;
    *out = g;
    return RWC_OK;
}
