// rwc_estimate: the pivot solve and the assembly of AppRWC (Algorithm 1) for the FastWalk
// estimate of Algorithm 3.
//
// The pivot column of calL^+ that Algorithm 1 obtains from one Laplacian solve is expressed
// through the hitting times to the pivot v: h_u = H_uv solves L_v h = d_{-v} (the first-step
// equations multiplied by D, grounded at v), and (calL^+)_uv = sqrt(d_u d_v)(RWC_v - h_u)/vol.
// Substituting into Eq. (3) with (calL_v^{-1})_uu estimated by t~_u = C_u / l gives
//     RWC_u = vol t~_u / d_u - 2 h_u + RWC_v,   RWC_v = sum_u d_u h_u / vol.
// L_v is symmetric positive definite, so the solve is Jacobi-preconditioned conjugate
// gradients in FP64.  Dot products use fixed partials summed in a fixed order, so results are
// bitwise reproducible run to run.  This file is compiled without FMA contraction.
//
// Three forms of the same iteration, by size (what an iteration costs besides its bytes is launches
// and dependent reductions: as five launches it took 17-20 us whatever the graph):
//  * pcg_small: graphs whose rows fit the LDS of one work-group run the whole solve in one launch
//    (ER(300, 8), 30 iterations: the call 1153 -> 567 us);
//  * up to kPairNodes nodes, two launches per iteration: the new direction z + beta p is formed where it
//    is gathered, from (z, p) pairs of 16 bytes, and every block sums the partials of the
//    launch before by itself (97 013-node mesh: 37 -> 24 us an iteration with the gaps);
//  * above, where the gathers are the cost and a pair would double their bytes, the direction step
//    is a launch of its own.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "common.hpp"
#include "roots.hpp"
#include "device.hpp"

namespace rwc {
namespace {

constexpr int kBlock = 256;
constexpr int kMaxBlocks = 2048;
// The iteration's kernels: blocks of 1024 threads, no more than are resident, so that the partials
// every block sums are few.
constexpr int kIterBlock = 1024;
constexpr int kIterBlocks = 512;

struct Scalars {
    double rz[2];   // r^T z at the start of the iteration, by its parity
    double rr;      // r^T r
    double rr0;     // ||b||^2
    double rwc_v;   // RWC of the pivot (of the root set for the group estimate)
    int32_t done;   // the residual met the tolerance: later iteration kernels return at once
    int32_t iters;  // iterations completed
};

// Grounded nodes: the pivot v, or the root set of the group estimate (bitmap of n bits).
__device__ __forceinline__ bool grounded(const uint32_t* __restrict__ gmask, int32_t v, int64_t u) {
    return gmask ? ((gmask[u >> 5] >> (u & 31)) & 1u) != 0 : u == v;
}

// v plus its copy moved by a data-parallel-primitive pattern (zero where nothing arrives).
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, kRows, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, kRows, 0xF, false);
    return v + __hiloint2double(hi, lo);
}

// Sum over the wave, valid in lane 63 (no LDS round trips: row shifts by 1, 2, 4, 8, then the row
// totals broadcast to the next row and to the upper half).
__device__ __forceinline__ double wave_sum_last(double v) {
    v = dpp_add<0x111, 0xF>(v);
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);
    return dpp_add<0x143, 0xC>(v);
}

// Sum over the block in every thread.  `lds` holds a double per wave; it may be reused after another
// barrier.
__device__ __forceinline__ double block_sum(double v, double* lds) {
    v = wave_sum_last(v);
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < static_cast<int>(blockDim.x) / kWave; ++w) s += lds[w];
    return s;
}

__global__ void pcg_init(int32_t n, int32_t v, const uint32_t* __restrict__ gmask, const double* __restrict__ d,
                         double* __restrict__ x, double* __restrict__ r, double* __restrict__ z, double* __restrict__ p,
                         double2* __restrict__ zp, double* __restrict__ part, Scalars* sc) {
    __shared__ double lds[2][kIterBlock / kWave];
    double rz = 0.0, rr = 0.0;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const bool gu = grounded(gmask, v, u);
        const double ru = gu ? 0.0 : d[u];
        const double zu = gu ? 0.0 : ru / d[u];
        x[u] = 0.0;
        r[u] = ru;
        if (zp) {
            zp[u] = make_double2(zu, 0.0);
        } else {
            z[u] = zu;
            p[u] = 0.0;
        }
        rz += ru * zu;
        rr += ru * ru;
    }
    rz = block_sum(rz, lds[0]);
    rr = block_sum(rr, lds[1]);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = rz;
        part[2 * blockIdx.x + 1] = rr;
        if (blockIdx.x == 0) {
            sc->done = 0;
            sc->iters = 0;
        }
    }
}

// Start of iteration `it`, in every block: sums the partials of r^T z and r^T r that the last
// update left, decides whether the solve is done and returns beta through *beta.  Block 0 records
// the scalars (r^T z by parity: the other blocks still read the last one's).  True: stop.
__device__ __forceinline__ bool begin_iteration(int it, const double* __restrict__ part, int nparts, Scalars* sc,
                                                double tol2, double* beta, double (*lds)[kIterBlock / kWave]) {
    if (sc->done) return true;
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) {
        a += part[2 * i];
        b += part[2 * i + 1];
    }
    const double last = sc->rz[(it + 1) & 1];
    a = block_sum(a, lds[0]);
    b = block_sum(b, lds[1]);
    const bool done = it == 0 ? b == 0.0 : b <= tol2 * sc->rr0;
    *beta = (it == 0 || last == 0.0) ? 0.0 : a / last;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->rz[it & 1] = a;
        sc->rr = b;
        if (it == 0) sc->rr0 = b;
        sc->iters = it;
        if (done) sc->done = 1;
    }
    return done;
}

// Direction step of the three-launch form: p = z + beta p.  With one block and n = 0 it only looks
// at convergence (the end of a batch of launches).
__global__ void __launch_bounds__(kIterBlock)
    update_p(int it, int32_t n, int32_t v, const uint32_t* __restrict__ gmask, Scalars* sc, double tol2,
             const double* __restrict__ part, int nparts, const double* __restrict__ z, double* __restrict__ p) {
    __shared__ double lds[2][kIterBlock / kWave];
    double beta;
    if (begin_iteration(it, part, nparts, sc, tol2, &beta, lds)) return;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x)
        if (!grounded(gmask, v, u)) p[u] = z[u] + beta * p[u];
}

// The vector an iteration gathers: p itself, or z + beta p from pairs.
template <bool kPair>
struct Direction;
template <>
struct Direction<false> {
    const double* p;
    double beta;
    __device__ double at(int64_t c) const { return p[c]; }
};
template <>
struct Direction<true> {
    const double2* zp;
    double beta;
    __device__ double at(int64_t c) const {
        const double2 q = zp[c];
        return q.x + beta * q.y;
    }
};

// y = L_v p on the grounded system (row and column v removed, p_v kept at zero), with p^T y.  kLanes
// lanes share a short row (strided over its entries, then a shuffle reduction; four on graphs of at
// most three edges a node, a wave above 80, sixteen otherwise); which block takes it is said below.  Rows longer than
// 16 kLanes are left out of that pass and then taken one at a time, in order, by the whole block:
// block b takes those among b, b + nb, b + 2 nb, ... (nb blocks), so that hub rows, which cluster at
// small indices in power-law graphs, land in different blocks.
// kPair: starts the iteration, and stores the new direction of the rows in zp_out.
template <bool kPair, int kLanes>
__global__ void __launch_bounds__(kIterBlock)
    spmv_dot(int it, int32_t n, int32_t v, int32_t max_degree, const uint32_t* __restrict__ gmask, Scalars* sc, double tol2,
             const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, const float* __restrict__ weight,
             const double* __restrict__ d, const double* __restrict__ part_in, int nparts,
             const double* __restrict__ p_in, const double2* __restrict__ zp_in, double2* __restrict__ zp_out,
             double* __restrict__ ap, double* __restrict__ part) {
    constexpr int kLongRow = 16 * kLanes;
    constexpr int kWaves = kIterBlock / kWave;
    __shared__ double lds[2][kWaves];
    __shared__ uint64_t long_mask[kWaves];
    Direction<kPair> dir;
    if constexpr (kPair) {
        dir.zp = zp_in;
        if (begin_iteration(it, part_in, nparts, sc, tol2, &dir.beta, lds)) return;
    } else {
        dir.p = p_in;
        if (sc->done) return;
    }
    const int sub = threadIdx.x & (kLanes - 1);
    const int group = threadIdx.x / kLanes;
    constexpr int kGroups = kIterBlock / kLanes;
    const int64_t b = blockIdx.x, nb = gridDim.x;
    double acc = 0.0;
    // A hub's row is as much work as many others, so rows are dealt to the blocks, eight neighbours at a
    // time, which share cache lines (dealt one by one, four and eight at a time: BA(200 000, 5) 22.5, 17.9,
    // 17.3 us, R-MAT of scale 21 119, 108, 108).  Where there are no long rows (four lanes, no row over 64
    // entries: meshes, sparse random graphs) rows are alike enough that a block takes consecutive ones,
    // and each XCD's L2 a consecutive eighth of them, since blocks go round the XCDs (97 013-node mesh
    // 14.9 us dealt, 7.0 us consecutive).  Sparse graphs with hubs are dealt: there the rows that are just short
    // enough lie side by side in the first blocks (solve of BA(200 000, 2): 2.62 ms consecutive, 2.06 dealt
    // with sixteen lanes, 1.65 with four; a tree of 189 290 nodes with hubs 123, 107, 85 ms).
    constexpr int kXcds = 8;
    const bool in_order = kLanes == 4 && max_degree <= kLongRow;
    const int64_t x = b % kXcds, chunk = x * (nb / kXcds) + (x < nb % kXcds ? x : nb % kXcds) + b / kXcds;
    // A row's loads form a chain (bounds, entries, gathers).  The next row's bounds and this
    // row's d and p are loaded before this row's entries, and a lane loads four entries, then
    // their four gathers, before it adds them (in entry order), so fewer latencies follow one
    // another.
    const int64_t ustep = static_cast<int64_t>(kGroups) * nb;
    int64_t u = in_order ? chunk * kGroups + group : (b + (group / 8) * nb) * 8 + group % 8;
    int32_t beg = 0, end = 0;
    if (u < n) {
        beg = row_ptr[u];
        end = row_ptr[u + 1];
    }
    while (u < n) {
        const int64_t un = u + ustep;
        int32_t nbeg = 0, nend = 0;
        if (un < n) {
            nbeg = row_ptr[un];
            nend = row_ptr[un + 1];
        }
        if (end - beg <= kLongRow) {
            const double du = d[u];
            const double pu = dir.at(u);
            double s = 0.0;
            uint32_t k = position(beg, sub);
            const uint32_t stop = position(end);
            for (; k + 3 * kLanes < stop; k += 4 * kLanes) {
                int32_t c[4];
                float w[4];
                double x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    c[i] = col[k + i * kLanes];
                    w[i] = weight[k + i * kLanes];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = dir.at(c[i]);
#pragma unroll
                for (int i = 0; i < 4; ++i) s += static_cast<double>(w[i]) * x[i];
            }
            for (; k < stop; k += kLanes) s += static_cast<double>(weight[k]) * dir.at(col[k]);
#pragma unroll
            for (int off = kLanes / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
            if (sub == 0) {
                const double y = grounded(gmask, v, u) ? 0.0 : du * pu - s;
                ap[u] = y;
                if constexpr (kPair) zp_out[u].y = pu;
                acc += pu * y;
            }
        }
        u = un;
        beg = nbeg;
        end = nend;
    }
    for (int64_t base = max_degree > kLongRow ? b : n; base < n; base += kIterBlock * nb) {
        const int64_t w = base + threadIdx.x * nb;
        const bool is_long = w < n && row_ptr[w + 1] - row_ptr[w] > kLongRow;
        const uint64_t m = __ballot(is_long);
        __syncthreads();
        if ((threadIdx.x & (kWave - 1)) == 0) long_mask[threadIdx.x / kWave] = m;
        __syncthreads();
        int turn = 0;
        for (int wv = 0; wv < kWaves; ++wv) {
            uint64_t bits = long_mask[wv];
            while (bits) {
                const int bit = __builtin_ctzll(bits);
                bits &= bits - 1;
                const int64_t r = base + (wv * kWave + bit) * nb;
                const int32_t rb = row_ptr[r], re = row_ptr[r + 1];
                double s = 0.0;
                for (uint32_t k = position(rb, threadIdx.x); k < position(re); k += kIterBlock)
                    s += static_cast<double>(weight[k]) * dir.at(col[k]);
                s = block_sum(s, lds[turn]);
                turn ^= 1;   // the other array's readers have passed this sum's barrier
                if (threadIdx.x == 0) {
                    const double pr = dir.at(r);
                    const double y = grounded(gmask, v, r) ? 0.0 : d[r] * pr - s;
                    ap[r] = y;
                    if constexpr (kPair) zp_out[r].y = pr;
                    acc += pr * y;
                }
            }
        }
    }
    __syncthreads();
    acc = block_sum(acc, lds[0]);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// x += alpha p, r -= alpha A p, z = r / d, with r^T z and r^T r; alpha from the product's partials,
// summed by every block.
template <bool kPair>
__global__ void __launch_bounds__(kIterBlock)
    update_xr(int it, int32_t n, int32_t v, const uint32_t* __restrict__ gmask, const Scalars* __restrict__ sc,
              const double* __restrict__ part_in, int nparts, const double* __restrict__ d, double* __restrict__ x,
              double* __restrict__ r, double* __restrict__ z, const double* __restrict__ p, double2* __restrict__ zp,
              const double* __restrict__ ap, double* __restrict__ part) {
    __shared__ double lds[3][kIterBlock / kWave];
    if (sc->done) return;
    double pap = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) pap += part_in[i];
    pap = block_sum(pap, lds[2]);
    const double alpha = (pap != 0.0) ? sc->rz[it & 1] / pap : 0.0;
    double rz = 0.0, rr = 0.0;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        if (grounded(gmask, v, u)) {
            if constexpr (kPair) zp[u] = make_double2(0.0, 0.0);
            continue;
        }
        const double pu = kPair ? zp[u].y : p[u];
        x[u] = x[u] + alpha * pu;
        const double ru = r[u] - alpha * ap[u];
        const double zu = ru / d[u];
        r[u] = ru;
        if constexpr (kPair)
            zp[u].x = zu;
        else
            z[u] = zu;
        rz += ru * zu;
        rr += ru * ru;
    }
    rz = block_sum(rz, lds[0]);
    rr = block_sum(rr, lds[1]);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = rz;
        part[2 * blockIdx.x + 1] = rr;
    }
}

// ---------------------------------------------------------------------------------------
// The whole solve in one work-group: rows in LDS (16-bit columns, float weights unless they are
// all 1), p and A p's gathered sums in LDS, the node's x, r and d in the registers of its thread.
// What bounds it is the latency of an iteration's four barriers, two block sums and LDS gathers.
// Eight lanes share a row; a row of more than kSmallLongRow entries is taken by a wave.
// ---------------------------------------------------------------------------------------
constexpr int kSmallThreads = 1024;
constexpr int kSmallPerThread = 4;
constexpr int kSmallNodes = kSmallThreads * kSmallPerThread;
constexpr size_t kSmallLds = 152 * 1024;
constexpr int kSmallLanes = 8;
constexpr int kSmallLongRow = 128;

struct SmallLayout {
    size_t p, s, rows, col, weight, list, total;   // byte offsets
    __host__ __device__ SmallLayout(int32_t n, int64_t nnz, bool weighted) {
        p = 0;
        s = p + 8 * static_cast<size_t>(n);
        rows = s + 8 * static_cast<size_t>(n);
        weight = rows + 4 * (static_cast<size_t>(n) + 1);
        col = weight + (weighted ? 4 * static_cast<size_t>(nnz) : 0);
        list = col + 2 * static_cast<size_t>(nnz);
        total = list + 2 * static_cast<size_t>(nnz / kSmallLongRow + 1);   // long rows
    }
};

bool solves_small(const rwc_csr& g) {
    return g.n <= kSmallNodes && SmallLayout(g.n, g.nnz, g.weighted != 0).total <= kSmallLds;
}

__global__ void __launch_bounds__(kSmallThreads)
    pcg_small(int32_t n, int32_t nnz, bool weighted, int32_t v, const uint32_t* __restrict__ gmask,
              const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, const float* __restrict__ weight,
              const double* __restrict__ d, double vol, double tol2, int max_iter, double* __restrict__ x_out,
              Scalars* sc, WsHeader* header) {
    extern __shared__ __align__(16) unsigned char small_lds[];
    __shared__ double red[3][kSmallThreads / kWave];
    __shared__ uint32_t nlong;
    const SmallLayout L(n, nnz, weighted);
    double* const p = reinterpret_cast<double*>(small_lds + L.p);
    double* const sum = reinterpret_cast<double*>(small_lds + L.s);
    int32_t* const rows = reinterpret_cast<int32_t*>(small_lds + L.rows);
    float* const lw = reinterpret_cast<float*>(small_lds + L.weight);
    uint16_t* const lc = reinterpret_cast<uint16_t*>(small_lds + L.col);
    uint16_t* const list = reinterpret_cast<uint16_t*>(small_lds + L.list);
    const int t = threadIdx.x, lane = t & (kWave - 1);
    if (t == 0) nlong = 0;
    for (int i = t; i <= n; i += kSmallThreads) rows[i] = row_ptr[i];
    for (int i = t; i < nnz; i += kSmallThreads) {
        lc[i] = static_cast<uint16_t>(col[i]);
        if (weighted) lw[i] = weight[i];
    }
    double x[kSmallPerThread], r[kSmallPerThread], dd[kSmallPerThread], ap[kSmallPerThread];
    bool live[kSmallPerThread];
    double rz = 0.0, rr = 0.0;
#pragma unroll
    for (int i = 0; i < kSmallPerThread; ++i) {
        const int u = t + i * kSmallThreads;
        live[i] = u < n && !grounded(gmask, v, u);
        dd[i] = live[i] ? d[u] : 1.0;
        x[i] = 0.0;
        ap[i] = 0.0;
        r[i] = live[i] ? dd[i] : 0.0;
        const double z = r[i] / dd[i];
        if (u < n) p[u] = z;
        rz += r[i] * z;
        rr += r[i] * r[i];
    }
    __syncthreads();
    for (int u = t; u < n; u += kSmallThreads)
        if (rows[u + 1] - rows[u] > kSmallLongRow) list[atomicAdd(&nlong, 1u)] = static_cast<uint16_t>(u);
    rz = block_sum(rz, red[0]);
    rr = block_sum(rr, red[1]);
    const double rr0 = rr;
    bool done = rr0 == 0.0;
    int it = 0;
    const int sub = t & (kSmallLanes - 1);
    while (!done && it < max_iter) {
        // (p is complete: the barrier of the last block sum, or the one at the end of the loop)
        for (int u = t / kSmallLanes; u < n; u += kSmallThreads / kSmallLanes) {
            const int beg = rows[u], end = rows[u + 1];
            if (end - beg > kSmallLongRow) continue;
            double s = 0.0;
            for (int k = beg + sub; k < end; k += kSmallLanes)
                s += weighted ? static_cast<double>(lw[k]) * p[lc[k]] : p[lc[k]];
#pragma unroll
            for (int off = kSmallLanes / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
            if (sub == 0) sum[u] = s;
        }
        for (uint32_t j = t / kWave; j < nlong; j += kSmallThreads / kWave) {
            const int u = list[j];
            double s = 0.0;
            for (int k = rows[u] + lane; k < rows[u + 1]; k += kWave)
                s += weighted ? static_cast<double>(lw[k]) * p[lc[k]] : p[lc[k]];
            s = wave_sum_last(s);
            if (lane == kWave - 1) sum[u] = s;
        }
        __syncthreads();
        double pap = 0.0;
#pragma unroll
        for (int i = 0; i < kSmallPerThread; ++i) {
            const int u = t + i * kSmallThreads;
            if (live[i]) {
                ap[i] = dd[i] * p[u] - sum[u];
                pap += p[u] * ap[i];
            }
        }
        pap = block_sum(pap, red[2]);
        const double alpha = pap != 0.0 ? rz / pap : 0.0;
        double nrz = 0.0, z[kSmallPerThread];
        rr = 0.0;
#pragma unroll
        for (int i = 0; i < kSmallPerThread; ++i) {
            const int u = t + i * kSmallThreads;
            z[i] = 0.0;
            if (live[i]) {
                x[i] = x[i] + alpha * p[u];
                r[i] = r[i] - alpha * ap[i];
                z[i] = r[i] / dd[i];
                nrz += r[i] * z[i];
                rr += r[i] * r[i];
            }
        }
        nrz = block_sum(nrz, red[0]);
        rr = block_sum(rr, red[1]);
        const double beta = rz != 0.0 ? nrz / rz : 0.0;
        rz = nrz;
        ++it;
        done = rr <= tol2 * rr0;
#pragma unroll
        for (int i = 0; i < kSmallPerThread; ++i) {
            const int u = t + i * kSmallThreads;
            if (live[i]) p[u] = z[i] + beta * p[u];
        }
        __syncthreads();
    }
    double h = 0.0;
#pragma unroll
    for (int i = 0; i < kSmallPerThread; ++i) {
        const int u = t + i * kSmallThreads;
        if (u < n) x_out[u] = x[i];
        if (live[i]) h += dd[i] * x[i];
    }
    h = block_sum(h, red[2]);
    if (t == 0) {
        sc->rz[0] = rz;
        sc->rr = rr;
        sc->rr0 = rr0;
        sc->rwc_v = h / vol;
        sc->done = done ? 1 : 0;
        sc->iters = it;
        header->iters = it;
        if (!done) atomicOr(&header->status, static_cast<uint32_t>(kErrNotConverged));
    }
}

__global__ void rwc_of_pivot(const double* __restrict__ part, int nparts, Scalars* sc, double vol) {
    __shared__ double lds[kBlock / kWave];
    double a = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) a += part[i];
    a = block_sum(a, lds);
    if (threadIdx.x == 0) sc->rwc_v = a / vol;
}

__global__ void pivot_partials(int32_t n, const double* __restrict__ d, const double* __restrict__ h,
                               double* __restrict__ part) {
    __shared__ double lds[kBlock / kWave];
    double s = 0.0;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x)
        s += d[u] * h[u];
    s = block_sum(s, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Thread per internal index u; the caller's arrays (counts in, RWC, standard errors and
// hitting times out) are indexed by input id node_id[u].
__global__ void assemble(int32_t n, int32_t v, double vol, double l, const int32_t* __restrict__ node_id,
                         const uint64_t* __restrict__ counts, const uint64_t* __restrict__ counts_sq,
                         const double* __restrict__ d, const double* __restrict__ h, const Scalars* __restrict__ sc,
                         double* __restrict__ rwc, double* __restrict__ se, double* __restrict__ hit) {
    const double rv = sc->rwc_v;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t id = node_id[u];
        const double t = static_cast<double>(counts[id]) / l;
        if (u == v) {
            rwc[id] = rv;
        } else {
            const double a = (vol * t) / d[u];
            const double b = 2.0 * h[u];
            rwc[id] = (a - b) + rv;
        }
        if (hit) hit[id] = h[u];
        if (se) {
            double s = 0.0;
            if (u != v && l > 1.0) {
                const double c1 = static_cast<double>(counts[id]);
                const double c2 = static_cast<double>(counts_sq[id]);
                double var = (c2 - (c1 * c1) / l) / (l - 1.0);
                var = var > 0.0 ? var : 0.0;
                s = (vol / d[u]) * sqrt(var / l);
            }
            se[id] = s;
        }
    }
}

// Eq. (3) from a given estimate of diag(calL_v^{-1}) (FastChol's tau~), by input id.
__global__ void assemble_diag(int32_t n, int32_t v, double vol, const int32_t* __restrict__ node_id,
                              const double* __restrict__ diag, const double* __restrict__ d,
                              const double* __restrict__ h, const Scalars* __restrict__ sc, double* __restrict__ rwc,
                              double* __restrict__ hit) {
    const double rv = sc->rwc_v;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t id = node_id[u];
        if (u == v) {
            rwc[id] = rv;
        } else {
            const double a = (vol * diag[id]) / d[u];
            const double b = 2.0 * h[u];
            rwc[id] = (a - b) + rv;
        }
        if (hit) hit[id] = h[u];
    }
}

// Group RWC of a root set S (hitting time to the set, H_S = sum_u pi_u h_u with h solving the
// system grounded at S) and, for every node u, the estimate of H_{S + u} from the S-rooted
// forests: removing u from the grounded system is a rank-one update, so with M = L_S,
//   h' = h - (h_u / (M^-1)_uu) M^-1 e_u   and   H_{S + u} = H_S - h_u^2 / (vol (M^-1)_uu),
// and the forests' visit totals estimate d_u (M^-1)_uu by t~_u = C_u / l (as in Lemma 5.2 for
// one root), so H_{S + u} ~ H_S - d_u h_u^2 / (vol t~_u).  Nodes of S keep H_S.
__global__ void assemble_group(int32_t n, const uint32_t* __restrict__ gmask, double vol, double l,
                               const int32_t* __restrict__ node_id, const uint64_t* __restrict__ counts,
                               const double* __restrict__ d, const double* __restrict__ h,
                               const Scalars* __restrict__ sc, double* __restrict__ marginal, double* __restrict__ hit,
                               double* __restrict__ group) {
    const double hs = sc->rwc_v;
    for (int64_t u = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; u < n;
         u += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t id = node_id[u];   // caller's arrays by input id
        if (u == 0) *group = hs;
        if (hit) hit[id] = h[u];
        if (grounded(gmask, -1, u)) {
            marginal[id] = hs;
        } else {
            const double t = static_cast<double>(counts[id]) / l;
            const double q = (d[u] * (h[u] * h[u])) / (vol * t);
            marginal[id] = hs - q;
        }
    }
}

// Root set of the group estimate as a bitmap; ids out of range or repeated are reported.
__global__ void clear_words(uint32_t* __restrict__ w, int64_t count) {
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < count;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        w[i] = 0u;
}

__global__ void mark_roots(const int32_t* __restrict__ roots, int32_t nroots, int32_t n,
                           const int32_t* __restrict__ node_index, uint32_t* __restrict__ gmask, WsHeader* header) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nroots) return;
    const int32_t id = roots[i];
    if (id < 0 || id >= n) {
        atomicOr(&header->status, static_cast<uint32_t>(kErrNodeRange));
        return;
    }
    const int32_t r = node_index[id];
    const uint32_t bit = 1u << (r & 31);
    if (atomicOr(&gmask[r >> 5], bit) & bit) atomicOr(&header->status, static_cast<uint32_t>(kErrDupRoot));
}

__global__ void header_start(WsHeader* header) { header_begin(header); }

// After the launched iterations: the iteration count, and an error bit if the residual never
// met the tolerance.
__global__ void solve_finish(const Scalars* __restrict__ sc, WsHeader* header) {
    header->iters = sc->iters;
    if (!sc->done) atomicOr(&header->status, static_cast<uint32_t>(kErrNotConverged));
}

// The two-launch form's pairs (16 bytes a node) stay in each XCD's 4 MB of L2 up to here.
constexpr int32_t kPairNodes = 200000;

struct EstLayout {
    WsHeader* header;
    double *x, *r, *z, *p, *ap, *part;
    double2* zp[2];   // (z, p) pairs, in turn (up to kPairNodes nodes)
    double* part_ap;  // partials of p^T A p
    Scalars* sc;
    uint32_t* gmask;
    int64_t mask_words;
    uint32_t* cover;   // [n] components holding a root (graphs of several components)
    size_t total;
};

EstLayout carve_est(void* ws, int32_t n, bool group) {
    Carver c(ws);
    EstLayout L{};
    L.header = c.take<WsHeader>(kHeaderBytes / sizeof(WsHeader));
    L.x = c.take<double>(n);
    L.r = c.take<double>(n);
    const bool pair = n <= kPairNodes;
    L.z = pair ? nullptr : c.take<double>(n);
    L.p = pair ? nullptr : c.take<double>(n);
    L.zp[0] = pair ? c.take<double2>(n) : nullptr;
    L.zp[1] = pair ? c.take<double2>(n) : nullptr;
    L.ap = c.take<double>(n);
    L.part = c.take<double>(kMaxBlocks);   // at least 2 kIterBlocks
    L.part_ap = c.take<double>(kIterBlocks);
    L.sc = c.take<Scalars>(1);
    L.mask_words = group ? (static_cast<int64_t>(n) + 31) / 32 : 0;
    L.gmask = group ? c.take<uint32_t>(L.mask_words) : nullptr;
    L.cover = group ? c.take<uint32_t>(n) : nullptr;
    L.total = c.used();
    return L;
}

// Iterations launched per call in stream-ordered mode (check_every < 0): the whole solve is
// enqueued at once, so it is bounded to keep a captured graph small.
constexpr int kMaxAsyncIter = 4096;

int check_solve_params(const rwc_solve_params* sp) {
    if (sp && sp->check_every < 0 && (sp->max_iter < 1 || sp->max_iter > kMaxAsyncIter))
        return fail(RWC_ERR_INVALID_ARG, "stream-ordered solves need max_iter in [1, %d]", kMaxAsyncIter);
    if (sp && (sp->max_iter < 0 || !(sp->tol >= 0.0)))
        return fail(RWC_ERR_INVALID_ARG, "max_iter and tol must not be negative");
    return RWC_OK;
}

// Jacobi-PCG on the system grounded at v (or at the set in L.gmask): x solves L_G x = d_{-G}, and
// RWC of the pivot (of the set).  Host-checked mode reads the scalars after `check` iterations
// and then after twice as many each time (at most kMaxCheck; always `check` if the caller chose
// it); stream-ordered mode (check < 0) launches max_iter iterations, which stop on the device at
// convergence, and leaves the outcome in the workspace header.  The iterations run do not
// depend on the mode.
constexpr int kMaxCheck = 128;

int pivot_solve(const rwc_csr* g, int32_t v, const EstLayout& L, const rwc_solve_params* sp, int32_t* iters,
                hipStream_t s, bool* async_out) {
    const int32_t n = g->n;
    const double tol = (sp && sp->tol > 0) ? sp->tol : 1e-12;
    const bool async = sp && sp->check_every < 0;
    const int max_iter = (sp && sp->max_iter > 0) ? sp->max_iter : (async ? 0 : 20000);
    const bool chosen = sp && sp->check_every > 0;
    const double tol2 = tol * tol;
    *async_out = async;
    Scalars host{};
    auto read = [&]() -> int {
        RWC_HIP(hipGetLastError());
        RWC_HIP(hipMemcpyAsync(&host, L.sc, sizeof(host), hipMemcpyDeviceToHost, s));
        RWC_HIP(hipStreamSynchronize(s));
        return RWC_OK;
    };
    auto outcome = [&]() -> int {
        if (iters) *iters = host.iters;
        if (!host.done)
            return fail(RWC_ERR_NOT_CONVERGED, "pivot solve: relative residual %.3e after %d iterations",
                        host.rr > 0 ? std::sqrt(host.rr / host.rr0) : 0.0, host.iters);
        return RWC_OK;
    };
    if (solves_small(*g)) {
        const bool weighted = g->weighted != 0;
        const size_t lds = SmallLayout(n, g->nnz, weighted).total;
        hipLaunchKernelGGL(pcg_small, dim3(1), dim3(kSmallThreads), lds, s, n, static_cast<int32_t>(g->nnz), weighted, v,
                           L.gmask, g->row_ptr, g->col, g->weight, g->strength, g->vol, tol2, max_iter, L.x, L.sc,
                           L.header);
        RWC_HIP(hipGetLastError());
        if (async) {
            if (iters) *iters = -1;
            return RWC_OK;
        }
        RWC_CHECK(read());
        return outcome();
    }
    const bool pair = n <= kPairNodes;
    const bool few = g->nnz <= 6 * static_cast<int64_t>(n);   // short rows on average: four lanes each
    const unsigned nb = std::min<unsigned>(blocks_for(n, kIterBlock), kIterBlocks);
    const bool dense = g->nnz > 160 * static_cast<int64_t>(n);   // a wave each (ER(10 000, 300): solve 0.68 -> 0.37 ms)
    // a group of lanes per row, and on dense graphs, whose long rows are taken one after the other by whole
    // blocks, a block for every four of its threads' loads (complete graph of 2000 nodes, 32 -> 512 blocks:
    // 1.10 -> 0.26 ms)
    const int64_t by_rows = blocks_for(static_cast<int64_t>(n) * (few ? 4 : dense ? 64 : 16), kIterBlock);
    const unsigned nbs = static_cast<unsigned>(
        std::min<int64_t>(std::max<int64_t>(by_rows, blocks_for(g->nnz, 4 * kIterBlock)), kIterBlocks));
    const int np = static_cast<int>(nb), nps = static_cast<int>(nbs);
    auto product = pair ? (few ? spmv_dot<true, 4> : dense ? spmv_dot<true, 64> : spmv_dot<true, 16>)
                        : (few ? spmv_dot<false, 4> : dense ? spmv_dot<false, 64> : spmv_dot<false, 16>);
    auto update = pair ? update_xr<true> : update_xr<false>;
    hipLaunchKernelGGL(pcg_init, dim3(nb), dim3(kIterBlock), 0, s, n, v, L.gmask, g->strength, L.x, L.r, L.z, L.p,
                       L.zp[0], L.part, L.sc);
    auto direction = [&](int it, int32_t nodes) {
        hipLaunchKernelGGL(update_p, dim3(nodes > 0 ? nb : 1), dim3(kIterBlock), 0, s, it, nodes, v, L.gmask, L.sc, tol2,
                           L.part, np, L.z, L.p);
    };
    auto iteration = [&](int it) {
        double2 *const in = L.zp[it & 1], *const out = L.zp[(it + 1) & 1];
        if (!pair) direction(it, n);
        hipLaunchKernelGGL(product, dim3(nbs), dim3(kIterBlock), 0, s, it, n, v, g->max_degree, L.gmask, L.sc, tol2, g->row_ptr, g->col,
                           g->weight, g->strength, L.part, np, L.p, in, out, L.ap, L.part_ap);
        hipLaunchKernelGGL(update, dim3(nb), dim3(kIterBlock), 0, s, it, n, v, L.gmask, L.sc, L.part_ap, nps, g->strength,
                           L.x, L.r, L.z, L.p, out, L.ap, L.part);
    };
    int launched = 0;
    for (int chunk = async ? max_iter : chosen ? sp->check_every : 16; launched < max_iter;
         chunk = chosen || 2 * chunk > kMaxCheck ? chunk : 2 * chunk) {
        const int stop = std::min(launched + chunk, max_iter);
        for (; launched < stop; ++launched) iteration(launched);
        direction(launched, 0);   // the last iteration's convergence
        if (async) break;
        RWC_CHECK(read());
        if (host.done) break;
    }
    hipLaunchKernelGGL(solve_finish, dim3(1), dim3(1), 0, s, L.sc, L.header);
    const unsigned np2 = blocks_for(n, kBlock) < kMaxBlocks ? blocks_for(n, kBlock) : kMaxBlocks;
    hipLaunchKernelGGL(pivot_partials, dim3(np2), dim3(kBlock), 0, s, n, g->strength, L.x, L.part);
    hipLaunchKernelGGL(rwc_of_pivot, dim3(1), dim3(kBlock), 0, s, L.part, static_cast<int>(np2), L.sc, g->vol);
    RWC_HIP(hipGetLastError());
    if (async) {
        if (iters) *iters = -1;
        return RWC_OK;
    }
    return outcome();
}

}  // namespace
}  // namespace rwc

using namespace rwc;

extern "C" int rwc_estimate_workspace(const rwc_csr* g, size_t* bytes) {
    clear_error();
    if (!g || !bytes) return fail(RWC_ERR_INVALID_ARG, "g and bytes must not be null");
    *bytes = carve_est(nullptr, g->n, false).total;
    return RWC_OK;
}

extern "C" int rwc_estimate(const rwc_csr* g, const uint64_t* counts, const uint64_t* counts_sq, int64_t l,
                            const rwc_solve_params* sp, double* rwc, double* hit, double* stderr_out, int32_t* iters,
                            void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (!g || !counts || !rwc) return fail(RWC_ERR_INVALID_ARG, "g, counts and rwc must not be null");
    RWC_CHECK(require_connected(g, "rwc_estimate (the pivot solve)"));
    if (l < 1) return fail(RWC_ERR_INVALID_ARG, "l must be positive");
    if (stderr_out && !counts_sq) return fail(RWC_ERR_INVALID_ARG, "stderr needs counts_sq");
    RWC_CHECK(check_solve_params(sp));
    const int32_t n = g->n;
    RWC_CHECK(check_workspace(ws, ws_bytes, carve_est(nullptr, n, false).total));
    EstLayout L = carve_est(ws, n, false);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int v = g->pivot_index;
    const unsigned nb = blocks_for(n, kBlock) < kMaxBlocks ? blocks_for(n, kBlock) : kMaxBlocks;
    hipLaunchKernelGGL(header_start, dim3(1), dim3(1), 0, s, L.header);
    bool async = false;
    RWC_CHECK(pivot_solve(g, v, L, sp, iters, s, &async));
    hipLaunchKernelGGL(assemble, dim3(nb), dim3(kBlock), 0, s, n, v, g->vol, static_cast<double>(l), g->node_id, counts,
                       counts_sq, g->strength, L.x, L.sc, rwc, stderr_out, hit);
    RWC_HIP(hipGetLastError());
    if (!async) RWC_HIP(hipStreamSynchronize(s));
    return RWC_OK;
}

extern "C" int rwc_estimate_diag(const rwc_csr* g, const double* diag, const rwc_solve_params* sp, double* rwc,
                                 double* hit, int32_t* iters, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (!g || !diag || !rwc) return fail(RWC_ERR_INVALID_ARG, "g, diag and rwc must not be null");
    RWC_CHECK(require_connected(g, "rwc_estimate_diag (the pivot solve)"));
    RWC_CHECK(check_solve_params(sp));
    const int32_t n = g->n;
    RWC_CHECK(check_workspace(ws, ws_bytes, carve_est(nullptr, n, false).total));
    EstLayout L = carve_est(ws, n, false);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int v = g->pivot_index;
    const unsigned nb = blocks_for(n, kBlock) < kMaxBlocks ? blocks_for(n, kBlock) : kMaxBlocks;
    hipLaunchKernelGGL(header_start, dim3(1), dim3(1), 0, s, L.header);
    bool async = false;
    RWC_CHECK(pivot_solve(g, v, L, sp, iters, s, &async));
    hipLaunchKernelGGL(assemble_diag, dim3(nb), dim3(kBlock), 0, s, n, v, g->vol, g->node_id, diag, g->strength, L.x,
                       L.sc, rwc, hit);
    RWC_HIP(hipGetLastError());
    if (!async) RWC_HIP(hipStreamSynchronize(s));
    return RWC_OK;
}

extern "C" int rwc_estimate_group_workspace(const rwc_csr* g, size_t* bytes) {
    clear_error();
    if (!g || !bytes) return fail(RWC_ERR_INVALID_ARG, "g and bytes must not be null");
    *bytes = carve_est(nullptr, g->n, true).total;
    return RWC_OK;
}

extern "C" int rwc_estimate_group(const rwc_csr* g, const int32_t* roots, int32_t num_roots, const uint64_t* counts,
                                  int64_t l, const rwc_solve_params* sp, double* group_rwc, double* marginal,
                                  double* hit, int32_t* iters, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (!g || !roots || !counts || !group_rwc || !marginal)
        return fail(RWC_ERR_INVALID_ARG, "g, roots, counts, group_rwc and marginal must not be null");
    if (l < 1) return fail(RWC_ERR_INVALID_ARG, "l must be positive");
    const int32_t n = g->n;
    if (num_roots < 1 || num_roots >= n) return fail(RWC_ERR_INVALID_ARG, "num_roots must be in [1, n - 1]");
    RWC_CHECK(check_solve_params(sp));
    RWC_CHECK(check_workspace(ws, ws_bytes, carve_est(nullptr, n, true).total));
    EstLayout L = carve_est(ws, n, true);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const unsigned nb = blocks_for(n, kBlock) < kMaxBlocks ? blocks_for(n, kBlock) : kMaxBlocks;
    hipLaunchKernelGGL(header_start, dim3(1), dim3(1), 0, s, L.header);
    hipLaunchKernelGGL(clear_words, dim3(blocks_for(L.mask_words, kBlock)), dim3(kBlock), 0, s, L.gmask, L.mask_words);
    hipLaunchKernelGGL(mark_roots, dim3(blocks_for(num_roots, kBlock)), dim3(kBlock), 0, s, roots, num_roots, n,
                       g->node_index, L.gmask, L.header);
    if (g->components > 1) check_root_cover(*g, roots, num_roots, L.cover, L.gmask, L.header, s);
    if (!(sp && sp->check_every < 0)) {
        // host-checked mode: a bad root set would leave the system singular, so stop here
        WsHeader h{};
        RWC_HIP(hipMemcpyAsync(&h, L.header, sizeof(h), hipMemcpyDeviceToHost, s));
        RWC_HIP(hipStreamSynchronize(s));
        RWC_CHECK(device_error_to_status(h.status));
    }
    bool async = false;
    RWC_CHECK(pivot_solve(g, -1, L, sp, iters, s, &async));
    hipLaunchKernelGGL(assemble_group, dim3(nb), dim3(kBlock), 0, s, n, L.gmask, g->vol, static_cast<double>(l),
                       g->node_id, counts, g->strength, L.x, L.sc, marginal, hit, group_rwc);
    RWC_HIP(hipGetLastError());
    if (!async) {
        // the root set is validated on the device: report it with the synchronous result
        WsHeader h{};
        RWC_HIP(hipMemcpyAsync(&h, L.header, sizeof(h), hipMemcpyDeviceToHost, s));
        RWC_HIP(hipStreamSynchronize(s));
        return device_error_to_status(h.status);
    }
    return RWC_OK;
}

// ---------------------------------------------------------------------------------------
// rwc_estimate_static: rwc_estimate over a fixed device array instead of a caller workspace,
// for callers that cannot allocate.  `scratch` is a host-side stand-in for the array in host
// code; its device address (one per GPU) comes from hipGetSymbolAddress on the first call on
// each device and is the only handle passed to kernels.
// ---------------------------------------------------------------------------------------
namespace rwc {
namespace {
constexpr size_t kStaticScratchBytes = size_t{128} << 20;   // 128 MiB: graphs up to ~3.35 M nodes
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

int static_scratch(void** out) {
    static std::mutex mu;
    static void* ptrs[64] = {};
    int dev = 0;
    RWC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(RWC_ERR_HIP, "device %d out of the supported range", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void* p = nullptr;
        RWC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(RWC_ERR_HIP, "hipGetSymbolAddress returned a null address");
        ptrs[dev] = p;
    }
    *out = ptrs[dev];
    return RWC_OK;
}
}  // namespace
}  // namespace rwc

extern "C" int rwc_estimate_static(const rwc_csr* g, const uint64_t* counts, const uint64_t* counts_sq, int64_t l,
                                   const rwc_solve_params* sp, double* rwc_out, double* hit, double* stderr_out,
                                   int32_t* iters, void* stream) {
    clear_error();
    if (!g) return fail(RWC_ERR_INVALID_ARG, "g must not be null");
    RWC_CHECK(require_connected(g, "rwc_estimate_static (the pivot solve)"));
    if (sp && sp->check_every < 0)
        return fail(RWC_ERR_INVALID_ARG, "rwc_estimate_static runs the host-checked solve only");
    const size_t need = carve_est(nullptr, g->n, false).total;
    if (need > kStaticScratchBytes)
        return fail(RWC_ERR_TOO_LARGE, "rwc_estimate_static: n = %d needs %zu bytes of scratch, the fixed array has %zu",
                    g->n, need, kStaticScratchBytes);
    void* ws = nullptr;
    RWC_CHECK(static_scratch(&ws));
    return rwc_estimate(g, counts, counts_sq, l, sp, rwc_out, hit, stderr_out, iters, ws, kStaticScratchBytes, stream);
}
