// rwc_fastchol: FastChol (Section 4, Algorithm 2) on the GPU.
//
// 1. IChol(calL_v, delta) (Lemma 4.1): incomplete Cholesky of the grounded normalised Laplacian
//    with threshold dropping, left-looking, columns in ascending input id (the pivot v removed).
//    Column j starts as A(j:N, j) = (1, -w_xy / sqrt(d_x d_y) for the later neighbours) and
//    loses R(j, k) R(j:N, k) for every earlier column k with R(j, k) != 0, in ascending k; the
//    pivot is the square root of what is left on the diagonal, and an off-diagonal entry
//    x = w_i / pivot is kept when x != 0 and |x| >= delta * ||A(j:N, j)||_1 (the threshold
//    variant of MATLAB's ichol, which the paper's experiments use).
// 2. The windowed, sparsified inverse (Lemma 4.3 and Algorithm 2's loop), right to left:
//      S*(:, u) = e_u / R_uu - sum_{i in (u, u + w_u], R_iu != 0} (R_iu / R_uu) S~(:, i),
//    w_u = min(floor(w_s (1 + d_u / d_max)), N); a column of more than zeta nonzeros keeps the
//    shortest prefix, by decreasing magnitude (ties by row), whose dropped tail has 1-norm at
//    most eps_p ||S*(:, u)||_1; tau~_u = ||S~(:, u)||^2.
//
// Both recursions are chains: column j needs every earlier column its row reaches (IChol) and
// column u the later columns of its window with a factor entry (the inverse).  IChol has two
// forms with the same result:
//   - dense (the default while the matrix's packed lower triangle fits): right-looking on that
//     triangle in HBM, in panels of 32 columns, one launch per panel;
//   - chain: left-looking on one wave, sparse throughout, for any size.
// The inverse's columns form a dependency DAG, which sixteen waves of one workgroup run, each
// column on one wave with its lanes over the column's entries.
// Every floating-point operation happens in the order the serial algorithm performs it (each
// entry's updates in ascending k, norms and tails summed one entry at a time, sorts by total
// orders), so the factor, S~ and tau~ are the serial ones bit for bit.
#include <algorithm>
#include <utility>

#include "common.hpp"
#include "device.hpp"

namespace rwc {
namespace {

constexpr int kSortCap = 4096;   // entries one column may hold while it is ordered in LDS

struct FcArgs {
    // the graph, in its internal order
    const int32_t* row_ptr;
    const int32_t* col;
    const float* weight;
    const double* strength;
    const int32_t* node_id;
    const int32_t* node_index;
    int32_t n;
    int32_t v;        // pivot, input id
    int32_t N;        // n - 1 columns
    int32_t zeta;
    double droptol, ws, eps_p;
    // factor R: column j is [r_ptr[j], r_ptr[j + 1]), diagonal first, rows ascending
    int64_t* r_ptr;
    int32_t* r_row;
    double* r_val;
    int64_t* r_colend;  // end of that column (r_ptr[column + 1]), so a row-list link needs no more
    int64_t* r_next;    // next entry of the same row (row lists in ascending column), -1 at the end
    int64_t* head;      // first and last entry of each row
    int64_t* tail;
    int64_t r_cap;
    // inverse S~: column u is s_len[u] entries from s_start[u], rows ascending
    int64_t* s_start;
    int32_t* s_len;
    int32_t* s_row;
    double* s_val;
    int64_t s_cap;
    // dense accumulators with stamps (entry i is live in column c when stamp[i] == c + 1)
    double* acc;
    int32_t* stamp;
    int32_t* touched;   // [N] the rows a column has reached, in the order reached (the inverse:
                        // acc, stamp and touched hold one slice of N per wave)
    int32_t* done;      // [N] the inverse: column published
    double* inv_val;    // the inverse: per wave, kSortCap entries to order a large column in
    int32_t* inv_row;
    double* dmax;
    double* dense;      // dense IChol: the lower triangle of S, packed by columns (column j holds
                        // rows j .. N - 1 from packed_column(j, N))
    double* colnorm;    // dense IChol: ||A(j:N, j)||_1 per column
    // dense IChol, two panels by parity: rows' entries R(i, J .. J + kPanel - 1) (dropped ones 0) ...
    double* prow;        // [2][N][kPanel]
    uint32_t* pmask;     // [2][N] which were kept
    double* pnext;       // [2][kPanel][kPanel] those of the next panel's rows, by column
    int32_t* act;        // [2][parts * kPanelRows] the rows below the panel with a kept entry, part by part
    uint32_t* act_cnt;   // [2][parts]
    uint32_t* act_skip;  // [2] how many of them are the next panel's
    uint32_t* col_cnt;   // [2][parts][kPanel] kept entries per column
    int32_t parts;
    double* tau;        // [n] output by input id
    WsHeader* header;
    int64_t* counters;  // [2]: entries of R and of S~
};

// Words one lane writes and another reads later (the dense accumulator, its stamps and the row
// lists): relaxed atomics.  They are used only on memory that one wave alone touches (the chain's
// kernel is a single wave; each wave of the inverse has its own slices), so their scope is the
// wavefront, and so is the scope of wave_order(): a wave's vector memory operations are
// performed in the order it issues them, so ordering them needs no wait for the memory system,
// only that the compiler keep them in program order.
template <class T>
__device__ __forceinline__ T ld(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <class T>
__device__ __forceinline__ void st(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

__device__ __forceinline__ int32_t node_of_column(int32_t j, int32_t v) { return j + (j >= v ? 1 : 0); }
__device__ __forceinline__ int32_t column_of_node(int32_t u, int32_t v) { return u - (u > v ? 1 : 0); }

// Lane l's value of x (l the same in every lane), exactly.
__device__ __forceinline__ double lane_value(double x, int l) {
    const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(x));
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(b & 0xffffffffull), l));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(b >> 32), l));
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

// Lanes whose flag is set, in lane order: this lane's rank among them and their number.
__device__ __forceinline__ uint32_t rank_of(bool flag, uint32_t& count) {
    const uint64_t m = __ballot(flag);
    const int lane = threadIdx.x & (kWave - 1);
    count = static_cast<uint32_t>(__popcll(m));
    return static_cast<uint32_t>(__popcll(m & ((lane == 0) ? 0ull : (~0ull >> (kWave - lane)))));
}

// Bitonic sort of len (<= kSortCap) entries, in LDS or in the wave's own global scratch, by one
// wave; less(a, b) a total order.
template <class Less>
__device__ void wave_sort(double* val, int32_t* row, int32_t len, Less less) {
    const int lane = threadIdx.x & (kWave - 1);
    int32_t size = 1;
    while (size < len) size <<= 1;
    for (int32_t i = len + lane; i < size; i += kWave) {   // padding sorts last
        val[i] = 0.0;
        row[i] = 0x7FFFFFFF;
    }
    wave_order();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the wave's LDS writes are done
    __builtin_amdgcn_wave_barrier();
    for (int32_t k = 2; k <= size; k <<= 1) {
        for (int32_t jj = k >> 1; jj > 0; jj >>= 1) {
            for (int32_t i = lane; i < size; i += kWave) {
                const int32_t p = i ^ jj;
                if (p > i) {
                    const bool up = (i & k) == 0;
                    const bool pad_i = row[i] == 0x7FFFFFFF, pad_p = row[p] == 0x7FFFFFFF;
                    // padding is larger than any entry
                    const bool p_before_i = pad_i ? !pad_p : (!pad_p && less(val[p], row[p], val[i], row[i]));
                    if (p_before_i == up) {
                        const double tv = val[i];
                        val[i] = val[p];
                        val[p] = tv;
                        const int32_t tr = row[i];
                        row[i] = row[p];
                        row[p] = tr;
                    }
                }
            }
            wave_order();   // the buffers may be in global memory: keep the stages in order
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
        }
    }
}

__global__ void fill_i32(int32_t* p, int64_t count, int32_t value) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = value;
}

__global__ void __launch_bounds__(kWave) fc_begin(FcArgs A) {
    const int lane = threadIdx.x;
    if (lane == 0) {
        header_begin(A.header);
        A.counters[0] = 0;
        A.counters[1] = 0;
        A.r_ptr[0] = 0;
    }
    double m = 0.0;
    for (int32_t x = lane; x < A.n; x += kWave)
        if (A.node_id[x] != A.v) m = A.strength[x] > m ? A.strength[x] : m;
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double o = __shfl_xor(m, off, kWave);
        m = o > m ? o : m;
    }
    if (lane == 0) *A.dmax = m;
    if (A.head) {   // the chain's row lists (absent for the dense factor)
        for (int64_t i = lane; i < A.N; i += kWave) {
            st(&A.head[i], int64_t{-1});
            st(&A.tail[i], int64_t{-1});
        }
    }
    for (int64_t u = lane; u < A.n; u += kWave) A.tau[u] = 0.0;
}

// One link of a row list in IChol's left-looking update: entry e = R(j, k), the next entry of
// row j, the end of column k, and kSpan entries of column k's suffix from some position p0 (lane
// l holds positions p0 + b kWave + l, clamped to written positions for the load).
constexpr int kBatch = 4;
constexpr int kSpan = kBatch * kWave;
struct Link {
    int64_t e, next, end;
    double rjk;
    int32_t row[kBatch];
    double val[kBatch];
};

__device__ __forceinline__ void load_span(const FcArgs& A, int64_t p0, int64_t rp, Link& L) {
    const int lane = threadIdx.x;
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
        const int64_t p = p0 + b * kWave + lane;
        const int64_t pc = p < rp ? p : rp - 1;
        L.row[b] = A.r_row[pc];
        L.val[b] = A.r_val[pc];
    }
}

// Starts the loads of the link at e; e outside [0, rp) ends the list (L.e = -1).
__device__ __forceinline__ Link open_link(const FcArgs& A, int64_t e, int64_t rp) {
    Link L;
    if (e < 0 || e >= rp) {
        L.e = -1;
        return L;
    }
    L.e = e;
    L.next = ld(&A.r_next[e]);
    L.rjk = A.r_val[e];
    L.end = A.r_colend[e];
    load_span(A, e, rp, L);
    return L;
}

// acc[i] -= R(i, k) R(j, k) for the loaded span's rows i < L.end; rows reached for the first time
// in this column start from 0 and join the touched list.  The rows of one column are distinct,
// so the span's loads of stamps and accumulators all precede its stores.
__device__ __forceinline__ void update(const FcArgs& A, int64_t p0, const Link& L, int32_t stamp, uint32_t& nt) {
    const int lane = threadIdx.x;
    int32_t i[kBatch], sg[kBatch];
    double cur[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
        i[b] = p0 + b * kWave + lane < L.end ? L.row[b] : -1;
        const int32_t ic = i[b] >= 0 ? i[b] : L.row[0];   // a valid address for every lane
        sg[b] = ld(&A.stamp[ic]);
        cur[b] = ld(&A.acc[ic]);
    }
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
        const bool fresh = i[b] >= 0 && sg[b] != stamp;
        uint32_t cnt = 0;
        const uint32_t r = rank_of(fresh, cnt);
        if (fresh) {
            st(&A.stamp[i[b]], stamp);
            st(&A.touched[nt + r], i[b]);   // distinct rows below N: nt never passes N
            cur[b] = 0.0;
        }
        nt += cnt;
        if (i[b] >= 0) st(&A.acc[i[b]], cur[b] - L.val[b] * L.rjk);
    }
    wave_order();
}

// IChol, one wave.
__global__ void __launch_bounds__(kWave) fc_ichol(FcArgs A) {
    __shared__ int32_t krow[kSortCap];   // the entries a column keeps, ordered by row here
    __shared__ double kval[kSortCap];
    int32_t* touched = A.touched;
    const int lane = threadIdx.x;
    const int32_t N = A.N, v = A.v;
    int64_t rp = 0;   // r_ptr[j], uniform
    for (int32_t j = 0; j < N; ++j) {
        const int32_t stamp = j + 1;
        const int32_t u = node_of_column(j, v);
        const int32_t x = A.node_index[u];
        const double du = A.strength[x];
        const int32_t beg = A.row_ptr[x], end = A.row_ptr[x + 1];
        // column j of A: the diagonal, then the later neighbours by ascending input id
        uint32_t nt = 0;
        if (lane == 0) {
            st(&A.acc[j], 1.0);
            st(&A.stamp[j], stamp);
            st(&touched[0], j);
        }
        nt = 1;
        double colnorm = 1.0;
        bool full = false;
        for (int32_t b0 = beg; b0 < end; b0 += kWave) {
            const int32_t k = b0 + lane;
            int32_t i = -1;
            double a = 0.0;
            if (k < end) {
                const int32_t y = A.col[k];
                const int32_t yid = A.node_id[y];
                if (yid > u && yid != v) {
                    i = column_of_node(yid, v);
                    a = -static_cast<double>(A.weight[k]) / sqrt(du * A.strength[y]);
                }
            }
            uint32_t cnt = 0;
            const uint32_t r = rank_of(i >= 0, cnt);
            if (i >= 0) {
                st(&A.acc[i], a);
                st(&A.stamp[i], stamp);
                st(&touched[nt + r], i);
            }
            nt += cnt;
            // the column's 1-norm, one entry at a time in row order
            for (int l = 0; l < kWave; ++l) {
                const double al = __shfl(a, l, kWave);
                const int32_t il = __shfl(i, l, kWave);
                if (il >= 0) colnorm += fabs(al);
            }
        }
        if (full) {
            if (lane == 0) atomicOr(&A.header->status, static_cast<uint32_t>(kErrCapacity));
            return;
        }
        wave_order();
        // left-looking update: every earlier column k with R(j, k) != 0, ascending k (a row has
        // at most j entries left of the diagonal: the guard stops a corrupt list).  Pipelined by
        // one link: the next link's entry, its column end and the first kSpan entries of its
        // column suffix are loaded before this link's accumulator update, so a link costs about
        // one memory round trip (the accumulator's) instead of four.
        int64_t links = 0;
        Link cur = open_link(A, ld(&A.head[j]), rp);
        while (cur.e >= 0) {
            if (++links > j) {
                full = true;
                break;
            }
            const Link nxt = open_link(A, cur.next, rp);
            // a suffix longer than kSpan: each further span is loaded before the previous one
            // is applied
            for (int64_t p0 = cur.e;; p0 += kSpan) {
                const bool more = p0 + kSpan < cur.end;
                Link span = cur;
                if (more) load_span(A, p0 + kSpan, rp, span);
                update(A, p0, cur, stamp, nt);
                if (!more) break;
                cur = span;
            }
            cur = nxt;
        }
        if (full) {
            if (lane == 0) atomicOr(&A.header->status, static_cast<uint32_t>(kErrCapacity));
            return;
        }
        wave_order();
        const double wjj = ld(&A.acc[j]);
        if (!(wjj > 0.0)) {
            if (lane == 0) atomicOr(&A.header->status, static_cast<uint32_t>(kErrPivot));
            return;
        }
        const double piv = sqrt(wjj);
        // the drop rule over the reached rows, the survivors ordered by row in LDS, then
        // appended after the diagonal
        const double thr = A.droptol * colnorm;
        uint32_t kept = 0;
        for (uint32_t t0 = 0; t0 < nt && !full; t0 += kSpan) {
            int32_t i[kBatch];
            double xv[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const uint32_t t = t0 + b * kWave + lane;
                i[b] = t < nt ? ld(&touched[t < nt ? t : 0]) : -1;
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) xv[b] = ld(&A.acc[i[b] >= 0 ? i[b] : j]);
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const double x = xv[b] / piv;
                const bool keep = i[b] >= 0 && i[b] != j && x != 0.0 && fabs(x) >= thr;
                uint32_t cnt = 0;
                const uint32_t r = rank_of(keep, cnt);
                if (kept + cnt > static_cast<uint32_t>(kSortCap)) {
                    full = true;
                    break;
                }
                if (keep) {
                    krow[kept + r] = i[b];
                    kval[kept + r] = x;
                }
                kept += cnt;
            }
        }
        if (full || rp + 1 + static_cast<int64_t>(kept) > A.r_cap) {
            if (lane == 0) atomicOr(&A.header->status, static_cast<uint32_t>(kErrCapacity));
            return;
        }
        wave_sort(kval, krow, static_cast<int32_t>(kept),
                  [](double, int32_t ra, double, int32_t rb) { return ra < rb; });
        const int64_t colend = rp + 1 + static_cast<int64_t>(kept);
        if (lane == 0) {
            A.r_row[rp] = j;
            A.r_val[rp] = piv;
            A.r_colend[rp] = colend;
            st(&A.r_next[rp], int64_t{-1});
        }
        for (uint32_t t = lane; t < kept; t += kWave) {
            const int32_t i = krow[t];
            const int64_t pos = rp + 1 + t;
            A.r_row[pos] = i;
            A.r_val[pos] = kval[t];
            A.r_colend[pos] = colend;
            st(&A.r_next[pos], int64_t{-1});
            // append to row i's list (each lane a different row)
            const int64_t last = ld(&A.tail[i]);
            if (last < 0)
                st(&A.head[i], pos);
            else
                st(&A.r_next[last], pos);
            st(&A.tail[i], pos);
        }
        rp += 1 + kept;
        if (lane == 0) A.r_ptr[j + 1] = rp;
        wave_order();
        __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) A.counters[0] = rp;
}

// ---- IChol, dense right-looking, in panels ----
// S starts as the lower triangle of calL_v, and every entry S(i, j) loses its products R(i, k)
// R(j, k) in ascending k, as in the left-looking chain, so the two forms give the same factor bit
// for bit.  A panel of kPanel columns is formed at once: its diagonal block is factored by one
// wave, column after column, and every row below then takes its kPanel entries by itself (a
// triangular solve with the drop rule), a thread per row.  Launch p forms panel p + 1, applying
// panel p's products to its columns as it reads them, while other workgroups subtract panel p's
// products from the columns to the right and others copy panel p into the compact factor.
//
// What bounds it: a launch's serial part (read and apply 18 us, 32 dependent columns of the diagonal
// block 11, 32 of the rows' solves 11) up to about 10 000 columns, then the updates' reads and writes
// of S.  Against a launch per column, each column's products applied as soon as it was formed (all of
// IChol, ms): BA(5000, 5) 46 -> 8.5, BA(20 000, 5) 219 -> 96, 10 000-node grid 92 -> 25; the whole call
// on BA(60 000, 5) 772 -> 576.
constexpr int kPanel = 32;
constexpr int kPanelRows = 256;                      // rows (threads) of a forming or copying workgroup
constexpr int kPanelBlock = kPanelRows + kWave;      // and a wave for the diagonal block
constexpr int kPanelWaves = kPanelBlock / kWave;
constexpr int kTile = 64;                            // active rows and columns of an update's tile
constexpr int kTilePitch = kPanel + 1;               // the last entry 0; odd: rows in different banks
constexpr int kTileCols = (kTile + kPanelWaves - 1) / kPanelWaves;   // columns of a wave
constexpr int kMaxParts = 4096;                      // kDenseMaxColumns / kPanelRows

// Offset of column j in the packed lower triangle of an N x N matrix (columns of N - j rows).
__host__ __device__ __forceinline__ int64_t packed_column(int64_t j, int64_t N) { return j * N - j * (j - 1) / 2; }

__global__ void fc_dense_clear(uint64_t* p, int64_t count) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = 0;
}

// S = the lower triangle of calL_v (S must be zero), and colnorm[j] = ||A(j:N, j)||_1 summed down
// the column from the diagonal, as the chain sums it.  One wave per column.
__global__ void __launch_bounds__(256) fc_dense_scatter(FcArgs A) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t N = A.N, v = A.v;
    const int32_t waves = static_cast<int32_t>(blockDim.x / kWave);
    for (int32_t j = blockIdx.x * waves + threadIdx.x / kWave; j < N; j += gridDim.x * waves) {
        const int32_t u = node_of_column(j, v);
        const int32_t x = A.node_index[u];
        const double du = A.strength[x];
        const int32_t beg = A.row_ptr[x], end = A.row_ptr[x + 1];
        double* Sj = A.dense + (packed_column(j, N) - j);   // Sj[i], i >= j
        if (lane == 0) {
            Sj[j] = 1.0;
        }
        double colnorm = 1.0;
        for (int32_t b0 = beg; b0 < end; b0 += kWave) {
            const int32_t k = b0 + lane;
            int32_t i = -1;
            double a = 0.0;
            if (k < end) {
                const int32_t y = A.col[k];
                const int32_t yid = A.node_id[y];
                if (yid > u && yid != v) {
                    i = column_of_node(yid, v);
                    a = -static_cast<double>(A.weight[k]) / sqrt(du * A.strength[y]);
                    Sj[i] = a;
                }
            }
            for (int l = 0; l < kWave; ++l) {
                const double al = __shfl(a, l, kWave);
                const int32_t il = __shfl(i, l, kWave);
                if (il >= 0) colnorm += fabs(al);
            }
        }
        if (lane == 0) A.colnorm[j] = colnorm;
    }
}

// A row of kPanel values that every lane needs: lane l holds values l % 16 and 16 + l % 16, and each
// value is broadcast within the rows of 16 lanes by one DPP move (from LDS, a wave's broadcast of
// 16 bytes takes eight cycles of the one port that all waves share: BA(20 000, 5)'s call took 151 ms
// instead of 115, with 166 registers instead of 126).
struct Spread {
    double lo, hi;
    __device__ __forceinline__ void load(const double* row) {
        const int l = threadIdx.x & 15;
        lo = row[l];
        hi = row[16 + l];
    }
    template <int kAt>
    __device__ __forceinline__ double get() const {
        const int64_t x = __builtin_bit_cast(int64_t, kAt < 16 ? lo : hi);
        const int64_t r = __builtin_amdgcn_update_dpp(x, x, 0x150 + (kAt & 15), 0xf, 0xf, true);   // row_newbcast
        return __builtin_bit_cast(double, r);
    }
};

// s[b] = s[b + kDown] - a row[b + kDown] for b < kCount - kDown.  Eight at a time, phase by phase: left
// to the compiler each product waits for the one before (they share its registers).
template <int kDown, int kFirst, int... kAt>
__device__ __forceinline__ void subtract_some(double* s, double a, const Spread& row, std::integer_sequence<int, kAt...>) {
    double x[sizeof...(kAt)] = {row.get<kFirst + kAt + kDown>()...};
    __builtin_amdgcn_sched_barrier(0);
    ((x[kAt] = a * x[kAt]), ...);
    __builtin_amdgcn_sched_barrier(0);
    ((s[kFirst + kAt] = s[kFirst + kAt + kDown] - x[kAt]), ...);
    __builtin_amdgcn_sched_barrier(0);
}
template <int kDown, int kCount, int kFirst = 0>
__device__ __forceinline__ void subtract(double* s, double a, const Spread& row) {
    constexpr int kNow = kCount - kDown - kFirst < 8 ? kCount - kDown - kFirst : 8;
    subtract_some<kDown, kFirst>(s, a, row, std::make_integer_sequence<int, kNow>{});
    if constexpr (kFirst + kNow < kCount - kDown) subtract<kDown, kCount, kFirst + kNow>(s, a, row);
}

// Steps j0 .. j0 + 7 of the diagonal block's factorisation, a row per lane, and of a row's solve.
// s[b] is the row's entry in column j + b: a step takes s[0] and moves the others down by one, so
// that the loop is short code on registers.  D[j][b] = R(J + j + b, J + j), 0 past the block's last
// row; kLeft = kPanel - j0 columns are left at the first step.
constexpr int kSteps = 8;

template <int kLeft>
__device__ __forceinline__ bool factor_steps(double* s, double* D, double thr, int lane, int nb) {
    bool fine = true;
    const int last = nb < kPanel - kLeft + kSteps ? nb : kPanel - kLeft + kSteps;
    for (int j = kPanel - kLeft; j < last; ++j) {
        const double wjj = lane_value(s[0], j);
        fine = fine && wjj > 0.0;
        const double piv = sqrt(wjj);
        double x = s[0] / piv;
        x = lane > j && lane < nb && x != 0.0 && fabs(x) >= lane_value(thr, j) ? x : 0.0;
        if (lane >= j && lane < j + kPanel) D[j * kPanel + lane - j] = lane == j ? piv : x;
        wave_order();
        Spread d;
        d.load(D + j * kPanel);
        subtract<1, kLeft>(s, x, d);
    }
    if constexpr (kLeft > kSteps) fine = factor_steps<kLeft - kSteps>(s, D, thr, lane, nb) && fine;
    return fine;
}

// take(j, x, keep) may replace the entry and the decision.
template <int kLeft, class Take>
__device__ __forceinline__ void solve_steps(double* s, const double* D, const double* thr_of, int nb, Take&& take) {
    const int last = nb < kPanel - kLeft + kSteps ? nb : kPanel - kLeft + kSteps;
    for (int j = kPanel - kLeft; j < last; ++j) {
        Spread d;
        d.load(D + j * kPanel);
        double x = s[0] / d.get<0>();
        x = take(j, x, x != 0.0 && fabs(x) >= thr_of[j]);
        subtract<1, kLeft>(s, x, d);
    }
    if constexpr (kLeft > kSteps) solve_steps<kLeft - kSteps>(s, D, thr_of, nb, take);
}

// Forms columns J .. J + nb - 1 of R (panel p + 1) on the rows of part q, J + q kPanelRows and on.
__device__ void form_panel(const FcArgs& A, int32_t p, int32_t q, double* D /* [kPanel][kPanel] */,
                           double* next /* [kPanel][kPanel] */, double* thr_of /* [kPanel] */,
                           uint32_t* counts /* [4][kPanel + 1] */, int32_t* bad) {
    const int64_t N = A.N, J = static_cast<int64_t>(p + 1) * kPanel;
    const int nb = N - J < kPanel ? static_cast<int>(N - J) : kPanel;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const bool diag = wave == kPanelWaves - 1;   // this wave takes rows J + lane
    const int64_t i = J + (diag ? lane : q * kPanelRows + static_cast<int64_t>(threadIdx.x));
    const bool valid = i < N && !(diag && lane >= kPanel);
    const int64_t ic = valid ? i : J;
    if (diag) __builtin_amdgcn_s_setprio(3);   // the others wait for it
    // Row i of the panel's columns (entries above the diagonal are never used)
    double s[kPanel];
#pragma unroll
    for (int b = 0; b < kPanel; ++b) {
        const int64_t jb = J + b < N ? J + b : N - 1;
        const int64_t r = ic > jb ? ic : jb;
        s[b] = A.dense[packed_column(jb, N) + (r - jb)];
    }
    double thr = 0.0;
    if (diag) thr = A.droptol * A.colnorm[ic];
    if (p >= 0) {   // panel p's products
        const int par = p & 1;
        constexpr int kAhead = 4;   // entries of the row loaded ahead
        const double2* a2 = reinterpret_cast<const double2*>(A.prow + (par * N + ic) * kPanel);
        double2 ahead[kAhead / 2];
#pragma unroll
        for (int k = 0; k < kAhead / 2; ++k) ahead[k] = a2[k];
        for (int e = threadIdx.x; e < kPanel * kPanel; e += kPanelBlock) next[e] = A.pnext[par * kPanel * kPanel + e];
        __syncthreads();
        for (int k = 0; k < kPanel; k += kAhead) {
            double a[kAhead];
            Spread row[kAhead];
#pragma unroll
            for (int kk = 0; kk < kAhead; ++kk) row[kk].load(next + (k + kk) * kPanel);
#pragma unroll
            for (int kk = 0; kk < kAhead / 2; ++kk) {
                a[2 * kk] = ahead[kk].x;
                a[2 * kk + 1] = ahead[kk].y;
                if (k + kAhead < kPanel) ahead[kk] = a2[(k + kAhead) / 2 + kk];
            }
#pragma unroll
            for (int kk = 0; kk < kAhead; ++kk) {
                if (__ballot(a[kk] != 0.0) == 0ull) continue;
                subtract<0, kPanel>(s, a[kk], row[kk]);
            }
        }
    }
    if (diag) {
        if (lane < kPanel) thr_of[lane] = thr;
        const bool fine = factor_steps<kPanel>(s, D, thr, lane, nb);
        if (lane == 0) *bad = fine ? 0 : 1;
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
    if (*bad) {
        if (q == 0 && threadIdx.x == 0) atomicOr(&A.header->status, static_cast<uint32_t>(kErrPivot));
        if (threadIdx.x == 0) {   // nothing to copy or subtract
            const int64_t at = static_cast<int64_t>((p + 1) & 1) * A.parts + q;
            A.act_cnt[at] = 0;
            if (q == 0) A.act_skip[(p + 1) & 1] = 0;
            for (int c = 0; c < kPanel; ++c) A.col_cnt[at * kPanel + c] = 0;
        }
        if (i < N && !diag) A.pmask[((p + 1) & 1) * N + i] = 0;
        return;
    }
    const int par = (p + 1) & 1;
    const int t = threadIdx.x;
    const bool block = q == 0 && t < kPanel;   // a row of the diagonal block
    uint32_t mask = 0, mine = 0;
    if (!diag) {
        double* out = A.prow + (par * N + ic) * kPanel;
        solve_steps<kPanel>(s, D, thr_of, nb, [&](int j, double x, bool keep) {
            if (block) {
                x = t >= j ? D[j * kPanel + t - j] : 0.0;
                keep = x != 0.0;
            }
            keep = keep && valid;
            x = keep ? x : 0.0;
            mask |= keep ? 1u << j : 0u;
            const uint32_t c = static_cast<uint32_t>(__popcll(__ballot(keep)));
            if (lane == j) mine = c;
            if (valid) out[j] = x;
            if (q == 0 && t >= kPanel && t < 2 * kPanel) A.pnext[(par * kPanel + j) * kPanel + t - kPanel] = x;
            return x;
        });
        if (valid) A.pmask[par * N + i] = mask;
        if (lane < kPanel) counts[wave * (kPanel + 1) + lane] = mine;
        const uint64_t on = __ballot(mask != 0 && !block);
        if (lane == 0) counts[wave * (kPanel + 1) + kPanel] = static_cast<uint32_t>(__popcll(on));
        if (q == 0 && t == 0) A.act_skip[par] = static_cast<uint32_t>(__popcll(on));   // lanes kPanel .. 63
    }
    __syncthreads();
    const int64_t at = static_cast<int64_t>(par) * A.parts + q;
    if (t < kPanel) {
        uint32_t c = 0;
        for (int w = 0; w < kPanelWaves - 1; ++w) c += counts[w * (kPanel + 1) + t];
        A.col_cnt[at * kPanel + t] = c;
    }
    if (!diag) {
        uint32_t before = 0, all = 0;
        for (int w = 0; w < kPanelWaves - 1; ++w) {
            const uint32_t c = counts[w * (kPanel + 1) + kPanel];
            before += w < wave ? c : 0;
            all += c;
        }
        const uint64_t on = __ballot(mask != 0 && !block);
        if ((on >> lane) & 1ull)
            A.act[at * kPanelRows + before + __popcll(on & ((1ull << lane) - 1ull))] = static_cast<int32_t>(i);
        if (t == 0) A.act_cnt[at] = all;
    }
}

// Copies panel p's entries in the rows of part q into the compact factor (columns by ascending
// rows, the diagonal first).
__device__ void copy_panel(const FcArgs& A, int32_t p, int32_t q, int64_t* offset /* [kPanel] */,
                           uint32_t* counts /* [4][kPanel + 1] */, int32_t* full) {
    const int64_t N = A.N, J = static_cast<int64_t>(p) * kPanel;
    const int nb = N - J < kPanel ? static_cast<int>(N - J) : kPanel;
    const int par = p & 1, t = threadIdx.x, wave = t / kWave, lane = t & (kWave - 1);
    const int parts = static_cast<int>((N - J + kPanelRows - 1) / kPanelRows);
    const int64_t i = J + q * kPanelRows + static_cast<int64_t>(t);
    const bool valid = t < kPanelRows && i < N;
    const uint32_t mask = valid ? A.pmask[par * N + i] : 0u;
    if (wave == kPanelWaves - 1) {
        const uint32_t* cnt = A.col_cnt + static_cast<int64_t>(par) * A.parts * kPanel + (lane & (kPanel - 1));
        int64_t before = 0, all = 0;
        for (int w = 0; w < parts; ++w) {
            const uint32_t c = lane < nb ? cnt[w * kPanel] : 0u;
            before += w < q ? c : 0;
            all += c;
        }
        int64_t end = all;   // of the columns up to this one
        for (int off = 1; off < kPanel; off <<= 1) {
            const int64_t o = __shfl_up(end, off, kWave);
            if (lane >= off) end += o;
        }
        const int64_t rp = A.r_ptr[J];
        if (lane < kPanel) offset[lane] = rp + end - all + before;
        const int64_t total = rp + __shfl(end, kPanel - 1, kWave);
        if (lane == 0) *full = total > A.r_cap ? 1 : 0;
        if (q == 0) {
            if (lane < nb) A.r_ptr[J + lane + 1] = rp + end;
            if (lane == 0) A.counters[0] = total;
            if (lane == 0 && total > A.r_cap) atomicOr(&A.header->status, static_cast<uint32_t>(kErrCapacity));
        }
    } else {
        uint32_t mine = 0;
        for (int j = 0; j < kPanel; ++j) {
            const uint32_t c = static_cast<uint32_t>(__popcll(__ballot(((mask >> j) & 1u) != 0)));
            if (lane == j) mine = c;
        }
        if (lane < kPanel) counts[wave * (kPanel + 1) + lane] = mine;
    }
    __syncthreads();
    if (*full || wave == kPanelWaves - 1) return;
    for (int j = 0; j < nb; ++j) {
        const uint64_t m = __ballot(((mask >> j) & 1u) != 0);
        if ((mask >> j) & 1u) {
            int64_t pos = offset[j] + __popcll(m & ((1ull << lane) - 1ull));
            for (int w = 0; w < wave; ++w) pos += counts[w * (kPanel + 1) + j];
            A.r_row[pos] = static_cast<int32_t>(i);
            A.r_val[pos] = A.prow[(par * N + i) * kPanel + j];
        }
    }
}

// Subtracts panel p's products from S in tiles of kTile active rows by kTile active columns (the
// lower triangle of the panel's active rows past the next panel).  A column's kept entries are
// few (a fifth of the panel on BA(5000, 5)), and the same for all lanes: only they are gone through.
__device__ void update_tiles(const FcArgs& A, int32_t p, int64_t first, int64_t stride, double* ta, double* tb,
                             int32_t* ra, int32_t* rb, uint32_t* mb, uint32_t* prefix, int32_t* stop) {
    const int64_t N = A.N, J = static_cast<int64_t>(p) * kPanel;
    const int par = p & 1, t = threadIdx.x, wave = t / kWave, lane = t & (kWave - 1);
    const int parts = static_cast<int>((N - J + kPanelRows - 1) / kPanelRows);
    const uint32_t* cnt = A.act_cnt + static_cast<int64_t>(par) * A.parts;
    if (wave == 0) {   // where each part's active rows start
        uint32_t base = 0;
        for (int w0 = 0; w0 < parts; w0 += kWave) {
            uint32_t c = w0 + lane < parts ? cnt[w0 + lane] : 0u, end = c;
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t o = __shfl_up(end, off, kWave);
                if (lane >= off) end += o;
            }
            if (w0 + lane < parts) prefix[w0 + lane] = base + end - c;
            base += __shfl(end, kWave - 1, kWave);
        }
        if (lane == 0) {
            prefix[parts] = base;
            *stop = __hip_atomic_load(&A.header->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ? 1 : 0;
        }
    }
    __syncthreads();
    if (*stop) return;
    const int64_t skip = A.act_skip[par], count = static_cast<int64_t>(prefix[parts]) - skip;
    const int64_t side = (count + kTile - 1) / kTile, tiles = side * (side + 1) / 2;
    auto row_of = [&](int64_t x) {   // the x-th active row past the next panel, -1 past the end
        if (x >= count) return int32_t{-1};
        const uint32_t at = static_cast<uint32_t>(x + skip);
        int lo = 0, hi = parts;   // prefix[lo] <= at < prefix[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (prefix[mid] <= at)
                lo = mid;
            else
                hi = mid;
        }
        return A.act[(static_cast<int64_t>(par) * A.parts + lo) * kPanelRows + (at - prefix[lo])];
    };
    for (int64_t tile = first; tile < tiles; tile += stride) {
        int64_t h = static_cast<int64_t>((sqrt(8.0 * static_cast<double>(tile) + 1.0) - 1.0) * 0.5);
        while (h * (h + 1) / 2 > tile) --h;
        while ((h + 1) * (h + 2) / 2 <= tile) ++h;
        const int64_t g = tile - h * (h + 1) / 2;   // rows h, columns g <= h
        if (t < kTile) ra[t] = row_of(h * kTile + t);
        if (t >= kTile && t < 2 * kTile) {
            const int32_t r = row_of(g * kTile + t - kTile);
            rb[t - kTile] = r;
            mb[t - kTile] = r >= 0 ? A.pmask[par * N + r] : 0u;
        }
        __syncthreads();
        for (int e = t; e < 2 * kTile * (kPanel / 2); e += kPanelBlock) {
            const int l = (e / (kPanel / 2)) & (kTile - 1), k = 2 * (e % (kPanel / 2));
            const bool rows = e < kTile * (kPanel / 2);
            const int32_t r = rows ? ra[l] : rb[l];
            const double2 x = r >= 0 ? *reinterpret_cast<const double2*>(A.prow + (par * N + r) * kPanel + k) : double2{0.0, 0.0};
            double* to = (rows ? ta : tb) + l * kTilePitch + k;
            to[0] = x.x;
            to[1] = x.y;
        }
        if (t < 2 * kTile) (t < kTile ? ta : tb)[(t & (kTile - 1)) * kTilePitch + kPanel] = 0.0;
        const int32_t r = ra[lane];
        const uint32_t mr = r >= 0 ? A.pmask[par * N + r] : 0u;
        uint32_t any = mr;   // of all rows
        for (int off = kWave / 2; off > 0; off >>= 1) any |= __shfl_xor(any, off, kWave);
        double s[kTileCols];
        uint32_t touched = 0;
#pragma unroll
        for (int c = 0; c < kTileCols; ++c) {
            const int b = c * kPanelWaves + wave;
            const int32_t rc = b < kTile ? rb[b] : -1;
            const bool on = rc >= 0 && r >= rc && (mr & mb[b]) != 0;
            touched |= on ? 1u << c : 0u;
            s[c] = on ? A.dense[packed_column(rc, N) + (r - rc)] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kTileCols; ++c) {
            const int b = c * kPanelWaves + wave;
            if (b >= kTile) continue;
            uint32_t m = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(mb[b] & any)));
            while (m != 0) {   // four entries at a time; past the last the zeros at kPanel
                double x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int e = m != 0 ? __builtin_ctz(m) : kPanel;
                    m &= m - 1;
                    x[k] = ta[lane * kTilePitch + e] * tb[b * kTilePitch + e];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) s[c] = s[c] - x[k];
            }
            if ((touched >> c) & 1u) A.dense[packed_column(rb[b], N) + (r - rb[b])] = s[c];
        }
        __syncthreads();   // the tiles are rewritten
    }
}

// Launch p: workgroups 0 .. form - 1 form panel p + 1, the next `copy` ones copy panel p into the
// factor, the others subtract panel p's products.
__global__ void __launch_bounds__(kPanelBlock) fc_panel(FcArgs A, int32_t p, int32_t form, int32_t copy) {
    __shared__ double tiles[2 * kTile * kTilePitch];   // forming: two blocks of kPanel x kPanel
    __shared__ double thr_of[kPanel];
    __shared__ int64_t offset[kPanel];
    __shared__ uint32_t counts[(kPanelWaves - 1) * (kPanel + 1)];
    __shared__ uint32_t prefix[kMaxParts + 1];
    __shared__ int32_t ra[kTile], rb[kTile];
    __shared__ uint32_t mb[kTile];
    __shared__ int32_t flag;
    const int32_t w = static_cast<int32_t>(blockIdx.x);
    if (w < form)
        form_panel(A, p, w, tiles, tiles + kPanel * kPanel, thr_of, counts, &flag);
    else if (w < form + copy)
        copy_panel(A, p, w - form, offset, counts, &flag);
    else
        update_tiles(A, p, w - form - copy, static_cast<int64_t>(gridDim.x) - form - copy, tiles, tiles + kTile * kTilePitch,
                     ra, rb, mb, prefix, &flag);
}

// The windowed, sparsified inverse and tau~.  Column u needs exactly the later columns i of its
// window with R(i, u) != 0, so the columns form a DAG, on BA(5000, 5) 2225 deep: what bounds it is
// the latency of one column.  kInvWaves waves of one workgroup take columns in descending order from
// a counter and each waits, on a flag, for the columns it reads.  The wave holding the largest
// unfinished column never waits, so every wave finishes; a wait that outlasts kInvSpinLimit
// polls, or any error, stops the kernel.  A column's arithmetic is the serial one; only its place in
// the S~ pool depends on the schedule.
//
// The last kRing columns are also kept in LDS, up to kRingLen entries each, and a column with a window
// of at most kRingWindow and at most kInvEntries distinct rows stays in LDS altogether: its rows are
// found in a hash table while it waits, the sums are kept there, and the two orders (by magnitude, by row) are
// ranks counted against all entries: 4.7 us a level (32.1 -> 10.4 ms; BA(20 000, 5) 18.6 -> 5.9).  Eight
// waves instead of sixteen: BA(5000, 5)'s call 17.9 instead of 18.2 ms, BA(20 000, 5)'s 105 instead of 102.
// The others have a dense accumulator, stamps and a touched list (a slice of N of each per wave) in the
// workspace, and order a column in LDS when it has at most kInvLds nonzeros, else in their own
// kSortCap-entry slice of it (14 us a level).  Windows over twice kRingWindow throughout make columns of
// hundreds of entries, which eight waves do faster (BA(2000, 5), 128 columns: 402 ms, sixteen 412, held up
// for slots in LDS that nothing reads 419); over kRingWindow sixteen (a 4000-node mesh, 33 columns: 96, 106).
// (Shorter windows can make such columns too: ring of 100 cliques of 20, windows of 12, 671 with eight and 710 with
// sixteen; letting the upper waves leave at the first such column cost the columns in LDS 1 to 2 %, taken back.)
constexpr int kInvWaves = 16;
constexpr int kInvWidestWaves = 8;
constexpr int kInvLds = 512;
constexpr int64_t kInvSpinLimit = int64_t{1} << 26;
constexpr int kRing = 64;          // columns, a power of two
constexpr int kRingLen = 64;       // one entry per lane
constexpr int kRingWindow = 32;    // columns up to kRing - kRingWindow apart can be under way
constexpr int kInvEntries = 127;   // distinct rows besides u: with it two per lane
constexpr int kInvTable = 256;     // of them and one column more, at most three quarters full

// LDS of one wave: the hash table (rows, sums), each read entry's place in it, the table's places
// in the order they were taken, and two arrays to order entries by.  The general path uses it as one array.
struct InvWave {
    double sum[kInvTable];
    double val[kInvEntries + 1];
    int32_t key[kInvTable];   // -1: empty
    int32_t row[kInvEntries + 1];
    uint8_t place[kRingWindow * kRingLen];
    uint8_t taken[kInvEntries + 1];
};
static_assert(sizeof(InvWave) >= kInvLds * 12 && sizeof(InvWave) % 16 == 0);

struct InvShared {
    InvWave wave[kInvWaves];
    double val[kRing * kRingLen];
    int32_t row[kRing * kRingLen];
    int32_t len[kRing];             // -1: not kept here
    int32_t column[kRing];          // which column a slot holds, once it is published
    int32_t current[kInvWaves];     // the column each wave is at
    int32_t next_col, abort_all;
    unsigned long long pool;
};
static_assert(sizeof(InvShared) <= 160 * 1024);

template <class T>
__device__ __forceinline__ T shared_load(const RWC_LDS T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class T>
__device__ __forceinline__ void shared_store(RWC_LDS T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// A wave's LDS operations are performed in the order it issues them; this also waits for them.
__device__ __forceinline__ void lds_order() {
    wave_order();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
}

// A wave stops on an error of its own or of another wave.
__device__ void inv_fail(const FcArgs& A, RWC_LDS InvShared* S, uint32_t code) {
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicOr(&A.header->status, code);
        shared_store(&S->abort_all, 1);
    }
}

// Column u's slot in LDS may be written once no wave can be reading the column it held, u + kRing:
// the readers of that are at columns from u + kRing - kRingWindow on.
__device__ bool wait_for_slot(RWC_LDS InvShared* S, int32_t u) {
    const int lane = threadIdx.x & (kWave - 1);
    int64_t spins = 0;
    while (__ballot(lane < kInvWaves && shared_load(&S->current[lane < kInvWaves ? lane : 0]) >= u + kRing - kRingWindow) !=
           0ull) {
        if (shared_load(&S->abort_all) != 0 || ++spins > kInvSpinLimit) return false;
        __builtin_amdgcn_s_sleep(1);
    }
    return true;
}

enum InvResult { kInvDone, kInvGeneral, kInvStop };

// Column u in LDS.  i, coef: lane d's d-th entry of the window (rows ascending), `deps` of them.
__device__ InvResult ring_column(const FcArgs& A, RWC_LDS InvShared* S, int32_t u, double ruu, int32_t i, double coef,
                                 int deps) {
    const int lane = threadIdx.x & (kWave - 1);
    RWC_LDS InvWave* const W = &S->wave[threadIdx.x / kWave];
    // every row's place in the table, columns in the order they become ready
    uint32_t nt = 0;
    bool general = false;
    for (int d = deps - 1; d >= 0 && !general; --d) {
        const int32_t c = __builtin_amdgcn_readlane(i, d), slot = c & (kRing - 1);
        int64_t spins = 0;
        int32_t len, r;
        while (true) {   // what is read after the flag belongs to it
            const int32_t held = shared_load(&S->column[slot]);
            wave_order();
            len = shared_load(&S->len[slot]);
            r = shared_load(&S->row[slot * kRingLen + lane]);
            const int32_t stop = shared_load(&S->abort_all);
            if (__builtin_amdgcn_readfirstlane(held) == c) break;
            if (stop != 0 || ++spins > kInvSpinLimit) return kInvStop;
            __builtin_amdgcn_s_sleep(1);
        }
        wave_order();
        len = __builtin_amdgcn_readfirstlane(len);
        if (len < 0) {
            general = true;
            break;
        }
        uint32_t h = (static_cast<uint32_t>(r) * 0x9E3779B1u) >> 24;
        bool fresh = false, open = lane < len;
        while (__ballot(open) != 0ull) {   // at most kInvEntries + kRingLen rows in kInvTable places
            if (open) {
                int32_t old = -1;
                __hip_atomic_compare_exchange_strong(&W->key[h], &old, r, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WAVEFRONT);
                fresh = old == -1;
                open = !fresh && old != r;
                h = open ? (h + 1) & (kInvTable - 1) : h;
            }
        }
        if (lane < len) W->place[d * kRingLen + lane] = static_cast<uint8_t>(h);
        uint32_t cnt = 0;
        const uint32_t rank = rank_of(fresh, cnt);
        if (fresh) {
            W->sum[h] = 0.0;
            if (nt + rank <= kInvEntries) W->taken[nt + rank] = static_cast<uint8_t>(h);
        }
        nt += cnt;
        general = nt > static_cast<uint32_t>(kInvEntries);
    }
    lds_order();
    if (general) {   // empty the table
        for (int k = lane; k < kInvTable; k += kWave) W->key[k] = -1;
        lds_order();
        return kInvGeneral;
    }
    // the sums, in ascending row order of column u (the next column's entries are read ahead)
    if (deps > 0) {
        auto read = [&](int d, int32_t& len, uint32_t& h, double& x) {
            const int32_t slot = __builtin_amdgcn_readlane(i, d) & (kRing - 1);
            len = S->len[slot];
            h = W->place[d * kRingLen + lane];
            x = lane_value(coef, d) * S->val[slot * kRingLen + lane];
        };
        int32_t len, len1 = 0;
        uint32_t h, h1 = 0;
        double x, x1 = 0.0;
        read(0, len, h, x);
        for (int d = 0; d < deps; ++d) {
            if (d + 1 < deps) read(d + 1, len1, h1, x1);
            if (lane < len) W->sum[h] = W->sum[h] - x;
            wave_order();
            len = len1;
            h = h1;
            x = x1;
        }
    }
    // entry e of lane e % 64: the diagonal, then the table's rows
    const int m = static_cast<int>(nt) + 1;
    double a[2];
    int32_t row[2];
    bool live[2];
    uint32_t nz = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int e = lane + k * kWave;
        a[k] = 1.0 / ruu;
        row[k] = u;
        live[k] = e < m;
        if (live[k] && e > 0) {
            const uint32_t h = W->taken[e - 1];
            row[k] = W->key[h];
            a[k] = W->sum[h];
            W->key[h] = -1;
        }
        live[k] = live[k] && a[k] != 0.0;
        nz += static_cast<uint32_t>(__popcll(__ballot(live[k])));
    }
    wave_order();
    int32_t keep = static_cast<int32_t>(nz);
    bool kept[2] = {live[0], live[1]};
    // What every lane needs of all entries is read from LDS eight at a time (one at a time each read is
    // waited for; from the lanes' registers, by v_readlane: 20.8 ms for BA(5000, 5)'s call).
    int listed = m;   // W->row's entries to order the kept ones by
    if (static_cast<int64_t>(nz) > A.zeta) {
        // by decreasing magnitude, ties by row
        double mag[2];
        int32_t before[2] = {0, 0};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            mag[k] = live[k] ? fabs(a[k]) : 0.0;
            W->val[lane + k * kWave] = mag[k];
            W->row[lane + k * kWave] = row[k];
        }
        lds_order();
        for (int j = 0; j < m; j += 8) {   // (past m: zeros, which are larger than none)
            double o[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = W->val[j + q];
#pragma unroll
            for (int q = 0; q < 8; ++q) before[0] += o[q] > mag[0] ? 1 : 0;
            if (m > kWave) {
#pragma unroll
                for (int q = 0; q < 8; ++q) before[1] += o[q] > mag[1] ? 1 : 0;
            }
        }
        // equal magnitudes share a rank
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (live[k]) W->taken[before[k]] = static_cast<uint8_t>(lane + k * kWave);
        lds_order();
        bool shared = false;
#pragma unroll
        for (int k = 0; k < 2; ++k) shared = shared || (live[k] && W->taken[before[k]] != lane + k * kWave);
        if (__ballot(shared) != 0ull) {
            for (int j = 0; j < m; ++j) {
                const double o = W->val[j];
                const int32_t r = W->row[j];
                before[0] += o == mag[0] && r < row[0] ? 1 : 0;
                before[1] += o == mag[1] && r < row[1] ? 1 : 0;
            }
        }
        lds_order();
#pragma unroll
        for (int k = 0; k < 2; ++k)
        {
            if (lane + k * kWave >= keep) W->val[lane + k * kWave] = 0.0;
            if (live[k]) {
                W->val[before[k]] = mag[k];
                W->row[before[k]] = row[k];
            }
        }
        lds_order();
        // the 1-norm in that order (past the end zeros), then the tail grown from the smallest entry
        double l1 = 0.0;
        for (int32_t j = 0; j < keep; j += 8) {
            double o[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = W->val[j + q];
#pragma unroll
            for (int q = 0; q < 8; ++q) l1 += o[q];
        }
        const double lim = A.eps_p * l1;
        double tail = 0.0;
        for (bool more = true; more && keep > 0;) {
            double o[8];
            const int32_t from = keep;
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = W->val[from > q ? from - 1 - q : 0];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double next = tail + o[q];
                more = more && from > q && next <= lim;
                tail = more ? next : tail;
                keep -= more ? 1 : 0;
            }
        }
        keep = __builtin_amdgcn_readfirstlane(keep);
#pragma unroll
        for (int k = 0; k < 2; ++k) kept[k] = live[k] && before[k] < keep;
        listed = keep;
    } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) W->row[lane + k * kWave] = live[k] ? row[k] : 0x7FFFFFFF;
        lds_order();
    }
    int32_t at[2] = {0, 0};   // by ascending row
    for (int j = 0; j < listed; j += 8) {
        int32_t r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = W->row[j + q];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int32_t x = j + q < listed ? r[q] : 0x7FFFFFFF;
            at[0] += x < row[0] ? 1 : 0;
            at[1] += x < row[1] ? 1 : 0;
        }
    }
    lds_order();
    if (!wait_for_slot(S, u)) return kInvStop;
    const int32_t slot = u & (kRing - 1);
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (kept[k]) {
            W->val[at[k]] = a[k];
            if (keep <= kRingLen) {
                S->val[slot * kRingLen + at[k]] = a[k];
                S->row[slot * kRingLen + at[k]] = row[k];
            }
        }
    if (lane == 0) S->len[slot] = keep <= kRingLen ? keep : -1;
    lds_order();
    if (lane == 0) shared_store(&S->column[slot], u);   // what waits for column u goes on
    unsigned long long got = 0;
    if (lane == 0) got = __hip_atomic_fetch_add(&S->pool, static_cast<unsigned long long>(keep), __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
    const int64_t sp = static_cast<int64_t>(__shfl(got, 0, kWave));
    if (sp + keep > A.s_cap) {
        inv_fail(A, S, static_cast<uint32_t>(kErrCapacity));
        return kInvStop;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (kept[k]) {
            A.s_row[sp + at[k]] = row[k];
            A.s_val[sp + at[k]] = a[k];
        }
    double t2 = 0.0;   // ||S~(:, u)||^2 in row order
    for (int32_t j = 0; j < keep; j += 8) {
        double o[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = j + q < keep ? W->val[j + q] : 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) t2 += o[q] * o[q];
    }
    if (lane == 0) {
        A.s_start[u] = sp;
        A.s_len[u] = keep;
        A.tau[node_of_column(u, A.v)] = t2;
    }
    return kInvDone;
}

// Column u by the dense accumulator, the window's entries [c0 + 1, c1) of any number.  ring: some column
// may read it from LDS.
__device__ InvResult general_column(const FcArgs& A, RWC_LDS InvShared* S, int32_t u, int64_t c0, int64_t c1, double ruu,
                                    int64_t w, bool ring) {
    const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const int64_t N = A.N;
    double* acc = A.acc + static_cast<int64_t>(wave) * N;
    int32_t* stamps = A.stamp + static_cast<int64_t>(wave) * N;
    int32_t* touched = A.touched + static_cast<int64_t>(wave) * N;
    const int32_t stamp = -(u + 1);   // negative stamps: the factor's are positive
    uint32_t nt = 1;
    if (lane == 0) {
        st(&acc[u], 1.0 / ruu);
        st(&stamps[u], stamp);
        st(&touched[0], u);
    }
    wave_order();
    // the window's entries of column u, 64 at a time (lane l: entry p0 + l); their columns of
    // S~ are waited for together, then added in ascending row order, each a dependent load of
    // its entries and then of their stamps and accumulators
    for (int64_t p0 = c0 + 1; p0 < c1; p0 += kWave) {
        const int64_t p = p0 + lane;
        int32_t i = -1;
        double coef = 0.0;
        if (p < c1) {
            const int32_t r = A.r_row[p];
            if (r <= u + w) {
                i = r;
                coef = A.r_val[p] / ruu;
            }
        }
        const uint64_t live = __ballot(i >= 0);   // a prefix: rows ascend
        if (live == 0ull) break;
        int64_t spins = 0;
        while (__ballot(i >= 0 && __hip_atomic_load(&A.done[i], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0) !=
               0ull) {
            if (shared_load(&S->abort_all) != 0 || ++spins > kInvSpinLimit) return kInvStop;
            __builtin_amdgcn_s_sleep(2);
        }
        int64_t s0 = 0;
        int32_t sl = 0;
        if (i >= 0) {
            s0 = A.s_start[i];
            sl = A.s_len[i];
        }
        for (uint64_t bits = live; bits != 0ull; bits &= bits - 1) {
            const int l = __builtin_ctzll(bits);
            const double cf = __shfl(coef, l, kWave);
            const int64_t b0 = __shfl(s0, l, kWave);
            const int32_t bl = __shfl(sl, l, kWave);
            for (int32_t q0 = 0; q0 < bl; q0 += kWave) {
                const int32_t q = q0 + lane;
                int32_t r = -1;
                double sv = 0.0;
                if (q < bl) {
                    r = A.s_row[b0 + q];
                    sv = A.s_val[b0 + q];
                }
                const int32_t rc = r >= 0 ? r : u;   // a valid address for every lane
                const int32_t sg = ld(&stamps[rc]);
                const double old = ld(&acc[rc]);
                const bool fresh = r >= 0 && sg != stamp;
                uint32_t cnt = 0;
                const uint32_t rk = rank_of(fresh, cnt);
                if (fresh) {
                    st(&stamps[r], stamp);
                    st(&touched[nt + rk], r);   // distinct rows below N
                }
                nt += cnt;
                if (r >= 0) st(&acc[r], (fresh ? 0.0 : old) - cf * sv);
            }
            wave_order();
        }
    }
    wave_order();
    // the nonzeros of S*(:, u), in LDS when they fit, else in this wave's global scratch
    const bool small = nt <= static_cast<uint32_t>(kInvLds);
    double* const lds = (double*)(&S->wave[wave]);
    double* val = small ? lds : A.inv_val + static_cast<int64_t>(wave) * kSortCap;
    int32_t* row = small ? reinterpret_cast<int32_t*>(lds + kInvLds) : A.inv_row + static_cast<int64_t>(wave) * kSortCap;
    uint32_t nz = 0;
    for (uint32_t t0 = 0; t0 < nt; t0 += kWave) {
        const uint32_t tt = t0 + lane;
        int32_t r = -1;
        double a = 0.0;
        if (tt < nt) {
            r = ld(&touched[tt]);
            a = ld(&acc[r]);
        }
        const bool live = r >= 0 && a != 0.0;
        uint32_t cnt = 0;
        const uint32_t rk = rank_of(live, cnt);
        if (nz + cnt > static_cast<uint32_t>(kSortCap)) {
            inv_fail(A, S, static_cast<uint32_t>(kErrCapacity));
            return kInvStop;
        }
        if (live) {
            val[nz + rk] = a;
            row[nz + rk] = r;
        }
        nz += cnt;
    }
    lds_order();
    int32_t keep = static_cast<int32_t>(nz);
    if (static_cast<int64_t>(nz) > A.zeta) {
        wave_sort(val, row, static_cast<int32_t>(nz), [](double va, int32_t ra, double vb, int32_t rb) {
            const double a = fabs(va), b = fabs(vb);
            return a > b || (a == b && ra < rb);
        });
        // the 1-norm in sorted order, then the tail grown from the smallest entry: every lane
        // adds the same values in the same order, read from the lanes that loaded them
        double l1 = 0.0;
        for (int32_t t0 = 0; t0 < static_cast<int32_t>(nz); t0 += kWave) {
            const int32_t t = t0 + lane;
            const double a = t < static_cast<int32_t>(nz) ? fabs(val[t]) : 0.0;
            const int32_t m = static_cast<int32_t>(nz) - t0 < kWave ? static_cast<int32_t>(nz) - t0 : kWave;
            for (int32_t l = 0; l < m; ++l) l1 += lane_value(a, l);
        }
        const double lim = A.eps_p * l1;
        double tail = 0.0;
        int32_t k = static_cast<int32_t>(nz);
        for (bool more = true; more && k > 0;) {
            const int32_t base = k > kWave ? k - kWave : 0;   // entries [base, k), largest index first
            const int32_t t = base + lane;
            const double a = t < k ? fabs(val[t]) : 0.0;
            for (int32_t l = k - 1 - base; l >= 0; --l) {
                const double x = lane_value(a, l);
                if (!(tail + x <= lim)) {
                    more = false;
                    break;
                }
                tail += x;
                --k;
            }
        }
        keep = k;
    }
    wave_sort(val, row, keep, [](double, int32_t ra, double, int32_t rb) { return ra < rb; });
    unsigned long long got = 0;
    if (lane == 0) got = __hip_atomic_fetch_add(&S->pool, static_cast<unsigned long long>(keep), __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
    const int64_t sp = static_cast<int64_t>(__shfl(got, 0, kWave));
    if (sp + keep > A.s_cap) {
        inv_fail(A, S, static_cast<uint32_t>(kErrCapacity));
        return kInvStop;
    }
    for (int32_t k = lane; k < keep; k += kWave) {
        A.s_row[sp + k] = row[k];
        A.s_val[sp + k] = val[k];
    }
    double t2 = 0.0;   // ||S~(:, u)||^2 in row order, as above
    for (int32_t t0 = 0; t0 < keep; t0 += kWave) {
        const int32_t t = t0 + lane;
        const double a = t < keep ? val[t] : 0.0;
        const int32_t m = keep - t0 < kWave ? keep - t0 : kWave;
        for (int32_t l = 0; l < m; ++l) {
            const double x = lane_value(a, l);
            t2 += x * x;
        }
    }
    if (lane == 0) {
        A.s_start[u] = sp;
        A.s_len[u] = keep;
        A.tau[node_of_column(u, A.v)] = t2;
    }
    // the columns kept in LDS, then the table empty again
    if (!ring) return kInvDone;
    if (!wait_for_slot(S, u)) return kInvStop;
    const int32_t slot = u & (kRing - 1);
    if (lane < keep && keep <= kRingLen) {
        S->val[slot * kRingLen + lane] = val[lane];
        S->row[slot * kRingLen + lane] = row[lane];
    }
    if (lane == 0) S->len[slot] = keep <= kRingLen ? keep : -1;
    lds_order();
    if (lane == 0) shared_store(&S->column[slot], u);
    for (int k = lane; k < kInvTable; k += kWave) S->wave[wave].key[k] = -1;
    lds_order();
    return kInvDone;
}

__global__ void __launch_bounds__(kInvWaves * kWave) fc_inverse(FcArgs A) {
    extern __shared__ double inv_lds[];
    RWC_LDS InvShared* const S = (RWC_LDS InvShared*)inv_lds;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const int32_t N = A.N, v = A.v;
    if (threadIdx.x == 0) {
        S->next_col = 0;
        S->pool = 0;
        S->abort_all = A.header->status != 0 ? 1 : 0;   // the factor is incomplete
    }
    for (int k = threadIdx.x; k < kRing; k += blockDim.x) S->column[k] = -1;
    if (threadIdx.x < kInvWaves) S->current[threadIdx.x] = static_cast<int>(threadIdx.x) * kWave < static_cast<int>(blockDim.x) ? N : -1;
    for (int k = lane; k < kInvTable; k += kWave) S->wave[wave].key[k] = -1;
    __syncthreads();
    const double dmax = *A.dmax;
    // with windows over kRingWindow columns throughout none is read from LDS, so none is held up until its slot
    // there is free
    const bool ring = A.ws < kRingWindow + 1 || N <= kRingWindow;
    while (shared_load(&S->abort_all) == 0) {
        int32_t t = 0;
        if (lane == 0) t = __hip_atomic_fetch_add(&S->next_col, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        t = __builtin_amdgcn_readfirstlane(t);
        if (t >= N) break;
        const int32_t u = N - 1 - t;
        if (lane == 0) shared_store(&S->current[wave], u);
        wave_order();
        const int32_t x = A.node_index[node_of_column(u, v)];
        const int64_t c0 = A.r_ptr[u], c1 = A.r_ptr[u + 1];
        const double ruu = A.r_val[c0];
        int64_t w = static_cast<int64_t>(floor(A.ws * (1.0 + A.strength[x] / dmax)));
        if (w > N) w = N;
        InvResult result = kInvGeneral;
        if (w <= kRingWindow) {   // its entries in the window are among the first 32 below the diagonal
            const int64_t p = c0 + 1 + lane;
            int32_t i = -1;
            double coef = 0.0;
            if (p < c1) {
                const int32_t r = A.r_row[p];
                if (r <= u + w) {
                    i = r;
                    coef = A.r_val[p] / ruu;
                }
            }
            result = ring_column(A, S, u, ruu, i, coef, static_cast<int>(__popcll(__ballot(i >= 0))));
        }
        if (result == kInvGeneral) result = general_column(A, S, u, c0, c1, ruu, w, ring);
        if (result == kInvStop) {
            if (shared_load(&S->abort_all) == 0) inv_fail(A, S, static_cast<uint32_t>(kErrWait));   // a wait ran out (not expected)
            break;
        }
        // every lane's stores of column u are done before the flag that publishes it
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) __hip_atomic_store(&A.done[u], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        lds_order();
    }
    if (lane == 0) shared_store(&S->current[wave], -1);
    __syncthreads();
    if (threadIdx.x == 0 && S->abort_all == 0) A.counters[1] = static_cast<int64_t>(S->pool);
}

struct FcLayout {
    WsHeader* header;
    int64_t* counters;
    double* dmax;
    int64_t *r_ptr, *r_next, *r_colend, *head, *tail, *s_start;
    int32_t *r_row, *s_len, *s_row, *stamp, *touched, *done, *inv_row;
    double* inv_val;
    double *r_val, *s_val, *acc, *colnorm, *dense, *prow, *pnext;
    uint32_t *pmask, *act_cnt, *act_skip, *col_cnt;
    int32_t* act;
    int32_t parts;
    size_t total;
};

// Dense IChol needs the (n - 1)(n) / 2 doubles of a packed triangle; the automatic choice takes
// it up to this many bytes (an eighth of the device's 288 GB: n - 1 <= 92681; BA(60000, 5)'s
// triangle factors 47x faster than the chain).
constexpr uint64_t kDenseAutoBytes = uint64_t{32} << 30;
constexpr int64_t kDenseMaxColumns = int64_t{1} << 20;

bool use_dense(const rwc_fastchol_params* p, int32_t n) {
    const uint64_t N = static_cast<uint64_t>(n - 1);
    if (p->method == RWC_FASTCHOL_DENSE) return true;
    if (p->method == RWC_FASTCHOL_CHAIN) return false;
    return N * (N + 1) / 2 * sizeof(double) <= kDenseAutoBytes;
}

static_assert(2 * kPanel * sizeof(double) >= kInvWaves * 16);

FcLayout carve_fc(void* ws, int32_t n, int64_t r_cap, int64_t s_cap, bool dense) {
    Carver c(ws);
    FcLayout L{};
    const int64_t N = n - 1;
    L.header = c.take<WsHeader>(kHeaderBytes / sizeof(WsHeader));
    L.counters = c.take<int64_t>(2);
    L.dmax = c.take<double>(1);
    L.r_ptr = c.take<int64_t>(N + 1);
    L.s_start = c.take<int64_t>(N);
    L.s_len = c.take<int32_t>(N);
    // the accumulators, stamps and touched lists of the inverse (and the chain); before them, the dense
    // form's panels, which are larger
    L.acc = c.take<double>(2 * kPanel * N);
    L.stamp = reinterpret_cast<int32_t*>(L.acc + kInvWaves * N);
    L.touched = L.stamp + kInvWaves * N;
    L.done = c.take<int32_t>(N);
    L.inv_val = c.take<double>(kInvWaves * kSortCap);
    L.inv_row = c.take<int32_t>(kInvWaves * kSortCap);
    L.r_row = c.take<int32_t>(r_cap);
    L.r_val = c.take<double>(r_cap);
    L.s_row = c.take<int32_t>(s_cap);
    L.s_val = c.take<double>(s_cap);
    if (!dense) {   // the chain's row lists
        L.head = c.take<int64_t>(N);
        L.tail = c.take<int64_t>(N);
        L.r_next = c.take<int64_t>(r_cap);
        L.r_colend = c.take<int64_t>(r_cap);
    } else {
        L.colnorm = c.take<double>(N);
        L.parts = static_cast<int32_t>((N + kPanelRows - 1) / kPanelRows);
        L.prow = L.acc;
        L.pmask = c.take<uint32_t>(2 * N);
        L.pnext = c.take<double>(2 * kPanel * kPanel);
        L.act = c.take<int32_t>(static_cast<size_t>(2) * L.parts * kPanelRows);
        L.act_cnt = c.take<uint32_t>(2 * L.parts);
        L.act_skip = c.take<uint32_t>(2);
        L.col_cnt = c.take<uint32_t>(static_cast<size_t>(2) * L.parts * kPanel);
        L.dense = c.take<double>(static_cast<size_t>(N) * static_cast<size_t>(N + 1) / 2);
    }
    L.total = c.used();
    return L;
}

int check_fc(const rwc_csr* g, const rwc_fastchol_params* p) {
    if (!g || !p) return fail(RWC_ERR_INVALID_ARG, "g and p are required");
    if (g->n < 2 || !g->row_ptr || !g->node_id) return fail(RWC_ERR_INVALID_ARG, "g is not a built CSR");
    RWC_CHECK(require_connected(g, "rwc_fastchol"));
    if (!(p->droptol >= 0.0) || !(p->window >= 1.0) || p->zeta < 0 || !(p->eps_p >= 0.0))
        return fail(RWC_ERR_INVALID_ARG, "droptol and eps_p must be >= 0, window >= 1, zeta >= 0");
    if (p->factor_capacity < g->n - 1 || p->inverse_capacity < 0)
        return fail(RWC_ERR_INVALID_ARG, "factor_capacity must be at least n - 1 and inverse_capacity >= 0");
    if (p->method != RWC_FASTCHOL_AUTO && p->method != RWC_FASTCHOL_CHAIN && p->method != RWC_FASTCHOL_DENSE)
        return fail(RWC_ERR_INVALID_ARG, "method must be RWC_FASTCHOL_AUTO, _CHAIN or _DENSE");
    if (p->method == RWC_FASTCHOL_DENSE && g->n - 1 > kDenseMaxColumns)
        return fail(RWC_ERR_TOO_LARGE, "dense IChol takes at most %lld columns", static_cast<long long>(kDenseMaxColumns));
    return RWC_OK;
}

}  // namespace
}  // namespace rwc

using namespace rwc;

extern "C" int rwc_fastchol_workspace(const rwc_csr* g, const rwc_fastchol_params* p, size_t* bytes) {
    clear_error();
    if (!bytes) return fail(RWC_ERR_INVALID_ARG, "bytes is null");
    RWC_CHECK(check_fc(g, p));
    *bytes = carve_fc(nullptr, g->n, p->factor_capacity, p->inverse_capacity, use_dense(p, g->n)).total;
    return RWC_OK;
}

extern "C" int rwc_fastchol(const rwc_csr* g, const rwc_fastchol_params* p, double* tau, void* ws, size_t ws_bytes,
                            void* stream) {
    clear_error();
    RWC_CHECK(check_fc(g, p));
    if (!tau) return fail(RWC_ERR_INVALID_ARG, "tau is required");
    const bool dense = use_dense(p, g->n);
    RWC_CHECK(check_workspace(ws, ws_bytes,
                              carve_fc(nullptr, g->n, p->factor_capacity, p->inverse_capacity, dense).total));
    FcLayout L = carve_fc(ws, g->n, p->factor_capacity, p->inverse_capacity, dense);
    FcArgs A{};
    A.row_ptr = g->row_ptr;
    A.col = g->col;
    A.weight = g->weight;
    A.strength = g->strength;
    A.node_id = g->node_id;
    A.node_index = g->node_index;
    A.n = g->n;
    A.v = g->pivot;
    A.N = g->n - 1;
    A.zeta = p->zeta;
    A.droptol = p->droptol;
    A.ws = p->window;
    A.eps_p = p->eps_p;
    A.r_ptr = L.r_ptr;
    A.r_row = L.r_row;
    A.r_val = L.r_val;
    A.r_next = L.r_next;
    A.r_colend = L.r_colend;
    A.head = L.head;
    A.tail = L.tail;
    A.r_cap = p->factor_capacity;
    A.s_start = L.s_start;
    A.s_len = L.s_len;
    A.s_row = L.s_row;
    A.s_val = L.s_val;
    A.s_cap = p->inverse_capacity;
    A.acc = L.acc;
    A.stamp = L.stamp;
    A.touched = L.touched;
    A.done = L.done;
    A.inv_val = L.inv_val;
    A.inv_row = L.inv_row;
    A.dmax = L.dmax;
    A.dense = L.dense;
    A.colnorm = L.colnorm;
    A.prow = L.prow;
    A.pmask = L.pmask;
    A.pnext = L.pnext;
    A.act = L.act;
    A.act_cnt = L.act_cnt;
    A.act_skip = L.act_skip;
    A.col_cnt = L.col_cnt;
    A.parts = L.parts;
    A.tau = tau;
    A.header = L.header;
    A.counters = L.counters;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(fc_begin, dim3(1), dim3(kWave), 0, s, A);
    const int64_t N = g->n - 1;
    auto clear_stamps = [&] {
        hipLaunchKernelGGL(fill_i32, dim3(blocks_for(kInvWaves * N, 256)), dim3(256), 0, s, L.stamp, kInvWaves * N, 0);
    };
    hipLaunchKernelGGL(fill_i32, dim3(blocks_for(N, 256)), dim3(256), 0, s, L.done, N, 0);
    if (dense) {
        const int64_t cells = N * (N + 1) / 2;
        hipLaunchKernelGGL(fc_dense_clear, dim3(static_cast<unsigned>(std::min<int64_t>(blocks_for(cells, 256), 8192))),
                           dim3(256), 0, s, reinterpret_cast<uint64_t*>(L.dense), cells);
        hipLaunchKernelGGL(fc_dense_scatter, dim3(blocks_for(N, 256 / kWave)), dim3(256), 0, s, A);
        // launch p reads what every workgroup of launch p - 1 wrote; the last one only copies
        const int64_t panels = (N + kPanel - 1) / kPanel;
        for (int64_t q = -1; q < panels; ++q) {
            const int64_t J0 = q * kPanel, J1 = J0 + kPanel;
            const int64_t form = J1 < N ? (N - J1 + kPanelRows - 1) / kPanelRows : 0;
            const int64_t copy = q >= 0 ? (N - J0 + kPanelRows - 1) / kPanelRows : 0;
            const int64_t side = J1 + kPanel < N ? (N - J1 - kPanel + kTile - 1) / kTile : 0;   // at most, in tiles
            const int64_t tiles = q >= 0 ? std::min<int64_t>(side * (side + 1) / 2, 3 * device_cu_count()) : 0;
            hipLaunchKernelGGL(fc_panel, dim3(static_cast<unsigned>(form + copy + tiles)), dim3(kPanelBlock), 0, s, A,
                               static_cast<int32_t>(q), static_cast<int32_t>(form), static_cast<int32_t>(copy));
        }
        clear_stamps();   // where the panels were
    } else {
        clear_stamps();
        hipLaunchKernelGGL(fc_ichol, dim3(1), dim3(kWave), 0, s, A);
    }
    // the longest windows on fewer waves, whose accumulators and sort buffers share the caches better
    const int waves = p->window <= 2 * kRingWindow ? kInvWaves : kInvWidestWaves;
    hipLaunchKernelGGL(fc_inverse, dim3(1), dim3(waves * kWave), sizeof(InvShared), s, A);
    RWC_HIP(hipGetLastError());
    return RWC_OK;
}

extern "C" int rwc_fastchol_sizes(const void* ws, int64_t* factor_entries, int64_t* inverse_entries, void* stream) {
    clear_error();
    if (!ws || !factor_entries || !inverse_entries) return fail(RWC_ERR_INVALID_ARG, "ws and outputs are required");
    FcLayout L = carve_fc(const_cast<void*>(ws), 2, 1, 0, false);
    int64_t c[2] = {0, 0};
    hipStream_t s = static_cast<hipStream_t>(stream);
    RWC_HIP(hipMemcpyAsync(c, L.counters, sizeof(c), hipMemcpyDeviceToHost, s));
    RWC_HIP(hipStreamSynchronize(s));
    *factor_entries = c[0];
    *inverse_entries = c[1];
    return RWC_OK;
}
