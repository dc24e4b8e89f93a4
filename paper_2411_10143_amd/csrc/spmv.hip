// SpMV kernel family for gfx950: y = alpha*A*x + beta*y.
//
// The configuration space follows the paper's (Section III-B-2): several
// storage formats, several algorithms for CSR, and a thread-count parameter
// for CSR-vector.  On MI355X the kernels are written for wave64:
//
//   spmv_csr_vector<L>  L lanes (1..64) share one row, strided over its
//                       entries; a DPP sum over the L lanes adds them
//                       (Bell & Garland's CSR-vector; the paper's TpV).
//   spmv_csr_scalar     one lane per row; the workgroup first forms the
//                       products of its 256-row block in LDS with coalesced
//                       loads, then each lane sums its row from LDS.
//   spmv_merge          merge-path load balancing (Merrill & Garland): every
//                       thread takes an equal share of the merged sequence
//                       (row ends + entries); rows cut by a thread or block
//                       boundary are completed by a deterministic carry pass.
//   spmv_ell            column-major ELLPACK, one lane per row.
//   spmv_coo            row-sorted triples, equal entry shares per thread,
//                       the same carry scheme as merge-path.
//   spmv_dia, HYB       diahyb.hip (HYB's ELL part is spmv_hyb_ell below).
//
// Matrix arrays are streamed with non-temporal loads so the cache keeps the
// gathered vector; row blocks are mapped so that each XCD works on one
// contiguous slice of rows (its L2 then holds the x entries that slice uses).
// Every reduction has a fixed order, so a configuration always returns the
// same bits for the same input.
#include <algorithm>

#include "diahyb.hpp"
#include "matrix.hpp"
#include "panel.hpp"
#include "slices.hpp"
#include "solvers.hpp"

using ck::ld_stream;

constexpr int kMergeIPT = 8;   // merged items per thread  (2048 per workgroup)
constexpr int kMergeSlack = 64;   // items a workgroup may start before its nominal start
constexpr int kMergeSpan = 256 * kMergeIPT - kMergeSlack;   // merged items between nominal starts
constexpr int kCooIPT = 8;     // entries per thread       (2048 per workgroup)
constexpr int kScalarCap = 4096;  // products staged per LDS chunk (CSR-scalar)

// ---------------------------------------------------------------------------
// Row-blocked kernels process row groups g = b, b+G, b+2G, ... with
// G = min(groups, kRowBlocks) logical blocks: at every step the 8 XCDs each
// cover one contiguous slice of rows, and no launch needs more workgroups
// than the dispatcher can issue in a few microseconds.
//
// Fused CG step: every block adds q_i * p_i over its rows (x = p, y = q) and
// stores its partial; the r update (or a one-block finish) sums them in block order
// and sets alpha = rho / sigma (or flags a breakdown when sigma <= 0).
template <typename T, bool DOT>
__device__ __forceinline__ void cg_sigma_epilogue(T mine, ck::CgDev<T> *cg, T *partials,
                                                  int64_t b, int64_t G) {
    if constexpr (DOT) {
        __shared__ T lds[4];
        const T d = ck::block_sum(mine, lds);
        if (threadIdx.x == 0)
            partials[b] = d;
    }
}

__device__ __forceinline__ bool skipped(const int *skip) { return skip != nullptr && *skip != 0; }

template <int L, typename T, bool BETA, bool DOT>
__global__ __launch_bounds__(256) void spmv_csr_vector(int n, int64_t G,
                                                       const int *__restrict__ rp,
                                                       const int *__restrict__ col,
                                                       const T *__restrict__ val, T alpha,
                                                       const T *__restrict__ x, T beta,
                                                       T *__restrict__ y,
                                                       const int *__restrict__ skip,
                                                       ck::CgDev<T> *cg,
                                                       T *__restrict__ partials) {
    if (skipped(skip))
        return;
    const int64_t b = ck::xcd_block(G);
    if (b < 0)
        return;
    constexpr int R = 256 / L;
    const int lane = threadIdx.x & (L - 1);
    const int64_t groups = ((int64_t)n + R - 1) / R;
    T mine = 0;
    for (int64_t g = b; g < groups; g += G) {
        const int64_t row = g * R + threadIdx.x / L;
        T sum = 0;
        if (row < n) {
            const int k0 = rp[row], k1 = rp[row + 1];
            T s0 = 0, s1 = 0;
            int k = k0 + lane;
            for (; k + L < k1; k += 2 * L) {
                s0 += ld_stream(&val[k]) * x[ld_stream(&col[k])];
                s1 += ld_stream(&val[k + L]) * x[ld_stream(&col[k + L])];
            }
            if (k < k1)
                s0 += ld_stream(&val[k]) * x[ld_stream(&col[k])];
            sum = s0 + s1;
        }
        sum = ck::group_sum_last<L>(sum);   // valid in lane L - 1
        if (lane == L - 1 && row < n) {
            T out = alpha * sum;
            if (BETA)
                out += beta * y[row];
            y[row] = out;
            if (DOT)
                mine += out * x[row];
        }
    }
    cg_sigma_epilogue<T, DOT>(mine, cg, partials, b, G);
}

template <typename T, bool BETA, bool DOT>
__global__ __launch_bounds__(256) void spmv_csr_scalar(int n, int64_t G,
                                                       const int *__restrict__ rp,
                                                       const int *__restrict__ col,
                                                       const T *__restrict__ val, T alpha,
                                                       const T *__restrict__ x, T beta,
                                                       T *__restrict__ y,
                                                       const int *__restrict__ skip,
                                                       ck::CgDev<T> *cg,
                                                       T *__restrict__ partials) {
    __shared__ T prod[kScalarCap];
    __shared__ int srp[257];
    if (skipped(skip))
        return;
    const int64_t b = ck::xcd_block(G);
    if (b < 0)
        return;
    const int tid = threadIdx.x;
    const int64_t groups = ((int64_t)n + 255) / 256;
    T mine = 0;
    for (int64_t g = b; g < groups; g += G) {
        const int64_t r0 = g * 256;
        const int rows = (int)min<int64_t>(256, n - r0);
        __syncthreads();   // srp/prod of the previous group are no longer read
        for (int t = tid; t <= rows; t += 256)
            srp[t] = rp[r0 + t];
        __syncthreads();
        const int k0 = srp[0], k1 = srp[rows];
        const int my_lo = tid < rows ? srp[tid] : 0;
        const int my_hi = tid < rows ? srp[tid + 1] : 0;
        T acc = 0;
        for (int base = k0; base < k1; base += kScalarCap) {
            const int cnt = min(kScalarCap, k1 - base);
            // eight products per thread per step, their loads and gathers in
            // flight together (index clamped, store masked)
            for (int t0 = 0; t0 < cnt; t0 += 8 * 256) {
                int cc[8];
                T vv[8], xv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int t = min(t0 + u * 256 + tid, cnt - 1);
                    cc[u] = ld_stream(&col[base + t]);
                    vv[u] = ld_stream(&val[base + t]);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    xv[u] = x[cc[u]];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (t0 + u * 256 + tid < cnt)
                        prod[t0 + u * 256 + tid] = vv[u] * xv[u];
            }
            __syncthreads();
            const int lo = max(my_lo, base), hi = min(my_hi, base + cnt);
            for (int k = lo; k < hi; ++k)
                acc += prod[k - base];
            __syncthreads();
        }
        if (tid < rows) {
            const int64_t row = r0 + tid;
            T out = alpha * acc;
            if (BETA)
                out += beta * y[row];
            y[row] = out;
            if (DOT)
                mine += out * x[row];
        }
    }
    cg_sigma_epilogue<T, DOT>(mine, cg, partials, b, G);
}

template <typename T, bool BETA, bool DOT>
__device__ __forceinline__ void ell_rows(int n, int64_t G, int K, int64_t pitch,
                                         const int *__restrict__ ecol,
                                         const T *__restrict__ evl, T alpha,
                                         const T *__restrict__ x, T beta, T *__restrict__ y,
                                         ck::CgDev<T> *cg, T *__restrict__ partials) {
    const int64_t b = ck::xcd_block(G);
    if (b < 0)
        return;
    const int64_t groups = ((int64_t)n + 255) / 256;
    T mine = 0;
    for (int64_t g = b; g < groups; g += G) {
        const int64_t row = g * 256 + threadIdx.x;
        if (row < n) {
            // four slots per step: their column and value loads, then their x
            // gathers, are each in flight together.  Padding (column -1) only
            // trails a row, so masking it equals stopping at the first one;
            // x[0] stands in for a masked gather (K > 0 implies ncols > 0).
            constexpr int S = 4;
            T sum = 0;
            for (int s0 = 0; s0 < K; s0 += S) {
                int c[S];
                T v[S], xv[S];
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    const int64_t s = min(s0 + u, K - 1);
                    c[u] = s0 + u < K ? ld_stream(&ecol[s * pitch + row]) : -1;
                    v[u] = ld_stream(&evl[s * pitch + row]);
                }
#pragma unroll
                for (int u = 0; u < S; ++u)
                    xv[u] = x[c[u] >= 0 ? c[u] : 0];
#pragma unroll
                for (int u = 0; u < S; ++u)
                    if (c[u] >= 0)
                        sum += v[u] * xv[u];
                if (c[S - 1] < 0)
                    break;
            }
            T out = alpha * sum;
            if (BETA)
                out += beta * y[row];
            y[row] = out;
            if (DOT)
                mine += out * x[row];
        }
    }
    cg_sigma_epilogue<T, DOT>(mine, cg, partials, b, G);
}

template <typename T, bool BETA, bool DOT>
__global__ __launch_bounds__(256) void spmv_ell(int n, int64_t G, int K, int64_t pitch,
                                                const int *__restrict__ ecol,
                                                const T *__restrict__ evl, T alpha,
                                                const T *__restrict__ x, T beta,
                                                T *__restrict__ y, const int *__restrict__ skip,
                                                ck::CgDev<T> *cg, T *__restrict__ partials) {
    if (skipped(skip))
        return;
    ell_rows<T, BETA, DOT>(n, G, K, pitch, ecol, evl, alpha, x, beta, y, cg, partials);
}

// The ELL part of a HYB product (its own symbol, so profiles tell it apart).
template <typename T, bool BETA>
__global__ __launch_bounds__(256) void spmv_hyb_ell(int n, int64_t G, int K, int64_t pitch,
                                                    const int *__restrict__ ecol,
                                                    const T *__restrict__ evl, T alpha,
                                                    const T *__restrict__ x, T beta,
                                                    T *__restrict__ y,
                                                    const int *__restrict__ skip) {
    if (skipped(skip))
        return;
    ell_rows<T, BETA, false>(n, G, K, pitch, ecol, evl, alpha, x, beta, y, nullptr, nullptr);
}

// Sum of the partials of the run of equal s_crow ending at thread p (s_cval
// holds each wave's segmented scan): its wave's part, then the runs ending
// each earlier wave while the run goes on.
template <typename T>
__device__ __forceinline__ T carry_run(const int *s_crow, const T *s_cval, int p) {
    const int key = s_crow[p];
    T tot = s_cval[p];
    for (int u = (p >> 6) - 1; u >= 0; --u) {
        if (s_crow[64 * u + 63] != key)
            break;
        tot += s_cval[64 * u + 63];
        if (s_crow[64 * u] != key)
            break;
    }
    return tot;
}

// ---- carry completion of COO -------------------------------------------------
// Every thread passes the row it ended inside (crow, -1 if none) with its
// partial (cval), and the first row it completed (frow, -1 if none) with its
// own part of that row (fval).  Across the workgroup, equal crow values form
// one contiguous run of threads (rows only grow with the thread index).  The
// first completed row of a thread started in the run just before it: add
// that run's partials.  Thread 0 then records the block's own carry-out (the
// run ending at the last active thread) for carry_fixup.  The run sums come
// from a segmented scan: within each wave by DPP moves, then across the four
// waves through LDS, so a row spanning the whole workgroup costs a few steps
// instead of one LDS round trip per thread.
template <typename T, bool BETA>
__device__ __forceinline__ void finish_carries(int *s_crow, T *s_cval, int crow, T cval,
                                               int frow, T fval, int last_active, int64_t b,
                                               T alpha, T beta, T *__restrict__ y,
                                               int *__restrict__ crow_g,
                                               T *__restrict__ cval_g) {
    const int tid = threadIdx.x;
    s_crow[tid] = crow;
    s_cval[tid] = ck::wave_seg_scan(cval, crow);
    __syncthreads();
    if (frow >= 0) {
        T tot = tid > 0 && s_crow[tid - 1] == frow
                    ? carry_run(s_crow, s_cval, tid - 1)
                    : T(0);
        tot += fval;
        T out = alpha * tot;
        if (BETA)
            out += beta * y[frow];
        y[frow] = out;
    }
    if (tid == 0) {
        const int R = last_active >= 0 ? s_crow[last_active] : -1;
        crow_g[b] = R;
        cval_g[b] = R >= 0 ? carry_run(s_crow, s_cval, last_active) : T(0);
    }
}

// Merge-path coordinates (row ends, entries) where workgroup q starts.  The
// nominal start is merged item kMergeSpan q; when the row it falls into has
// at most kMergeSlack entries before it, the workgroup starts at that row
// instead, so a matrix with no row longer than kMergeSlack has no row cut by
// a workgroup boundary and needs no carry_fixup.  A workgroup covers at most
// kMergeSpan + kMergeSlack = 256 kMergeIPT items.
__device__ __forceinline__ int2 merge_start(int n, int nnz, const int *__restrict__ rp,
                                            int64_t q) {
    const int64_t d = min<int64_t>(q * kMergeSpan, (int64_t)n + nnz);
    int lo = (int)max<int64_t>(0, d - nnz), hi = (int)min<int64_t>(d, n);
    while (lo < hi) {   // row ends among the first d items
        const int mid = (lo + hi) >> 1;
        if ((int64_t)rp[mid + 1] <= d - mid - 1)
            lo = mid + 1;
        else
            hi = mid;
    }
    int j = (int)(d - lo);
    if (lo < n && j - rp[lo] <= kMergeSlack)
        j = rp[lo];
    return make_int2(lo, j);
}

// part[q] = the coordinates of workgroup q = 0 .. G (G: the end).
__global__ __launch_bounds__(256) void merge_partition(int n, int nnz, int64_t G,
                                                       const int *__restrict__ rp,
                                                       int2 *__restrict__ part) {
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q <= G)
        part[q] = merge_start(n, nnz, rp, q);
}

// The merged sequence as one bit per item, 1 = row end: byte t of workgroup
// q holds thread t's items D0 + 8 t .. D0 + 8 t + 7, items past the
// workgroup's end 0.
__global__ __launch_bounds__(256) void merge_bits(int64_t G, const int *__restrict__ rp,
                                                  const int2 *__restrict__ part,
                                                  unsigned *__restrict__ bits) {
    static_assert(kMergeIPT == 8, "one byte of row-end bits per thread");
    __shared__ unsigned w[64];
    for (int64_t q = blockIdx.x; q < G; q += gridDim.x) {
        if (threadIdx.x < 64)
            w[threadIdx.x] = 0;
        __syncthreads();
        const int2 c0 = part[q], c1 = part[q + 1];
        for (int r = c0.x + threadIdx.x; r < c1.x; r += 256) {
            const int at = rp[r + 1] - c0.y + (r - c0.x);
            atomicOr(&w[at >> 5], 1u << (at & 31));
        }
        __syncthreads();
        if (threadIdx.x < 64)
            bits[64 * q + threadIdx.x] = w[threadIdx.x];
    }
}

// LDS slot of staged product e: one slot of padding per eight, so the threads
// of a wave, whose reads are about eight slots apart, use different banks.
__device__ __forceinline__ int pad8(int e) { return e + (e >> 3); }

// The products of the workgroup's entries j0 .. j0 + nents - 1 into LDS
// (coalesced loads, eight gathers per thread in flight), zeros after them.
template <typename T>
__device__ __forceinline__ void stage_products(int j0, int nents, const int *__restrict__ col,
                                               const T *__restrict__ val,
                                               const T *__restrict__ x, T *s_prod) {
    const int tid = threadIdx.x;
    int cc[kMergeIPT];
    T vv[kMergeIPT], xv[kMergeIPT];
    if (nents > 0) {
        const int *colb = col + j0;
        const T *valb = val + j0;
#pragma unroll
        for (int u = 0; u < kMergeIPT; ++u) {
            const int t = min(u * 256 + tid, nents - 1);
            cc[u] = ld_stream(&colb[t]);
            vv[u] = ld_stream(&valb[t]);
        }
#pragma unroll
        for (int u = 0; u < kMergeIPT; ++u)
            xv[u] = x[cc[u]];
        __builtin_amdgcn_sched_barrier(0);   // all gathers in flight before the first use
    }
#pragma unroll
    for (int u = 0; u < kMergeIPT; ++u) {
        const int t = u * 256 + tid;
        s_prod[pad8(t)] = t < nents ? vv[u] * xv[u] : T(0);
    }
}

// Merge-path CSR.  Workgroup b owns at most 2048 merged items: the merge of
// the row ends rp[1..n] with the entries 0..nnz-1 between the coordinates of
// merge_start.  It stages the products of its entries in LDS; every thread
// then sums its eight items: entries add to the running row, row ends close
// it.  Which items are row ends comes from the matrix's plan (part and bits,
// built by the conversion), so a thread needs no search and no row pointers,
// its eight products are read together, and its place in the rows is a
// prefix sum of bit counts; without a plan (a product before any conversion)
// two threads search the workgroup's coordinates and the bits are made in LDS
// from the row pointers: the same items per thread, and so the same result.
// Rows cut by thread boundaries are completed in LDS, rows cut by workgroup
// boundaries by carry_fixup; the finished rows leave LDS in row order.
//
// Bound by the L2 requests of the x gathers (one line each, about 190 G/s).
// Searching and walking the merged items in LDS, eight slots apart without
// padding (16-way bank conflicts), and a carry_fixup per product cost on top
// of them; whole products before -> now: FP32 uniform rows, n = 180K (all of
// x in every L2): 40.7 -> 34.6 us; CSR-panel, uniform rows, n = 2M: 486 ->
// 410 us; CSR-panel, power-law rows, n = 1.2M: 229 -> 205 us.
template <typename T, bool BETA, bool PLAN>
__device__ __forceinline__ void merge_rows(int n, int nnz, int64_t G, const int *__restrict__ rp,
                                           const int *__restrict__ col,
                                           const T *__restrict__ val, T alpha,
                                           const T *__restrict__ x, T beta, T *__restrict__ y,
                                           int *__restrict__ crow_g, T *__restrict__ cval_g,
                                           const int2 *__restrict__ part,
                                           const unsigned char *__restrict__ bits) {
    constexpr int ITEMS = 256 * kMergeIPT;
    __shared__ int s_crow[256];
    __shared__ T s_cval[256];
    __shared__ T s_prod[ITEMS + ITEMS / 8];   // the products, then the row sums
    __shared__ unsigned s_bits[PLAN ? 1 : 64];
    __shared__ int s_wave[4];
    __shared__ int2 s_coord[2];
    const int64_t b = ck::xcd_block(G);
    if (b < 0)
        return;
    const int tid = threadIdx.x;
    int2 c0, c1;
    unsigned mask = 0;   // this thread's row ends
    if constexpr (PLAN) {
        c0 = part[b];
        c1 = part[b + 1];
        mask = bits[b * 256 + tid];
    } else {
        if (tid < 2)
            s_coord[tid] = merge_start(n, nnz, rp, b + tid);
        if (tid < 64)
            s_bits[tid] = 0;
        __syncthreads();
        c0 = s_coord[0];
        c1 = s_coord[1];
    }
    const int i0 = c0.x, nends = c1.x - c0.x, nents = c1.y - c0.y;
    const int items = nends + nents;
    if constexpr (!PLAN)   // as merge_bits
        for (int t = tid; t < nends; t += 256) {
            const int at = rp[i0 + t + 1] - c0.y + t;
            atomicOr(&s_bits[at >> 5], 1u << (at & 31));
        }
    stage_products<T>(c0.y, nents, col, val, x, s_prod);
    if constexpr (!PLAN) {
        __syncthreads();
        mask = ((const unsigned char *)s_bits)[tid];
    }
    const int dl = tid * kMergeIPT;   // this thread's first item
    const int pc = __popc(mask);
    const int sc = ck::wave_scan(pc);
    if ((tid & 63) == 63)
        s_wave[tid >> 6] = sc;
    __syncthreads();
    int a = sc - pc;                  // row ends before it
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int w = 0; w < 3; ++w)
        a += w < wave ? s_wave[w] : 0;
    T v[kMergeIPT];   // item d: its product, or the sum of the row it ends
#pragma unroll
    for (int d = 0; d < kMergeIPT; ++d) {
        const int e = dl - a + d - __popc(mask & ((1u << d) - 1));
        v[d] = s_prod[pad8(e)];   // e < 2048: items are in order
    }
    T acc = 0;
#pragma unroll
    for (int d = 0; d < kMergeIPT; ++d) {
        if (mask & (1u << d)) {
            v[d] = acc;
            acc = 0;
        } else {
            acc += v[d];
        }
    }
    const int after = a + __popc(mask);   // the row this thread ends in
    const int crow = dl < items && i0 + after < n ? i0 + after : -1;
    s_crow[tid] = crow;
    s_cval[tid] = ck::wave_seg_scan(acc, crow);
    __syncthreads();   // also: every product has been read
    bool first = true;
    int r = a;
#pragma unroll
    for (int d = 0; d < kMergeIPT; ++d)
        if (mask & (1u << d)) {
            if (first && tid > 0 && s_crow[tid - 1] == i0 + a)
                v[d] = carry_run(s_crow, s_cval, tid - 1) + v[d];
            s_prod[r++] = v[d];
            first = false;
        }
    if (tid == 0) {   // the row the workgroup ends in
        const int last = (items + kMergeIPT - 1) / kMergeIPT - 1;
        const int R = last >= 0 ? s_crow[last] : -1;
        crow_g[b] = R;
        cval_g[b] = R >= 0 ? carry_run(s_crow, s_cval, last) : T(0);
    }
    __syncthreads();
    for (int t = tid; t < nends; t += 256) {
        T out = alpha * s_prod[t];
        if (BETA)
            out += beta * y[i0 + t];
        y[i0 + t] = out;
    }
}

template <typename T, bool BETA, bool PLAN>
__global__ __launch_bounds__(256) void spmv_merge(int n, int nnz, int64_t G,
                                                  const int *__restrict__ rp,
                                                  const int *__restrict__ col,
                                                  const T *__restrict__ val, T alpha,
                                                  const T *__restrict__ x, T beta,
                                                  T *__restrict__ y, int *__restrict__ crow_g,
                                                  T *__restrict__ cval_g,
                                                  const int2 *__restrict__ part,
                                                  const unsigned char *__restrict__ bits,
                                                  const int *__restrict__ skip) {
    if (skipped(skip))
        return;
    merge_rows<T, BETA, PLAN>(n, nnz, G, rp, col, val, alpha, x, beta, y, crow_g, cval_g, part,
                              bits);
}

// CSR-panel products: the merge path over the panel-major arrays read as one
// CSR of P*n rows, into the partial vectors (its own symbol, so profiles tell
// it apart from CSR-merge).
template <typename T>
__global__ __launch_bounds__(256) void spmv_panel_merge(int rows, int nnz, int64_t G,
                                                        const int *__restrict__ pcol,
                                                        const T *__restrict__ pval,
                                                        const T *__restrict__ x,
                                                        T *__restrict__ ypart,
                                                        int *__restrict__ crow_g,
                                                        T *__restrict__ cval_g,
                                                        const int2 *__restrict__ part,
                                                        const unsigned char *__restrict__ bits,
                                                        const int *__restrict__ skip) {
    if (skipped(skip))
        return;
    merge_rows<T, false, true>(rows, nnz, G, nullptr, pcol, pval, T(1), x, T(0), ypart, crow_g,
                               cval_g, part, bits);
}

template <typename T, bool BETA>
__global__ __launch_bounds__(256) void spmv_coo(int n, int nnz, int64_t G,
                                                const int *__restrict__ row,
                                                const int *__restrict__ col,
                                                const T *__restrict__ val, T alpha,
                                                const T *__restrict__ x, T beta,
                                                T *__restrict__ y, int *__restrict__ crow_g,
                                                T *__restrict__ cval_g,
                                                const int *__restrict__ skip) {
    constexpr int ITEMS = 256 * kCooIPT;
    __shared__ int s_crow[256];
    __shared__ T s_cval[256];
    __shared__ int s_row[ITEMS + 1];   // row of entries K0 .. K0+cnt (the last: next row or n)
    __shared__ T s_prod[ITEMS];
    if (skipped(skip))
        return;
    const int64_t b = ck::xcd_block(G);
    if (b < 0)
        return;
    const int tid = threadIdx.x;
    // stage this workgroup's entries: rows and products, coalesced, with the
    // eight gathers of a thread in flight together
    const int64_t K0 = b * ITEMS;
    const int cnt = (int)min<int64_t>(ITEMS, nnz - K0);
    {
        int cc[kCooIPT];
        T vv[kCooIPT], xv[kCooIPT];
#pragma unroll
        for (int u = 0; u < kCooIPT; ++u) {
            const int t = min(u * 256 + tid, cnt - 1);
            cc[u] = ld_stream(&col[K0 + t]);
            vv[u] = ld_stream(&val[K0 + t]);
        }
#pragma unroll
        for (int u = 0; u < kCooIPT; ++u)
            xv[u] = x[cc[u]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kCooIPT; ++u)
            if (u * 256 + tid < cnt)
                s_prod[u * 256 + tid] = vv[u] * xv[u];
    }
    for (int t = tid; t <= cnt; t += 256)
        s_row[t] = K0 + t < nnz ? ld_stream(&row[K0 + t]) : n;
    __syncthreads();
    const int k0 = tid * kCooIPT;   // this thread's first local entry
    int crow = -1, frow = -1;
    T cval = 0, fval = 0;
    if (k0 < cnt) {
        const int k1 = min(k0 + kCooIPT, cnt);
        if (K0 + k0 == 0) {   // rows before the first stored entry are empty
            const int r_first = s_row[0];
            for (int r = 0; r < r_first; ++r)
                y[r] = BETA ? beta * y[r] : T(0);
        }
        int cur = s_row[k0];
        T acc = 0;
        bool first = true;
        for (int k = k0; k < k1; ++k) {
            acc += s_prod[k];
            const int nxt = s_row[k + 1];
            if (nxt != cur) {
                if (first) {
                    frow = cur;
                    fval = acc;
                    first = false;
                } else {
                    T out = alpha * acc;
                    if (BETA)
                        out += beta * y[cur];
                    y[cur] = out;
                }
                for (int r = cur + 1; r < nxt; ++r)   // empty rows in the gap
                    y[r] = BETA ? beta * y[r] : T(0);
                acc = 0;
                cur = nxt;
            }
        }
        if (s_row[k1] == s_row[k1 - 1]) {   // the thread ends inside a row
            crow = s_row[k1 - 1];
            cval = acc;
        }
    }
    const int64_t first_k = b * 256 * kCooIPT;
    const int last_active = (int)min<int64_t>(255, (nnz - first_k + kCooIPT - 1) / kCooIPT - 1);
    finish_carries<T, BETA>(s_crow, s_cval, crow, cval, frow, fval, last_active, b, alpha, beta,
                            y, crow_g, cval_g);
}

// Rows cut by a workgroup boundary: each run of equal carry rows is summed in
// block order by the run's first entry and added once.  The carries are read
// eight at a time (loads issued together, indexes clamped to the array), so a
// row spanning many workgroups does not wait one load latency per workgroup.
template <typename T>
__global__ __launch_bounds__(256) void carry_fixup(int64_t G, const int *__restrict__ crow,
                                                   const T *__restrict__ cval, T alpha,
                                                   T *__restrict__ y,
                                                   const int *__restrict__ skip) {
    if (skipped(skip))
        return;
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= G)
        return;
    const int R = crow[b];
    if (R < 0 || (b > 0 && crow[b - 1] == R))
        return;
    T tot = 0;
    for (int64_t e0 = b; e0 < G; e0 += 8) {
        int r[8];
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t e = min<int64_t>(e0 + u, G - 1);
            r[u] = crow[e];
            v[u] = cval[e];
        }
        bool more = true;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            more = more && e0 + u < G && r[u] == R;
            if (more)
                tot += v[u];
        }
        if (!more)
            break;
    }
    y[R] += alpha * tot;
}

template <typename T, bool BETA>
__global__ __launch_bounds__(256) void scale_rows(int64_t n, T beta, T *__restrict__ y,
                                                  const int *__restrict__ skip) {
    if (skipped(skip))
        return;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        y[i] = BETA ? beta * y[i] : T(0);
}

// ---------------------------------------------------------------------------
namespace ck {

bool config_valid(const ck_config &c) {
    if (c.format == CK_FMT_ELL || c.format == CK_FMT_COO || c.format == CK_FMT_DIA ||
        c.format == CK_FMT_HYB)
        return true;
    if (c.format != CK_FMT_CSR)
        return false;
    if (c.algorithm == CK_ALG_SCALAR || c.algorithm == CK_ALG_MERGE ||
        c.algorithm == CK_ALG_PANEL)
        return true;
    if (c.algorithm != CK_ALG_VECTOR)
        return false;
    return c.lanes >= 1 && c.lanes <= 64 && (c.lanes & (c.lanes - 1)) == 0;
}

bool spmv_fuses_dot(const ck_config &c) {
    return c.format == CK_FMT_ELL || c.format == CK_FMT_DIA ||
           (c.format == CK_FMT_CSR && (c.algorithm == CK_ALG_VECTOR ||
                                       c.algorithm == CK_ALG_SCALAR ||
                                       c.algorithm == CK_ALG_PANEL));
}

static int64_t row_groups(const ck_matrix &M, const ck_config &c) {
    if (c.format == CK_FMT_CSR && c.algorithm == CK_ALG_VECTOR)
        return ceil_div(M.n, 256 / c.lanes);
    return ceil_div(M.n, 256);
}

int64_t spmv_dot_blocks(const ck_matrix &M, const ck_config &c) {
    if (!spmv_fuses_dot(c))
        return 0;
    const int64_t g = std::max<int64_t>(row_groups(M, c), 1);
    if (c.format == CK_FMT_DIA)
        return dia_blocks(M, g);
    return std::min<int64_t>(g, c.algorithm == CK_ALG_PANEL && c.format == CK_FMT_CSR
                                    ? kFoldPartials : kMaxPartials);
}

static int64_t carry_blocks(const ck_matrix &M, const ck_config &c) {
    if (c.format == CK_FMT_COO)
        return ceil_div(M.nnz, 256 * kCooIPT);
    if (c.format == CK_FMT_CSR && c.algorithm == CK_ALG_MERGE)
        return ceil_div(M.n + M.nnz, kMergeSpan);
    return 0;
}

// Carries of G workgroups, each array at a multiple of 256 bytes.
static int64_t carry_array_bytes(int64_t G, bool fp32) {
    return ((G * (int64_t)sizeof(int) + 255) / 256) * 256 + G * (fp32 ? 4 : 8) + 256;
}

// CSR-panel: per-panel partial sums, then (merge-path panels) the carries of the
// merge over the panel rows in workgroups of `items`; sized for the dense P*n
// layout (an upper bound: the row-list layout has fewer rows, and the size is
// also needed before the conversion decides).
static int64_t panel_work_bytes(const ck_matrix &M, int64_t items, bool fp32) {
    const int64_t rows = (int64_t)panel_count_for(M.ncols, 8) * M.n;
    return ((rows * (fp32 ? 4 : 8) + 255) / 256) * 256 +
           carry_array_bytes(ceil_div(rows + M.nnz, items), fp32);
}

// The same for slices of x, if M takes them: at most 64 MiB.
static int64_t slices_work_bytes_of(const ck_matrix &M, bool fp32) {
    return slices_work_bytes(M.n, slices_of(M.n, M.ncols, M.nnz, M.max_row, M.span), fp32);
}

int64_t spmv_carry_bytes(const ck_matrix &M, const ck_config &c, bool fp32) {
    if (c.format == CK_FMT_CSR && c.algorithm == CK_ALG_PANEL)
        return std::max(panel_work_bytes(M, kMergeSpan, fp32), slices_work_bytes_of(M, fp32));
    return carry_array_bytes(carry_blocks(M, c), fp32);
}

int64_t spmv_noalloc_bytes(const ck_matrix &M, const ck_config &c) {
    if (c.format == CK_FMT_CSR && c.algorithm == CK_ALG_PANEL)
        return std::max(panel_work_bytes(M, 256 * kMergeIPT, false),
                        slices_work_bytes_of(M, false));
    return spmv_carry_bytes(M, c, false);
}

// ---- merge-path plan: G + 1 coordinate pairs and 64 words of row-end bits per
// workgroup ---------------------------------------------------------------------
static int64_t plan_blocks(int64_t rows, int64_t nnz) { return ceil_div(rows + nnz, kMergeSpan); }

int64_t merge_plan_ints(int64_t rows, int64_t nnz) {
    const int64_t G = plan_blocks(rows, nnz);
    return 2 * (G + 1) + 64 * G;
}

static const unsigned char *plan_bits(const int32_t *plan, int64_t G) {
    return (const unsigned char *)(plan + 2 * (G + 1));
}

ck_status launch_merge_plan(int64_t rows, int64_t nnz, const int32_t *rp, int32_t *plan,
                            hipStream_t s) {
    const int64_t G = plan_blocks(rows, nnz);
    int2 *part = (int2 *)plan;
    hipLaunchKernelGGL(merge_partition, dim3(ceil_div(G + 1, 256)), dim3(256), 0, s, (int)rows,
                       (int)nnz, G, rp, part);
    if (G > 0)
        hipLaunchKernelGGL(merge_bits, dim3(std::min<int64_t>(G, 4096)), dim3(256), 0, s, G, rp,
                           part, (unsigned *)(plan + 2 * (G + 1)));
    CK_HIP(hipGetLastError());
    return CK_OK;
}

bool merge_cuts_rows(int64_t max_row) { return max_row < 0 || max_row > kMergeSlack; }

ck_config default_config(int64_t n, int64_t nnz) {
    const int64_t mean = n > 0 ? nnz / n : 0;   // floor(nnz/n) has the same floor(log2)
    int L = 1;
    while ((int64_t)L * 2 <= mean && L < 64)
        L *= 2;
    if (L < 2)
        L = 2;
    return ck_config{CK_FMT_CSR, CK_ALG_VECTOR, L, 0};
}

const char *kernel_name(const ck_config &c, bool fp32) {
    static const char *vec64[7] = {
        "spmv_csr_vector<1, double, false, false>", "spmv_csr_vector<2, double, false, false>",
        "spmv_csr_vector<4, double, false, false>", "spmv_csr_vector<8, double, false, false>",
        "spmv_csr_vector<16, double, false, false>", "spmv_csr_vector<32, double, false, false>",
        "spmv_csr_vector<64, double, false, false>"};
    static const char *vec32[7] = {
        "spmv_csr_vector<1, float, false, false>", "spmv_csr_vector<2, float, false, false>",
        "spmv_csr_vector<4, float, false, false>", "spmv_csr_vector<8, float, false, false>",
        "spmv_csr_vector<16, float, false, false>", "spmv_csr_vector<32, float, false, false>",
        "spmv_csr_vector<64, float, false, false>"};
    if (c.format == CK_FMT_ELL)
        return fp32 ? "spmv_ell<float, false, false>" : "spmv_ell<double, false, false>";
    if (c.format == CK_FMT_DIA)
        return fp32 ? "spmv_dia<float, false, false, ND>" : "spmv_dia<double, false, false, ND>";
    if (c.format == CK_FMT_HYB)
        return fp32 ? "spmv_hyb_ell<float, false>" : "spmv_hyb_ell<double, false>";
    if (c.format == CK_FMT_COO)
        return fp32 ? "spmv_coo<float, false>" : "spmv_coo<double, false>";
    if (c.algorithm == CK_ALG_SCALAR)
        return fp32 ? "spmv_csr_scalar<float, false, false>" : "spmv_csr_scalar<double, false, false>";
    if (c.algorithm == CK_ALG_MERGE)
        return fp32 ? "spmv_merge<float, false, true>" : "spmv_merge<double, false, true>";
    if (c.algorithm == CK_ALG_PANEL)
        return fp32 ? "spmv_panel_merge<float>" : "spmv_panel_merge<double>";
    int idx = 0;
    while ((1 << idx) < c.lanes)
        ++idx;
    return fp32 ? vec32[idx] : vec64[idx];
}

template <typename T>
static const T *values(const ck_matrix &M) {
    if constexpr (sizeof(T) == 4)
        return M.val32;
    else
        return M.val;
}

template <typename T>
static const T *ell_values(const ck_matrix &M) {
    if constexpr (sizeof(T) == 4)
        return M.ell_val32;
    else
        return M.ell_val;
}

template <typename T>
static const T *dia_values(const ck_matrix &M) {
    if constexpr (sizeof(T) == 4)
        return M.dia_val32;
    else
        return M.dia_val;
}

template <typename T>
static const T *hyb_values(const ck_matrix &M) {
    if constexpr (sizeof(T) == 4)
        return M.hyb_val32;
    else
        return M.hyb_val;
}

template <int L, typename T, bool BETA, bool DOT>
static void go_vector(const ck_matrix &M, int64_t G, const SpmvArgs<T> &a, hipStream_t s) {
    hipLaunchKernelGGL((spmv_csr_vector<L, T, BETA, DOT>), dim3(xcd_grid(G)), dim3(256), 0, s,
                       (int)M.n, G, M.rp, M.col, values<T>(M), a.alpha, a.x, a.beta, a.y, a.skip,
                       a.cg, a.dot_partials);
}

template <typename T, bool BETA, bool DOT>
static ck_status dispatch_rows(const ck_matrix &M, const ck_config &c, const SpmvArgs<T> &a,
                               hipStream_t s) {
    const int64_t G = std::min<int64_t>(std::max<int64_t>(row_groups(M, c), 1), kRowBlocks);
    if (c.format == CK_FMT_DIA) {
        launch_dia_spmv<T, BETA, DOT>(M, dia_blocks(M, row_groups(M, c)), dia_values<T>(M), a, s);
        return CK_OK;
    }
    if (c.format == CK_FMT_HYB) {   // ELL part for every row, then the long rows' remainder
        if constexpr (DOT)
            return fail(CK_E_INVALID, "HYB does not fuse the CG dot product");
        hipLaunchKernelGGL((spmv_hyb_ell<T, BETA>), dim3(xcd_grid(G)), dim3(256), 0, s,
                           (int)M.n, G, (int)M.hyb_K, M.hyb_pitch, M.hyb_col, hyb_values<T>(M),
                           a.alpha, a.x, a.beta, a.y, a.skip);
        launch_hyb_tail<T>(M, values<T>(M), a, s);
        return CK_OK;
    }
    if (c.format == CK_FMT_ELL) {
        hipLaunchKernelGGL((spmv_ell<T, BETA, DOT>), dim3(xcd_grid(G)), dim3(256), 0, s,
                           (int)M.n, G, (int)M.ell_K, M.ell_pitch, M.ell_col, ell_values<T>(M),
                           a.alpha, a.x, a.beta, a.y, a.skip, a.cg, a.dot_partials);
        return CK_OK;
    }
    if (c.algorithm == CK_ALG_SCALAR) {
        hipLaunchKernelGGL((spmv_csr_scalar<T, BETA, DOT>), dim3(xcd_grid(G)), dim3(256), 0, s,
                           (int)M.n, G, M.rp, M.col, values<T>(M), a.alpha, a.x, a.beta, a.y,
                           a.skip, a.cg, a.dot_partials);
        return CK_OK;
    }
    switch (c.lanes) {
    case 1: go_vector<1, T, BETA, DOT>(M, G, a, s); break;
    case 2: go_vector<2, T, BETA, DOT>(M, G, a, s); break;
    case 4: go_vector<4, T, BETA, DOT>(M, G, a, s); break;
    case 8: go_vector<8, T, BETA, DOT>(M, G, a, s); break;
    case 16: go_vector<16, T, BETA, DOT>(M, G, a, s); break;
    case 32: go_vector<32, T, BETA, DOT>(M, G, a, s); break;
    case 64: go_vector<64, T, BETA, DOT>(M, G, a, s); break;
    default: return fail(CK_E_INVALID, "lanes must be a power of two in [1, 64]");
    }
    return CK_OK;
}

template <typename T, bool BETA>
static ck_status dispatch_carry(const ck_matrix &M, const ck_config &c, const SpmvArgs<T> &a,
                                hipStream_t s) {
    const int64_t G = carry_blocks(M, c);
    void *ws = a.carry;
    bool own = false;
    if (ws == nullptr) {
        CK_HIP(hipMallocAsync(&ws, (size_t)spmv_carry_bytes(M, c, sizeof(T) == 4), s));
        own = true;
    }
    int *crow = (int *)ws;
    T *cval = (T *)((char *)ws + ((G * (int64_t)sizeof(int) + 255) / 256) * 256);
    bool cut = true;   // rows may be cut by a workgroup boundary
    if (c.format == CK_FMT_COO) {
        hipLaunchKernelGGL((spmv_coo<T, BETA>), dim3(xcd_grid(G)), dim3(256), 0, s, (int)M.n,
                           (int)M.nnz, G, M.coo_row, M.col, values<T>(M), a.alpha, a.x, a.beta,
                           a.y, crow, cval, a.skip);
    } else if (M.has_merge_plan.load()) {
        cut = M.merge_cut;
        hipLaunchKernelGGL((spmv_merge<T, BETA, true>), dim3(xcd_grid(G)), dim3(256), 0, s,
                           (int)M.n, (int)M.nnz, G, M.rp, M.col, values<T>(M), a.alpha, a.x,
                           a.beta, a.y, crow, cval, (const int2 *)M.merge_plan,
                           plan_bits(M.merge_plan, G), a.skip);
    } else {
        hipLaunchKernelGGL((spmv_merge<T, BETA, false>), dim3(xcd_grid(G)), dim3(256), 0, s,
                           (int)M.n, (int)M.nnz, G, M.rp, M.col, values<T>(M), a.alpha, a.x,
                           a.beta, a.y, crow, cval, nullptr, nullptr, a.skip);
    }
    if (cut)
        hipLaunchKernelGGL((carry_fixup<T>), dim3(ceil_div(G, 256)), dim3(256), 0, s, G, crow,
                           cval, a.alpha, a.y, a.skip);
    if (own)
        CK_HIP(hipFreeAsync(ws, s));
    return CK_OK;
}

// CSR-panel: the panel-major arrays are one CSR of P*n rows (panel p's row i
// is row p*n + i), whose merge-path product writes the P partial vectors;
// panel_combine then sums them in panel order.  Logical block ranges are
// contiguous per XCD and a panel's rows are contiguous in the merged
// sequence, so each XCD works through its own consecutive panels and their x
// slices stay in its L2, while the merge balances hub rows.  (One to four
// lanes per panel row instead measured 1.3-2.7x slower: the short panel rows
// left the loads of a wave mostly idle and hub rows serialised.)
template <typename T>
static ck_status panel_merge_spmv(const ck_matrix &M, const SpmvArgs<T> &a, void *ws,
                                  int64_t G_dot, hipStream_t s) {
    const T *pv;
    if constexpr (sizeof(T) == 4)
        pv = M.panel_val32;
    else
        pv = M.panel_val;
    const int64_t rows = M.panel_rows;   // P*n, or the non-empty panel rows
    const int64_t Gt = plan_blocks(rows, M.nnz);
    T *ypart = (T *)ws;
    int *crow = (int *)((char *)ws + ((rows * (int64_t)sizeof(T) + 255) / 256) * 256);
    T *cval = (T *)((char *)crow + ((Gt * (int64_t)sizeof(int) + 255) / 256) * 256);
    if (Gt > 0) {   // no panel rows at all (no entries, row-list layout): combine only
        hipLaunchKernelGGL((spmv_panel_merge<T>), dim3(xcd_grid(Gt)), dim3(256), 0, s, (int)rows,
                           (int)M.nnz, Gt, M.panel_col, pv, a.x, ypart, crow, cval,
                           (const int2 *)M.panel_plan, plan_bits(M.panel_plan, Gt), a.skip);
        if (M.panel_cut)
            hipLaunchKernelGGL((carry_fixup<T>), dim3(ceil_div(Gt, 256)), dim3(256), 0, s, Gt,
                               crow, cval, T(1), ypart, a.skip);
    }
    CK_HIP(hipGetLastError());
    return launch_panel_combine<T>(M, a, ypart, G_dot, s);
}

template <typename T>
ck_status launch_spmv(const ck_matrix &M, const ck_config &c, const SpmvArgs<T> &a,
                      hipStream_t s) {
    if (!config_valid(c))
        return fail(CK_E_INVALID, "invalid SpMV configuration");
    if constexpr (sizeof(T) == 4) {
        if (!M.val32)
            return fail(CK_E_INVALID, "FP32 product needs a handle created with CK_KEEP_FP32");
    }
    if (c.format == CK_FMT_ELL && !M.has_ell.load())
        return fail(CK_E_INVALID, "ELL requested but the matrix has not been converted");
    if (c.format == CK_FMT_COO && !M.has_coo.load())
        return fail(CK_E_INVALID, "COO requested but the matrix has not been converted");
    if (c.format == CK_FMT_DIA && !M.has_dia.load())
        return fail(CK_E_INVALID, "DIA requested but the matrix has not been converted");
    if (c.format == CK_FMT_HYB && !M.has_hyb.load())
        return fail(CK_E_INVALID, "HYB requested but the matrix has not been converted");
    const bool panel = c.format == CK_FMT_CSR && c.algorithm == CK_ALG_PANEL;
    if (panel && !M.has_panel.load())
        return fail(CK_E_INVALID, "CSR-panel requested but the matrix has not been converted");
    const bool beta = a.beta != T(0);
    const bool dot = a.cg != nullptr;
    if (dot && (!spmv_fuses_dot(c) || a.dot_partials == nullptr))
        return fail(CK_E_INVALID, "this configuration does not fuse the CG dot product");
    if (M.n == 0)
        return CK_OK;
    ck_status st;
    if (panel) {
        void *ws = a.carry;
        if (ws == nullptr)
            CK_HIP(hipMallocAsync(&ws, (size_t)spmv_carry_bytes(M, c, sizeof(T) == 4), s));
        st = M.slice_val != nullptr ? launch_slices<T>(M, a, (T *)ws, spmv_dot_blocks(M, c), s)
                                    : panel_merge_spmv<T>(M, a, ws, spmv_dot_blocks(M, c), s);
        if (a.carry == nullptr)
            CK_HIP(hipFreeAsync(ws, s));
    } else if (M.nnz == 0 && !dot) {
        if (beta)
            hipLaunchKernelGGL((scale_rows<T, true>), dim3(ceil_div(M.n, 256)), dim3(256), 0, s,
                               M.n, a.beta, a.y, a.skip);
        else
            hipLaunchKernelGGL((scale_rows<T, false>), dim3(ceil_div(M.n, 256)), dim3(256), 0, s,
                               M.n, a.beta, a.y, a.skip);
        st = CK_OK;
    } else if (c.format == CK_FMT_COO || (c.format == CK_FMT_CSR && c.algorithm == CK_ALG_MERGE)) {
        st = beta ? dispatch_carry<T, true>(M, c, a, s) : dispatch_carry<T, false>(M, c, a, s);
    } else if (beta) {
        st = dot ? dispatch_rows<T, true, true>(M, c, a, s) : dispatch_rows<T, true, false>(M, c, a, s);
    } else {
        st = dot ? dispatch_rows<T, false, true>(M, c, a, s) : dispatch_rows<T, false, false>(M, c, a, s);
    }
    CK_TRY(st);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

template ck_status launch_spmv<double>(const ck_matrix &, const ck_config &,
                                       const SpmvArgs<double> &, hipStream_t);
template ck_status launch_spmv<float>(const ck_matrix &, const ck_config &,
                                      const SpmvArgs<float> &, hipStream_t);

}  // namespace ck
