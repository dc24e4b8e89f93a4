// CSR-panel products of matrices with even rows scattered over a short x: the
// gathers served from LDS, a slice of x at a time.
//
// A gather moves 64 bytes from L2, whatever the kernel, and the chip moves about 190 G
// of them a second: uniform-random rows of 4-64 entries at n = 180,000 (6.1M entries)
// took 37 us by merge path (FP32 34 us) where their bytes take 13 (9).  LDS gives a
// CU 8 bytes to every lane in a few cycles.  So the entries are stored by slices of x,
// in a slice by rows, with 16-bit columns counted from the slice's first.  A workgroup
// of 16 waves loads one slice and takes every so many'th group of rows in it; its waves
// then run on their own: the lanes take a group's entries in turn, put the products in
// LDS, and each row's lanes add the row's up.  The row sums of the slices (P vectors)
// are added in slice order by a second launch.  One workgroup per CU (two in FP32): the
// slice and the products take most of its LDS.
//
// Measured (before: merge path, the best there was): n = 180,000 36.8 -> 24.6 us, FP32
// 34.1 -> 17.0; n = 100,000 22.1 -> 17.6, FP32 20.6 -> 12.7; n = 300,000 57.8 -> 44.4,
// FP32 53.4 -> 28.7.  The conversion, 11 us of it the panels' count: n = 100,000 66 us,
// 180,000 84, 300,000 120.
// Bounds now: the entries (10 bytes, FP32 6) and the partial sums, written and read,
// 2/3 of it; the rest is the launch of the sum and the first loads' latency.
// Where every workgroup went through all slices instead, so that no partial sums were
// stored, L2 sent 256 copies of x at 12 TB/s: 43 us at n = 180,000.
//
// slices_of() draws the line.  Short rows leave little of a row to a slice: the
// partial sums then outweigh the gathers saved (n = 200,000, rows of 10-18, P = 14:
// 20.0 us by merge path, 23.3; n = 60,000, rows of 20-30, P = 4: 13.0, 12.2).
// Smaller matrices are bound by the two launches (1.0M entries: 9.6 us both ways;
// 1.5M: 13.0, 10.9).  Uneven rows leave workgroups waiting for others (power-law n =
// 100,000: 20.9, 45 us), and rows whose columns lie close together gather from L1.
#include <algorithm>
#include <numeric>
#include <vector>

#include "matrix.hpp"
#include "panel.hpp"
#include "slices.hpp"
#include "solvers.hpp"

namespace {

constexpr int kSliceW = 15360;       // columns per slice at most: 120 KB of FP64
constexpr int kSliceThreads = 1024;
constexpr int kSlicePass = 256;      // products of a wave kept at a time
constexpr int kSliceCUs = 256;
constexpr int kSlices = 32;          // slices at most
constexpr int kConvThreads = 512;
constexpr int64_t kSliceMinNnz = 5 << 18;   // 1.3M
constexpr int kLongSliceRow = 1023;  // 64 rows' entries in a slice are counted in 16 bits

// A workgroup of the conversion takes 64 rows, eight lanes each, `visit(row, k, slice,
// column, value)` being called for each of their entries (value 0 without `val`).
template <typename F>
__device__ __forceinline__ void visit_rows(int n, int W, const int *__restrict__ rp,
                                           const int *__restrict__ col,
                                           const double *__restrict__ val, const F &visit) {
    constexpr int L = kConvThreads / 64, U = 4;
    const int row = threadIdx.x / L, lane = threadIdx.x % L;
    const int i = blockIdx.x * 64 + row;
    const int k0 = i < n ? rp[i] : 0, k1 = i < n ? rp[i + 1] : 0;
    const float inv = 1.0f / (float)W;
    for (int t = k0; t < k1; t += L * U) {
        int c[U];
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = t + u * L + lane;
            c[u] = k < k1 ? col[k] : -1;
            v[u] = val != nullptr && k < k1 ? val[k] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c[u] >= 0) {
                const int s = ck::panel_of(c[u], W, inv);
                visit(row, t + u * L + lane, s, c[u] - s * W, v[u]);
            }
    }
}

// filled[block] = the block's sum of the rows' set bits in `panels`, held by all
// eight lanes of a row together.
__device__ __forceinline__ void store_filled(unsigned panels, int *__restrict__ filled) {
    constexpr int L = kConvThreads / 64;
    __shared__ int part[kConvThreads / 64];
#pragma unroll
    for (int off = 1; off < L; off <<= 1)
        panels |= __shfl_xor(panels, off, L);
    const int sum = ck::wave_sum(threadIdx.x % L == 0 ? __popc(panels) : 0);
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < kConvThreads / 64; ++w)
            t += part[w];
        filled[blockIdx.x] = t;
    }
}

// filled[g] = the rows' panels of group g that hold entries, x cut in eight.
__global__ __launch_bounds__(kConvThreads) void slices_eight(int n, int W8,
                                                    const int *__restrict__ rp,
                                                    const int *__restrict__ col,
                                                    int *__restrict__ filled) {
    unsigned panels = 0;
    visit_rows(n, W8, rp, col, nullptr,
               [&](int, int, int p, int, double) { panels |= 1u << p; });
    store_filled(panels, filled);
}

// ends[s*n + i] = entries in slice s of the rows of i's 64 up to i; total[s*G + g] =
// of all the rows of group g, filled[g] = their panels that hold entries, x cut in
// four (of W4 columns).  Also the zeros that end the entries' arrays.
__global__ __launch_bounds__(kConvThreads) void slices_count(int n, int W4, int P, int W, int G,
                                                    const int *__restrict__ rp,
                                                    const int *__restrict__ col,
                                                    unsigned short *__restrict__ ends,
                                                    int *__restrict__ total,
                                                    int *__restrict__ filled,
                                                    unsigned short *__restrict__ scol_end,
                                                    double *__restrict__ sval_end,
                                                    float *__restrict__ sval32_end) {
    __shared__ int s_cnt[64][kSlices + 1];
    const int lane = threadIdx.x & 63;
    for (int t = threadIdx.x; t < 64 * (kSlices + 1); t += kConvThreads)
        (&s_cnt[0][0])[t] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        filled[G] = 0;
    if (blockIdx.x == 0 && threadIdx.x < kSlicePass) {
        scol_end[threadIdx.x] = 0;
        sval_end[threadIdx.x] = 0;
        if (sval32_end != nullptr)
            sval32_end[threadIdx.x] = 0;
    }
    __syncthreads();
    unsigned panels = 0;   // of the thread's row
    visit_rows(n, W, rp, col, nullptr, [&](int row, int, int s, int c, double) {
        atomicAdd(&s_cnt[row][s], 1);
        c += s * W;
        panels |= c < 2 * W4 ? (c < W4 ? 1u : 2u) : (c < 3 * W4 ? 4u : 8u);
    });
    store_filled(panels, filled);   // its barrier orders the counts too
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    for (int s = threadIdx.x >> 6; s < P; s += kConvThreads / 64) {
        const int scan = ck::wave_scan(s_cnt[lane][s]);
        if (i < n)
            ends[(int64_t)s * n + i] = (unsigned short)scan;
        if (lane == 63)
            total[(int64_t)s * G + blockIdx.x] = scan;
    }
}

// The entries: row i's in slice s go to base[s*G + g] + ends[s*n + i - 1] onwards.
// They are put in order in LDS and leave it a slice's at a time, coalesced: stored
// from where they are read, a few bytes to a line, they took 115 us (n = 300,000,
// 10.2M entries; 62 us now).  Groups of more than kStage entries do that.
constexpr int kStage = 3072;

template <bool F32>
__global__ __launch_bounds__(kConvThreads) void slices_fill(
    int n, int P, int W, int G, const int *__restrict__ rp, const int *__restrict__ col,
    const double *__restrict__ val, const unsigned short *__restrict__ ends,
    const int *__restrict__ base, unsigned short *__restrict__ scol, double *__restrict__ sval,
    float *__restrict__ sval32, int *__restrict__ filled) {
    if (blockIdx.x == 0) {   // one workgroup adds up the groups' filled panels on the way
        int sum = 0;
        for (int g = threadIdx.x; g < G; g += kConvThreads)
            sum += filled[g];
        sum = ck::wave_sum(sum);
        if ((threadIdx.x & 63) == 0)
            atomicAdd(&filled[G], sum);
    }
    __shared__ double s_val[kStage];
    __shared__ unsigned short s_col[kStage];
    // destination of the row's entries minus their place in the CSR arrays
    __shared__ int s_shift[64][kSlices + 1];
    __shared__ unsigned short s_len[64][kSlices + 1];
    __shared__ int s_start[kSlices + 1];   // of the group's entries in LDS
    const int lane = threadIdx.x & 63;
    const int r0 = blockIdx.x * 64, last = min(r0 + 63, n - 1);
    const bool staged = rp[last + 1] - rp[r0] <= kStage;
    if (threadIdx.x < 64) {   // P <= kSlices < 64
        const int count = lane < P ? ends[(int64_t)lane * n + last] : 0;
        const int scan = ck::wave_scan(count);
        if (lane <= P)
            s_start[lane] = scan - count;
    }
    __syncthreads();
    const int64_t i = min(r0 + lane, n - 1);
    for (int s = threadIdx.x >> 6; s < P; s += kConvThreads / 64) {
        const int end = ends[(int64_t)s * n + i];
        const int up = __shfl_up(end, 1), before = lane > 0 ? up : 0;
        s_len[lane][s] = (unsigned short)(end - before);
        s_shift[lane][s] = before + (staged ? s_start[s] : base[(int64_t)s * G + blockIdx.x]);
    }
    __syncthreads();
    // less the row's entries before the slice
    if (threadIdx.x < 64) {
        int k = rp[i];
#pragma unroll 4
        for (int s = 0; s < P; ++s) {
            s_shift[lane][s] -= k;
            k += s_len[lane][s];
        }
    }
    __syncthreads();
    visit_rows(n, W, rp, col, val, [&](int row, int k, int s, int c, double v) {
        const int to = s_shift[row][s] + k;
        if (staged) {
            s_col[to] = (unsigned short)c;
            s_val[to] = v;
        } else {
            scol[to] = (unsigned short)c;
            sval[to] = v;
            if (F32)
                sval32[to] = (float)v;
        }
    });
    if (!staged)   // uniform
        return;
    __syncthreads();
    for (int s = threadIdx.x >> 6; s < P; s += kConvThreads / 64) {
        const int from = s_start[s], count = s_start[s + 1] - from;
        const int64_t to = base[(int64_t)s * G + blockIdx.x];
        for (int k = lane; k < count; k += 64) {
            scol[to + k] = s_col[from + k];
            const double v = s_val[from + k];
            sval[to + k] = v;
            if (F32)
                sval32[to + k] = (float)v;
        }
    }
}

// ypart[s*n + i] = row i's sum in slice s.  Groups of 64 / L rows, L lanes adding up
// each; C workgroups per slice.  The next group's row ends and entries are on their
// way in registers while a group is computed.  Instructions bound it about as much
// as the entries' bytes do, so nothing is masked that need not be: a group takes
// kSlicePass entries at once, the following groups' among them (kSlicePass zeros
// end the arrays), and only its own products are added up.
template <typename T, int L>
__global__ __launch_bounds__(kSliceThreads) void spmv_slices(
    int n, int ncols, int P, int W, int C, const int *__restrict__ base,
    const unsigned short *__restrict__ ends, const unsigned short *__restrict__ pcol,
    const T *__restrict__ pval, const T *__restrict__ x, T *__restrict__ ypart,
    const int *__restrict__ skip) {
    if (skip != nullptr && *skip != 0)
        return;
    constexpr int X = kSliceW / kSliceThreads, E = kSlicePass / 64, R = 64 / L, A = 4;
    constexpr int kWaves = kSliceThreads / 64;
    __shared__ T xs[kSliceW];
    __shared__ T s_prod[kWaves * kSlicePass + (A - 1) * L];   // read past, not used
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    T *prod = s_prod + wave * kSlicePass;
    const int s = blockIdx.x % P, step = C * kWaves, groups = (n + R - 1) / R;
    base += (int64_t)s * ((n + 63) / 64);
    ends += (int64_t)s * n;
    ypart += (int64_t)s * n;
    const int row = lane / L, part = lane % L;
    struct Rows {
        int base, first, end;   // of the 64 rows; entries before the group; the lane's row
    };
    struct Group {
        T v[E];
        int c[E], from, to, at, count;   // from, to: of the lane's row
    };
    auto fetch_rows = [&](int g, Rows &w) {   // rows past the last are empty
        const int r0 = g * R;
        w.base = base[r0 / 64];
        w.first = r0 % 64 != 0 ? ends[r0 - 1] : 0;
        w.end = ends[min(r0 + row, n - 1)];
    };
    auto fetch = [&](const Rows &w, Group &e) {
        e.at = w.base + w.first;
        e.to = w.end - w.first;
        e.count = __builtin_amdgcn_readlane(e.to, 63);
        e.from = __shfl_up(e.to, L);
        if (row == 0)
            e.from = 0;
        const unsigned short *pc = pcol + e.at;
        const T *pv = pval + e.at;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            e.c[u] = pc[u * 64 + lane];
            e.v[u] = pv[u * 64 + lane];
        }
    };
    int g = (int)(blockIdx.x / P) * kWaves + wave;
    Rows rows;   // of the next group
    Group e;
    if (g < groups) {
        fetch_rows(g, rows);
        fetch(rows, e);
        fetch_rows(min(g + step, groups - 1), rows);
    }
#pragma unroll
    for (int j = 0; j < X; ++j)
        xs[j * kSliceThreads + tid] = x[min(s * W + j * kSliceThreads + tid, ncols - 1)];
    __syncthreads();
    for (; g < groups; g += step) {
        Group next;
        fetch(rows, next);
        fetch_rows(min(g + 2 * step, groups - 1), rows);
#pragma unroll
        for (int u = 0; u < E; ++u)
            prod[u * 64 + lane] = e.v[u] * xs[e.c[u]];
        T acc = 0;
        for (int k0 = 0;;) {   // products k0 .. k0 + kSlicePass - 1 are in LDS
            __builtin_amdgcn_wave_barrier();
            const int last = min(e.to - k0, kSlicePass);
            for (int k = max(e.from - k0, 0) + part; k < last; k += A * L) {
                T p[A];
#pragma unroll
                for (int u = 0; u < A; ++u)
                    p[u] = prod[k + u * L];
#pragma unroll
                for (int u = 0; u < A; ++u)
                    acc += k + u * L < last ? p[u] : T(0);
            }
            k0 += kSlicePass;
            if (k0 >= e.count)   // uniform
                break;
            __builtin_amdgcn_wave_barrier();
            for (int k = lane; k < kSlicePass && k0 + k < e.count; k += 64)
                prod[k] = pval[e.at + k0 + k] * xs[pcol[e.at + k0 + k]];
        }
        __builtin_amdgcn_wave_barrier();
        acc = ck::group_sum<L>(acc);
        const int r = g * R + row;
        if (part == 0 && r < n)
            ypart[r] = acc;
        e = next;
    }
}

}  // namespace

namespace ck {

int slices_of(int64_t n, int64_t ncols, int64_t nnz, int64_t max_row, int64_t span) {
    if (n == 0 || nnz < kSliceMinNnz)
        return 0;
    const int64_t mean = ceil_div(nnz, n), P = ceil_div(ncols, kSliceW);
    if (P > kSlices || 2 * mean < 3 * P || max_row > 4 * mean || max_row > kLongSliceRow ||
        span < n * (ncols / 4) ||
        slices_work_bytes(n, (int)P, false) > kSliceWorkBytes ||
        P * ceil_div(n, 64) + panel_scan_tmp_elems(P * ceil_div(n, 64)) > 2 * nnz)
        return 0;
    return (int)P;
}

// The slices' arrays in one block, each 256-byte aligned, and the conversion's counts of
// filled panels: a group's each, and their sum.
struct SliceMem {
    int64_t ends, val32, col, base, filled, bytes;   // after the FP64 values
};
static SliceMem slice_mem(int64_t n, int64_t nnz, int P, bool fp32) {
    auto up = [](int64_t b) { return ceil_div(b, 256) * 256; };
    const int64_t entries = nnz + kSlicePass;
    SliceMem m;
    m.val32 = up(8 * entries);
    m.col = m.val32 + (fp32 ? up(4 * entries) : 0);
    m.ends = m.col + up(2 * entries);
    m.base = m.ends + up(2 * P * n);
    m.filled = m.base + up(4 * (P * ceil_div(n, 64) + 1));
    m.bytes = m.filled + 4 * (ceil_div(n, 64) + 1);
    return m;
}
int64_t slices_bytes(int64_t n, int64_t nnz, int P, bool fp32) {
    return slice_mem(n, nnz, P, fp32).bytes;
}

static int64_t slice_width(const ck_matrix &M, int P) {   // slices of equal width
    return ceil_div(ceil_div(M.ncols, P), 64) * 64;
}

int64_t slices_work_bytes(int64_t n, int P, bool fp32) { return P * n * (fp32 ? 4 : 8); }

ck_status build_slices(ck_matrix &M, int P, hipStream_t s) {
    const int64_t G = ceil_div(M.n, 64), N = P * G;
    const SliceMem m = slice_mem(M.n, M.nnz, P, M.val32 != nullptr);
    char *mem = nullptr;
    CK_TRY(mat_alloc(M, &mem, m.bytes, s));
    M.slice_P = P;
    M.slice_val = (double *)mem;
    M.slice_val32 = M.val32 ? (float *)(mem + m.val32) : nullptr;
    M.slice_col = (unsigned short *)(mem + m.col);
    M.slice_ends = (unsigned short *)(mem + m.ends);
    M.slice_base = (int *)(mem + m.base);
    // the groups' totals and the scan's scratch lie where the values come after them
    int *total = (int *)mem, *filled = (int *)(mem + m.filled);
    const int n = (int)M.n, W = (int)slice_width(M, P);
    hipLaunchKernelGGL(slices_count, dim3(G), dim3(kConvThreads), 0, s, n,
                       (int)ceil_div(M.ncols, 4), P, W, (int)G, M.rp, M.col, M.slice_ends, total,
                       filled, M.slice_col + M.nnz, M.slice_val + M.nnz,
                       M.val32 ? M.slice_val32 + M.nnz : nullptr);
    ck_status st = launch_scan_exclusive(N, total, M.slice_base, total + N, s);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(G), dim3(kConvThreads), 0, s, n, P, W, (int)G, M.rp, M.col,
                           M.val, M.slice_ends, M.slice_base, M.slice_col, M.slice_val,
                           M.slice_val32, filled);
    };
    if (st == CK_OK)
        M.val32 ? go(slices_fill<true>) : go(slices_fill<false>);
    if (hipGetLastError() != hipSuccess && st == CK_OK)
        st = fail(CK_E_HIP, "conversion to slices failed");
    CK_TRY(st);
    // the panels that CSR-panel would make of M, for ck_panel_layout: four where the
    // rows fill them, else eight, counted only then
    int four = 0;
    CK_HIP(hipMemcpyAsync(&four, filled + G, sizeof four, hipMemcpyDeviceToHost, s));
    CK_HIP(hipStreamSynchronize(s));
    if (panel_layout_of(M, 4, (unsigned)four))
        return CK_OK;
    std::vector<int> eight(G);
    hipLaunchKernelGGL(slices_eight, dim3(G), dim3(kConvThreads), 0, s, n,
                       (int)ceil_div(M.ncols, 8), M.rp, M.col, filled);
    CK_HIP(hipGetLastError());
    CK_HIP(hipMemcpyAsync(eight.data(), filled, G * sizeof(int), hipMemcpyDeviceToHost, s));
    CK_HIP(hipStreamSynchronize(s));
    panel_layout_of(M, 8, std::accumulate(eight.begin(), eight.end(), int64_t(0)));
    return CK_OK;
}

void free_slices(ck_matrix &M) {
    mat_free(M, M.slice_val);
    M.slice_val = nullptr;
}

template <typename T>
ck_status launch_slices(const ck_matrix &M, const SpmvArgs<T> &a, T *ypart, int64_t G_dot,
                        hipStream_t s) {
    const T *val;
    if constexpr (sizeof(T) == 4)
        val = M.slice_val32;
    else
        val = M.slice_val;
    const int P = M.slice_P;
    // a workgroup's LDS leaves room for one more of FP32 on its CU
    const int C = std::max<int>(1, (sizeof(T) == 4 ? 2 : 1) * kSliceCUs / P);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(P * C), dim3(kSliceThreads), 0, s, (int)M.n, (int)M.ncols,
                           P, (int)slice_width(M, P), C, M.slice_base, M.slice_ends, M.slice_col, val, a.x,
                           ypart, a.skip);
    };
    // groups of at most about 3/4 of the products kept
    const int64_t rows = (int64_t)kSlicePass * 3 / 4 * P * M.n / M.nnz;
    if (rows >= 64)
        go(spmv_slices<T, 1>);
    else if (rows >= 32)
        go(spmv_slices<T, 2>);
    else if (rows >= 16)
        go(spmv_slices<T, 4>);
    else if (rows >= 8)
        go(spmv_slices<T, 8>);
    else
        go(spmv_slices<T, 16>);
    CK_HIP(hipGetLastError());
    return launch_panel_combine<T>(M, a, ypart, G_dot, s);
}
template ck_status launch_slices<double>(const ck_matrix &, const SpmvArgs<double> &, double *,
                                         int64_t, hipStream_t);
template ck_status launch_slices<float>(const ck_matrix &, const SpmvArgs<float> &, float *,
                                        int64_t, hipStream_t);

}  // namespace ck
