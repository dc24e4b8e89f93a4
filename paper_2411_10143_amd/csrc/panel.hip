// CSR-panel SpMV: an MI355X-specific CSR algorithm for matrices whose column
// pattern is scattered (the gathered vector x does not fit one XCD's L2).
//
// The GPU has 8 XCDs, each with a private 4 MB L2.  The columns are split
// into P = 8q panels whose slice of x is at most 2 MB; the matrix is stored
// panel-major (all of panel 0, row by row, then panel 1, ...), which is one
// CSR of P*n rows.  Its product runs as a merge path (spmv.hip) whose
// contiguous per-XCD block ranges give each XCD its own consecutive panels,
// so the gathers find their x slice in that XCD's L2 instead of fetching a
// cache line from the fabric for every entry.  Each panel writes its partial
// row sums; a combine kernel adds the P partials in panel order
// (deterministic) and applies alpha/beta (and the fused CG dot).
#include <algorithm>

#include "matrix.hpp"
#include "panel.hpp"
#include "solvers.hpp"


// Rows longer than this are not run by their eight lanes entry by entry: with
// rows of 10,000 entries on eight lanes the copy of a power-law matrix (n =
// 1.2M, 33M entries) took 1,420 us, 328 us now.
constexpr int kLongPanelRow = 512;

// cnt[p*n + i] = entries of row i whose column lies in panel p, and *filled +=
// the panel rows that have any.  A workgroup takes 32 rows, eight lanes each,
// and eight panels at a time.  Rows of at most kCountRow entries are counted
// entry by entry, by comparing each column with the panels' ends (B of them;
// instructions bound the pass: dividing each column by W took 62 us where this
// takes 26); in longer rows each lane searches its panel's ends.  The counts go
// through LDS so that they are stored 32 rows to a panel.  One lane per row
// searching panel after panel took 97 us for 16M entries in four panels, one
// lane per panel 64 us.
constexpr int kCountRow = 64;
__global__ __launch_bounds__(256) void panel_count(int64_t n, int P, int W,
                                                   const int *__restrict__ rp,
                                                   const int *__restrict__ col,
                                                   int *__restrict__ cnt, unsigned *filled) {
    constexpr int L = 8, R = 256 / L, U = 4;
    __shared__ int s_len[R][L + 1];
    __shared__ unsigned part[4];
    const int tid = threadIdx.x, lane = tid & (L - 1), row = tid / L;
    unsigned full = 0;
    const int64_t groups = (n + R - 1) / R;
    // entries below each of the first B - 1 ends; the row's other entries of
    // these panels end the B-th
    auto count = [&](auto ends, int k0, int k1, int p0) {
        constexpr int B = decltype(ends)::value;
        int end[B], below[B];
#pragma unroll
        for (int e = 0; e < B; ++e) {
            end[e] = (int)min((int64_t)(p0 + e + 1) * W, (int64_t)INT_MAX);
            below[e] = 0;
        }
        for (int t = k0; t < k1; t += L * U) {
            int c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = t + u * L + lane;
                c[u] = k < k1 ? col[k] : INT_MAX;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < B; ++e)
                    below[e] += c[u] < end[e] ? 1 : 0;
        }
        int mine = 0, before = 0;
#pragma unroll
        for (int e = 0; e < B; ++e) {
            below[e] = ck::group_sum_last<L>(below[e]);   // in every lane
            if (lane == e)
                mine = below[e] - before;
            before = below[e];
        }
        s_len[row][lane] = mine;
        return before;
    };
    for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
        const int64_t i = g * R + row;
        int k0 = i < n ? rp[i] : 0;
        const int k1 = i < n ? rp[i + 1] : 0;
        const bool shrt = k1 - k0 <= kCountRow;
        for (int p0 = 0; p0 < P; p0 += L) {
            if (shrt) {
                if (P - p0 <= 4)   // uniform
                    k0 += count(std::integral_constant<int, 4>(), k0, k1, p0);
                else
                    k0 += count(std::integral_constant<int, 8>(), k0, k1, p0);
            } else {
                auto find = [&](int64_t first) {   // the first entry at or past column `first`
                    int lo = k0, top = k1;
                    while (lo < top) {
                        const int mid = (lo + top) >> 1;
                        if (col[mid] < first)
                            lo = mid + 1;
                        else
                            top = mid;
                    }
                    return lo;
                };
                const int64_t first = (int64_t)(p0 + lane) * W;
                const int at = find(first);
                int end = __shfl_down(at, 1, L);
                if (lane == L - 1)
                    end = p0 + L < P ? find(first + W) : k1;
                s_len[row][lane] = end - at;
            }
            __syncthreads();
            const int p = tid / R, r = tid % R;
            if (p0 + p < P && g * R + r < n) {
                const int len = s_len[r][p];
                cnt[(int64_t)(p0 + p) * n + g * R + r] = len;
                full += len > 0 ? 1u : 0u;
            }
            __syncthreads();
        }
    }
    full = ck::wave_sum(full);
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = full;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned t = part[0] + part[1] + part[2] + part[3];
        if (t)
            atomicAdd(&filled[blockIdx.x % ck::kSpread * ck::kSpreadInts], t);
    }
}

// Panel-major copy: row i's panel-p entries go to prp[p*n + i] onwards.  A
// workgroup takes 32 rows, eight lanes each, and eight panels at a time.  The
// rows' destinations and lengths in those panels (staged in LDS, read 32 rows
// to a panel) give each panel's first entry within the row, since a row's
// entries of consecutive panels are consecutive.  The eight lanes copy the
// row's entries of those panels together, lane l taking entries l, l + 8, ...
// (coalesced loads), an entry's panel being its column / W.  Rows over
// kLongPanelRow are copied at the end by the whole workgroup: power-law rows, 33M
// entries, 328 us.  STAGE (matrices with no such row): the entries are put in order
// in LDS and leave it panel by panel, coalesced, unless a group has more than
// kPanelStage of them.  Stored from where they are read, a few to a line, 16M
// entries in four panels took 113 us, 97 us this way; of rows of 27 in eight panels
// most lines are partial either way, and the LDS costs waves (328 us, 414).
constexpr int kPanelStage = 2048;

template <bool F32, bool STAGE>
__global__ __launch_bounds__(256) void panel_fill(int64_t n, int P, int W,
                                                  const int *__restrict__ rp,
                                                  const int *__restrict__ col,
                                                  const double *__restrict__ val,
                                                  const int *__restrict__ prp,
                                                  int *__restrict__ pcol, double *__restrict__ pval,
                                                  float *__restrict__ pval32) {
    constexpr int L = 8, R = 256 / L, U = 4;
    __shared__ int s_long[R], s_count;
    __shared__ int s_dst[L][R + 1];     // panel p0 + p, row r
    __shared__ int s_shift[R][L + 1];   // destination minus the entry's place in the row
    __shared__ int s_first[L + 1];      // of each panel's entries in LDS
    __shared__ double s_val[STAGE ? kPanelStage : 1];
    __shared__ int s_col[STAGE ? kPanelStage : 1];
    const int tid = threadIdx.x, lane = tid & (L - 1), row = tid / L;
    const int64_t i0 = (int64_t)blockIdx.x * R, i = i0 + row;
    const float inv = 1.0f / (float)W;
    auto put = [&](int dst, int c, double v) {
        pcol[dst] = c;
        pval[dst] = v;
        if (F32)
            pval32[dst] = (float)v;
    };
    if (tid == 0)
        s_count = 0;
    __syncthreads();
    int base = i < n ? rp[i] : 0;
    const bool shrt = i >= n || rp[i + 1] - base <= kLongPanelRow;
    if (!shrt && lane == 0)
        s_long[atomicAdd(&s_count, 1)] = row;
    for (int p0 = 0; p0 < P; p0 += L) {
        {   // rows past n end where row n - 1 does: empty
            const int p = tid / R, r = tid % R;
            if (p0 + p < P) {
                const int64_t at = (int64_t)(p0 + p) * n;
                s_dst[p][r] = prp[at + min(i0 + r, n)];
                if (r == R - 1)
                    s_dst[p][R] = prp[at + min(i0 + R, n)];
            } else {   // panels past the last: empty
                s_dst[p][r] = 0;
                if (r == R - 1)
                    s_dst[p][R] = 0;
            }
        }
        __syncthreads();
        const int dst = s_dst[lane][row], len = s_dst[lane][row + 1] - dst;
        int ex = len;   // inclusive scan over the group's lanes, then exclusive
#pragma unroll
        for (int off = 1; off < L; off <<= 1) {
            const int o = __shfl_up(ex, off, L);
            if (lane >= off)
                ex += o;
        }
        const int total = shrt ? __shfl(ex, L - 1, L) : 0;
        if (STAGE && tid < 64) {   // where the panels start in LDS
            const int count = tid < L ? s_dst[tid][R] - s_dst[tid][0] : 0;
            const int scan = ck::wave_scan(count);
            if (tid <= L)
                s_first[tid] = scan - count;
        }
        if (STAGE)
            __syncthreads();
        const bool staged = STAGE && s_count == 0 && s_first[L] <= kPanelStage;   // uniform
        s_shift[row][lane] = dst - (ex - len) - (staged ? s_dst[lane][0] - s_first[lane] : 0);
        __syncthreads();
        for (int k0 = 0; k0 < total; k0 += L * U) {
            int c[U];
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * L + lane;
                c[u] = k < total ? col[base + k] : -1;
                v[u] = k < total ? val[base + k] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (c[u] >= 0) {
                    const int to =
                        s_shift[row][ck::panel_of(c[u], W, inv) - p0] + k0 + u * L + lane;
                    if (staged) {
                        s_col[to] = c[u];
                        s_val[to] = v[u];
                    } else {
                        put(to, c[u], v[u]);
                    }
                }
        }
        base += total;
        __syncthreads();
        if (staged) {
            for (int p = tid >> 6; p < L; p += 4) {
                const int from = s_first[p], count = s_first[p + 1] - from, to = s_dst[p][0];
                for (int k = tid & 63; k < count; k += 64)
                    put(to + k, s_col[from + k], s_val[from + k]);
            }
            __syncthreads();   // s_dst, s_shift and s_first are rewritten
        }
    }
    const int count = s_count;   // written before the barriers, and not again
    for (int t = 0; t < count; ++t) {
        const int64_t r = i0 + s_long[t];
        int from = rp[r];
        for (int p0 = 0; p0 < P; p0 += L) {
            if (tid < L) {
                const bool has = p0 + tid < P;
                const int64_t at = (int64_t)(p0 + tid) * n + r;
                const int d = has ? prp[at] : 0;
                s_first[tid + 1] = has ? prp[at + 1] - d : 0;
                s_dst[tid][0] = d;
            }
            __syncthreads();
            if (tid == 0) {
                s_first[0] = 0;
                for (int q = 1; q <= L; ++q)
                    s_first[q] += s_first[q - 1];
            }
            __syncthreads();
            const int total = s_first[L];
            for (int k = tid; k < total; k += 256) {
                const int c = col[from + k];
                const int q = ck::panel_of(c, W, inv) - p0;
                put(s_dst[q][0] + (k - s_first[q]), c, val[from + k]);
            }
            from += total;
            __syncthreads();   // s_dst and s_first are rewritten
        }
    }
}

// Exclusive scan of Nin int counts into Nout >= Nin outputs (inputs past Nin
// read as 0, so out[Nin] is the total): 2048 items per workgroup, each thread
// scanning 8 consecutive items, then the 256 thread totals by wave scans.  The
// block totals go to sums[] for the next level.
__global__ __launch_bounds__(256) void scan_blocks(int64_t Nin, int64_t Nout,
                                                   const int *__restrict__ in,
                                                   int *__restrict__ out, int *__restrict__ sums) {
    __shared__ int s[2048 + 256];   // one slot of padding per eight (bank conflicts)
    const int64_t base = (int64_t)blockIdx.x * 2048;
    for (int t = threadIdx.x; t < 2048; t += 256)
        s[t + (t >> 3)] = base + t < Nin ? in[base + t] : 0;
    __syncthreads();
    int local[8];
    int acc = 0;
    for (int t = 0; t < 8; ++t) {
        local[t] = acc;
        acc += s[threadIdx.x * 9 + t];
    }
    __shared__ int wsum[4];
    const int sc = ck::wave_scan(acc), w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63)
        wsum[w] = sc;
    __syncthreads();
    int off = sc - acc;
#pragma unroll
    for (int u = 0; u < 3; ++u)
        off += u < w ? wsum[u] : 0;
    if (threadIdx.x == 255)
        sums[blockIdx.x] = off + acc;
    for (int t = 0; t < 8; ++t)
        s[threadIdx.x * 9 + t] = off + local[t];
    __syncthreads();
    for (int t = threadIdx.x; t < 2048; t += 256)
        if (base + t < Nout)
            out[base + t] = s[t + (t >> 3)];
}

__global__ __launch_bounds__(256) void scan_add(int64_t N, int *__restrict__ out,
                                                const int *__restrict__ offs) {
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g < N)
        out[g] += offs[g / 2048];
}

// flag[k] = 1 if panel row k holds entries (in place over the counts)
__global__ __launch_bounds__(256) void panel_nonempty(int64_t N, int *__restrict__ cnt) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < N)
        cnt[k] = cnt[k] > 0 ? 1 : 0;
}

// Row list of the non-empty panel rows: panel row k = p*n + i with entries
// becomes list entry pos[k] (row i, start prp[k]); the list ends at nnz.
__global__ __launch_bounds__(256) void panel_compact(int64_t N, int64_t n, int64_t NE, int nnz,
                                                     const int *__restrict__ prp,
                                                     const int *__restrict__ pos,
                                                     int *__restrict__ prow,
                                                     int *__restrict__ prp_ne) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k == 0)
        prp_ne[NE] = nnz;
    if (k >= N)
        return;
    const int start = prp[k];
    if (prp[k + 1] > start) {
        const int j = pos[k];
        prow[j] = (int)(k % n);
        prp_ne[j] = start;
    }
}

// boff[p*(B+1) + j] = list position of panel p's first row >= 256 j (rows
// past n clamp to n, so boff[p*(B+1) + B] ends panel p)
__global__ __launch_bounds__(256) void panel_block_offsets(int64_t n, int P, int64_t B,
                                                           const int *__restrict__ pos,
                                                           int *__restrict__ boff) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)P * (B + 1))
        return;
    const int64_t p = t / (B + 1), j = t % (B + 1);
    boff[t] = pos[p * n + min(j * 256, n)];
}

// Row-list combine: workgroup row block [256 blk, 256 blk + 256) adds, panel
// by panel in order, the partials of its rows' non-empty panel rows into an
// LDS accumulator (a row appears at most once per panel, so the threads of
// one panel step never share a slot); rows absent from a panel add nothing,
// which gives the dense combine's sum bit for bit (a partial is never -0).
template <typename T, bool BETA, bool DOT>
__global__ __launch_bounds__(256) void panel_combine_rows(
    int64_t n, int P, int64_t B, int64_t G, const int *__restrict__ boff,
    const int *__restrict__ prow, const T *__restrict__ ypart, T alpha, T beta,
    T *__restrict__ y, const T *__restrict__ x, T *__restrict__ partials,
    const int *__restrict__ skip) {
    if (skip != nullptr && *skip != 0)
        return;
    const int64_t b = ck::xcd_block(G);
    if (b < 0)
        return;
    __shared__ double acc[256];   // as in panel_combine
    const int tid = threadIdx.x;
    T mine = 0;
    for (int64_t blk = b; blk < B; blk += G) {
        const int64_t r0 = blk * 256;
        acc[tid] = 0;
        __syncthreads();
        for (int p = 0; p < P; ++p) {
            const int lo = boff[(int64_t)p * (B + 1) + blk];
            const int hi = boff[(int64_t)p * (B + 1) + blk + 1];
            for (int k = lo + tid; k < hi; k += 256)
                acc[prow[k] - r0] += ypart[k];
            __syncthreads();
        }
        const int64_t i = r0 + tid;
        if (i < n) {
            T out = alpha * (T)acc[tid];
            if (BETA)
                out += beta * y[i];
            y[i] = out;
            if (DOT)
                mine += out * x[i];
        }
        __syncthreads();   // acc is cleared for the next block only after every read
    }
    if constexpr (DOT) {
        __shared__ T lds[4];
        const T d = ck::block_sum(mine, lds);
        if (threadIdx.x == 0)
            partials[b] = d;
    }
}

// y = alpha * sum_p ypart[p] + beta * y   (+ per-block partial of y.x for CG).
// FP32 partial sums are added in FP64, which costs nothing here: with up to 22
// of them (slices of x) the FP32 sum's rounding showed in the result.
template <typename T, bool BETA, bool DOT>
__global__ __launch_bounds__(256) void panel_combine(int64_t n, int P, int64_t G,
                                                     const T *__restrict__ ypart, T alpha, T beta,
                                                     T *__restrict__ y, const T *__restrict__ x,
                                                     T *__restrict__ partials,
                                                     const int *__restrict__ skip) {
    if (skip != nullptr && *skip != 0)
        return;
    const int64_t b = ck::xcd_block(G);
    if (b < 0)
        return;
    T mine = 0;
    for (int64_t i = b * 256 + threadIdx.x; i < n; i += G * 256) {
        double s = 0;
        for (int p = 0; p < P; ++p)
            s += ypart[(int64_t)p * n + i];
        T out = alpha * (T)s;
        if (BETA)
            out += beta * y[i];
        y[i] = out;
        if (DOT)
            mine += out * x[i];
    }
    if constexpr (DOT) {
        __shared__ T lds[4];
        const T d = ck::block_sum(mine, lds);
        if (threadIdx.x == 0)
            partials[b] = d;
    }
}

namespace ck {

ck_status launch_scan_exclusive(int64_t N, const int *in, int *out, int *tmp, hipStream_t s);

int panel_count_for(int64_t ncols, int value_bytes) {
    const int64_t per_panel = (2 << 20) / value_bytes;        // x slice <= 2 MB
    const int64_t q = std::max<int64_t>(1, ceil_div(ncols, 8 * per_panel));
    return (int)(8 * q);
}

// A matrix whose x fits four slices of at most 2.5 MB, whose rows are of
// even length (the longest at most four times the mean) and have entries in
// nearly every one of four panels, takes P = 4 (two XCDs share a panel): its
// partial sums, kept dense, halve while each XCD's slice still stays in its
// 4 MB L2 (uniform-random rows of 4-64 entries: 292 -> 253 us at n = 1.2M,
// 185 -> 160 us at n = 0.76M).  Short-row matrices keep P = 8: their row
// lists gain little from fewer panels and lose L2 hits (power-law n = 1.2M:
// 272 -> 304 us with P = 4); so do hub-row graphs (14-31 % slower with P = 4
// on the training graphs) and matrices with a larger x (uniform n = 2M, a
// 4 MB slice: 465 -> 483 us).
constexpr int64_t kSliceP4 = 5 * (int64_t(1) << 19);   // 2.5 MB

// The per-row panel counts into cnt (P*n ints) and, read back, how many are not
// zero; their counters follow them.
static ck_status count_panels(const ck_matrix &M, int P, int64_t W, int *cnt, int64_t *filled,
                              hipStream_t s) {
    constexpr int64_t ints = kSpread * kSpreadInts;
    int *total = cnt + (int64_t)P * M.n;
    int host[ints];
    CK_TRY(launch_fill<int>(ints, total, 0, s));
    hipLaunchKernelGGL(panel_count, dim3(std::min<int64_t>(ceil_div(M.n, 256 / 8), 4096)), dim3(256),
                       0, s, M.n, P, (int)W, M.rp, M.col, cnt, (unsigned *)total);
    CK_HIP(hipGetLastError());
    CK_HIP(hipMemcpyAsync(host, total, sizeof host, hipMemcpyDeviceToHost, s));
    CK_HIP(hipStreamSynchronize(s));
    *filled = 0;
    for (int t = 0; t < kSpread; ++t)
        *filled += (unsigned)host[t * kSpreadInts];
    return CK_OK;
}

// Whether four panels are tried, and whether `filled` of `rows` panel rows make them dense.
static bool may_take_four(const ck_matrix &M) {
    return panel_count_for(M.ncols, 8) == 8 && M.ncols * 8 <= 4 * kSliceP4 &&
           M.max_row <= 4 * ceil_div(M.nnz, M.n);
}
static bool dense_rows(int64_t filled, int64_t rows) { return 4 * filled > 3 * rows; }

bool panel_layout_of(ck_matrix &M, int P, int64_t filled) {
    const bool dense = dense_rows(filled, P * M.n);
    if (P == 4 && !(may_take_four(M) && dense))
        return false;
    M.panel_P = P;
    M.panel_W = ceil_div(std::max<int64_t>(M.ncols, 1), P);
    M.panel_rows = dense ? P * M.n : filled;
    return true;
}

ck_status panel_choose_count(const ck_matrix &M, int *tmp, hipStream_t s, int *P_out,
                             int64_t *filled) {
    const int P8 = panel_count_for(M.ncols, 8);
    const int64_t W8 = ceil_div(std::max<int64_t>(M.ncols, 1), P8);
    *P_out = P8;
    *filled = 0;
    if (M.n == 0)
        return CK_OK;
    if (may_take_four(M)) {
        const int64_t W4 = ceil_div(std::max<int64_t>(M.ncols, 1), 4);
        CK_TRY(count_panels(M, 4, W4, tmp, filled, s));
        if (dense_rows(*filled, 4 * M.n)) {
            *P_out = 4;
            return CK_OK;
        }
    }
    return count_panels(M, P8, W8, tmp, filled, s);
}

int64_t panel_tmp_ints(int64_t N) {
    return N + std::max<int64_t>(kSpread * kSpreadInts, panel_scan_tmp_elems(N));
}

int64_t panel_convert_bytes(int64_t n, int64_t ncols, int64_t nnz, int value_bytes) {
    const int64_t P = panel_count_for(ncols, 8), N = P * n;
    const int64_t all = nnz * (4 + value_bytes) + 4 * panel_tmp_ints(N);
    // dense panel rows: their pointers and the plan
    const int64_t dense = 4 * (N + 1) + 4 * merge_plan_ints(N, nnz);
    // row list: its arrays beside the dense pointers and the scan (panel_make_rows),
    // then beside the plan alone
    const int64_t NE = std::min(3 * N / 4, nnz);
    const int64_t list = 4 * NE + 4 * (NE + 1) + 4 * P * (ceil_div(n, 256) + 1);
    const int64_t make = 4 * (N + 1) + 4 * (N + 1 + panel_scan_tmp_elems(N));
    return all + std::max(dense, list + std::max(make, 4 * merge_plan_ints(NE, nnz)));
}

int64_t panel_scan_tmp_elems(int64_t N) {
    const int64_t b1 = ceil_div(N + 1, 2048);
    const int64_t b2 = ceil_div(b1, 2048);
    return b1 + b1 + b2 + b2 + 2048 + 64;
}

// Exclusive scan of N ints (N + 1 outputs: out[N] = total), up to three levels.
ck_status launch_scan_exclusive(int64_t N, const int *in, int *out, int *tmp, hipStream_t s) {
    const int64_t M = N + 1;                     // in[N] is read as 0 via the bound
    const int64_t b1 = ceil_div(M, 2048);
    int *s1 = tmp, *s1x = tmp + b1;              // block sums and their scan
    const int64_t b2 = ceil_div(b1, 2048);
    int *s2 = s1x + b1, *s2x = s2 + b2;
    int *s3 = s2x + b2;
    if (b2 > 2048)
        return fail(CK_E_UNSUPPORTED, "scan too large");
    hipLaunchKernelGGL(scan_blocks, dim3(b1), dim3(256), 0, s, N, M, in, out, s1);
    hipLaunchKernelGGL(scan_blocks, dim3(b2), dim3(256), 0, s, b1, b1, s1, s1x, s2);
    if (b2 > 1) {
        hipLaunchKernelGGL(scan_blocks, dim3(1), dim3(256), 0, s, b2, b2, s2, s2x, s3);
        hipLaunchKernelGGL(scan_add, dim3(ceil_div(b1, 256)), dim3(256), 0, s, b1, s1x, s2x);
    }
    hipLaunchKernelGGL(scan_add, dim3(ceil_div(M, 256)), dim3(256), 0, s, M, out, s1x);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

ck_status launch_to_panel(const ck_matrix &M, int P, int64_t W, int *cnt, int *tmp, int *prp,
                          int *pcol, double *pval, float *pval32, hipStream_t s) {
    CK_TRY(launch_scan_exclusive((int64_t)P * M.n, cnt, prp, tmp, s));
    const int64_t g8 = ceil_div(M.n, 256 / 8);
    const int Wi = (int)W;   // W <= ncols < 2^31
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(g8), dim3(256), 0, s, M.n, P, Wi, M.rp, M.col, M.val, prp,
                           pcol, pval, pval32);
    };
    const bool stage = M.max_row <= kLongPanelRow && M.max_row * M.n <= 4 * M.nnz;
    if (pval32)
        stage ? go(panel_fill<true, true>) : go(panel_fill<true, false>);
    else
        stage ? go(panel_fill<false, true>) : go(panel_fill<false, false>);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

ck_status panel_make_rows(ck_matrix &M, int *cnt, int64_t filled, hipStream_t s) {
    const int64_t n = M.n, N = (int64_t)M.panel_P * n, NE = filled;
    M.panel_rows = N;
    if (dense_rows(NE, N) || N == 0)   // dense rows are cheaper
        return CK_OK;
    int *pos = nullptr;
    CK_TRY(mat_alloc(M, &pos, N + 1 + panel_scan_tmp_elems(N), s));
    hipLaunchKernelGGL(panel_nonempty, dim3(ceil_div(N, 256)), dim3(256), 0, s, N, cnt);
    ck_status st = launch_scan_exclusive(N, cnt, pos, pos + N + 1, s);
    if (st != CK_OK) {
        (void)hipStreamSynchronize(s);
        mat_free(M, pos);
        return st;
    }
    const int64_t B = ceil_div(n, 256);
    int *prow = nullptr, *prp_ne = nullptr, *boff = nullptr;
    st = mat_alloc(M, &prow, NE, s);
    if (st == CK_OK)
        st = mat_alloc(M, &prp_ne, NE + 1, s);
    if (st == CK_OK)
        st = mat_alloc(M, &boff, (int64_t)M.panel_P * (B + 1), s);
    if (st == CK_OK) {
        hipLaunchKernelGGL(panel_compact, dim3(ceil_div(N, 256)), dim3(256), 0, s, N, n, NE,
                           (int)M.nnz, M.panel_rp, pos, prow, prp_ne);
        hipLaunchKernelGGL(panel_block_offsets, dim3(ceil_div((int64_t)M.panel_P * (B + 1), 256)),
                           dim3(256), 0, s, n, M.panel_P, B, pos, boff);
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
            st = fail(CK_E_HIP, "panel row list failed");
    }
    (void)hipStreamSynchronize(s);
    mat_free(M, pos);
    if (st != CK_OK) {
        mat_free(M, prow);
        mat_free(M, prp_ne);
        mat_free(M, boff);
        return st;
    }
    mat_free(M, M.panel_rp);
    M.panel_rp = prp_ne;
    M.panel_row = prow;
    M.panel_boff = boff;
    M.panel_rows = NE;
    M.panel_B = B;
    return CK_OK;
}

template <typename T>
ck_status launch_panel_combine(const ck_matrix &M, const SpmvArgs<T> &a, const T *ypart,
                               int64_t G_dot, hipStream_t s) {
    const bool beta = a.beta != T(0);
    const bool dot = a.cg != nullptr;
    const int64_t G = dot ? G_dot : std::min<int64_t>(ceil_div(M.n, 256), kRowBlocks);
    const dim3 grid(xcd_grid(G));
    if (M.panel_row != nullptr) {
        const int64_t B = M.panel_B;
        if (dot)
            hipLaunchKernelGGL((panel_combine_rows<T, false, true>), grid, dim3(256), 0, s, M.n,
                               M.panel_P, B, G, M.panel_boff, M.panel_row, ypart, a.alpha, a.beta,
                               a.y, a.x, a.dot_partials, a.skip);
        else if (beta)
            hipLaunchKernelGGL((panel_combine_rows<T, true, false>), grid, dim3(256), 0, s, M.n,
                               M.panel_P, B, G, M.panel_boff, M.panel_row, ypart, a.alpha, a.beta,
                               a.y, a.x, a.dot_partials, a.skip);
        else
            hipLaunchKernelGGL((panel_combine_rows<T, false, false>), grid, dim3(256), 0, s, M.n,
                               M.panel_P, B, G, M.panel_boff, M.panel_row, ypart, a.alpha, a.beta,
                               a.y, a.x, a.dot_partials, a.skip);
        CK_HIP(hipGetLastError());
        return CK_OK;
    }
    const int P = M.slice_val != nullptr ? M.slice_P : M.panel_P;
    if (dot)
        hipLaunchKernelGGL((panel_combine<T, false, true>), grid, dim3(256), 0, s, M.n, P, G, ypart, a.alpha, a.beta, a.y, a.x, a.dot_partials, a.skip);
    else if (beta)
        hipLaunchKernelGGL((panel_combine<T, true, false>), grid, dim3(256), 0, s, M.n, P, G, ypart, a.alpha, a.beta, a.y, a.x, a.dot_partials, a.skip);
    else
        hipLaunchKernelGGL((panel_combine<T, false, false>), grid, dim3(256), 0, s, M.n, P, G,
                           ypart, a.alpha, a.beta, a.y, a.x, a.dot_partials, a.skip);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

template ck_status launch_panel_combine<double>(const ck_matrix &, const SpmvArgs<double> &,
                                                const double *, int64_t, hipStream_t);
template ck_status launch_panel_combine<float>(const ck_matrix &, const SpmvArgs<float> &,
                                               const float *, int64_t, hipStream_t);

}  // namespace ck
