// GMRES(m) kernels (the solver of the paper's evaluation, Section IV).
//
// One Arnoldi step j is classical Gram-Schmidt applied twice (CGS2):
//   h1 = V_j^T w, w' = w - V_j h1, h2 = V_j^T w',
//   h_{j+1,j} = ||w' - V_j h2|| = sqrt(||w'||^2 - ||h2||^2) (Pythagoras: the
//   subtracted part is w''s projection on the orthonormal V_j),
//   v_{j+1} = (w' - V_j h2) / h_{j+1,j},  column j of H = h1 + h2,
// with w = A v_j.  Forming v_{j+1} would take a third sweep over the basis;
// instead it is left for the next step, which applies the SpMV to w' itself
// (z = A w', written to column j+2) and opens with one sweep that forms both
// v_{j+1} = (w' - V_j h2) / h and A v_{j+1} = (z - V_{j+1} u) / h, where
// u = Hbar_j h2 is A (V_j h2) expressed in the basis through the Arnoldi
// relation A V_j = V_{j+1} Hbar_j, and that also sums the partials of
// V_{j+1}^T A v_{j+1}.  So each step streams the basis twice, in two kernels
// after its SpMV:
//   step 0:  pass 1 (partials of V_0^T w)
//   step j:  pass 3+1: every block sums the previous step's pass-2 partials
//            (h2, ||w'||^2) and forms h_{j,j-1} and u itself, then v_j, A v_j in
//            place and the partials of V_j^T A v_j; one more block does the
//            previous step's Givens work (H column, rotations, residual estimate
//            |g|, the cycle stop decision)
//   then     pass 2: every block sums the first-pass partials (h1) itself,
//            then w' = w - V_j h1, partials of V_j^T w' (h2) and ||w'||^2.
// (One-block kernels between the passes took 4.6 and 5.3 us and two launch
// gaps a step; summed in every block they take about 1.5 and 2.5 us, with at
// most 256 partials a column.  A step of FP64 GMRES(30) with DIA: n = 22,500
// 34.4 -> 21.2 us, 160,000 36.1 -> 25.0, 1,048,576 74.3 -> 69.8, of which the
// two sweeps run at 6.2 TB/s.)
// The Givens work of a cycle's last step opens the back substitution.  A
// step issued after the stop decision forms a column that is not used.
// After the first projection h2 is of rounding size relative to w', so the
// corrections through h2 and u change w' and z by rounding-size amounts.
// The last step of a cycle needs no v_{j+1}: the update x += V_k y uses
// v_0 .. v_{k-1}.  Per-column sums are reduced in a fixed order (wave
// butterfly, 4 waves, then block order), so results are deterministic.  The
// least-squares solve and the solution update close the cycle on the
// device; nothing returns to the host inside a cycle.
#include <algorithm>

#include "solvers.hpp"

using ck::GmDev;

namespace {

// The passes below are written for NC >= ncols columns with no branch per
// column: column c >= ncols reloads column ncols - 1 (an L2 hit), its
// coefficient h[c] is 0 (so the subtraction is exact) and its accumulator is
// never written out.  Without branches every column's load of an element is
// in flight at once; with a branch per column each load waited for the one
// before it.
__device__ __forceinline__ int64_t clampc(int c, int ncols) { return c < ncols ? c : ncols - 1; }

constexpr int kGmWaves = ck::kGmThreads / 64;

// partials[c*G + b] = block b's sum of acc[c]  (c < ncols), and of `extra` as
// column ncols if EXTRA.  The wave sums run back to back at the end of the
// pass, so they use register-to-register (DPP) moves, valid in lane 63.
template <bool EXTRA, typename T, int NC>
__device__ __forceinline__ void block_cols(const T (&acc)[NC], T extra, int ncols, T *partials,
                                           int64_t b, int64_t G) {
    __shared__ T lds[kGmWaves][NC + 1];
    const int w = threadIdx.x / 64, lane = threadIdx.x & 63;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (c < ncols) {
            const T v = ck::wave_sum_last(acc[c]);
            if (lane == 63)
                lds[w][c] = v;
        }
    }
    if constexpr (EXTRA) {
        const T v = ck::wave_sum_last(extra);
        if (lane == 63)
            lds[w][ncols] = v;
    }
    __syncthreads();
    const int cols = ncols + (EXTRA ? 1 : 0);
    if ((int)threadIdx.x < cols) {
        const int c = threadIdx.x;
        T t = 0;
#pragma unroll
        for (int v = 0; v < kGmWaves; v += 4)
            t += (lds[v][c] + lds[v + 1][c]) + (lds[v + 2][c] + lds[v + 3][c]);
        partials[c * G + b] = t;
    }
}

// out[c] = sum over the G blocks of partials[c*G + b], c < ncols, by the waves
// of a block: wave w takes columns w, w + kGmWaves, ..., four at a time, its
// lanes striding the blocks (up to four loads of each column in flight), then
// a wave sum.  Fixed order.  `out` is in LDS; a barrier must follow.
template <typename T>
__device__ __forceinline__ void sum_cols(int ncols, int64_t G, const T *__restrict__ partials,
                                         T *out) {
    constexpr int U = 4, C = 4;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int c0 = w; c0 < ncols; c0 += C * kGmWaves) {
        T sum[C];
#pragma unroll
        for (int k = 0; k < C; ++k)
            sum[k] = 0;
        for (int64_t b0 = lane; b0 < G; b0 += 64 * U) {
            T v[C][U];
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const int c = min(c0 + k * kGmWaves, ncols - 1);
#pragma unroll
                for (int t = 0; t < U; ++t)
                    v[k][t] = partials[c * G + (b0 + 64 * t < G ? b0 + 64 * t : G - 1)];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < C; ++k)
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (b0 + 64 * t < G)
                        sum[k] += v[k][t];
        }
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const T t = ck::wave_sum_last(sum[k]);   // valid in lane 63
            if (lane == 63 && c0 + k * kGmWaves < ncols)
                out[c0 + k * kGmWaves] = t;
        }
    }
}

// What the end of step s leaves for the next kernel, formed by a block from
// the step's pass-2 partials: h2 (column s + 1: ||w'||^2), the unrotated
// column s of H, h_{s+1,s} and u = Hbar_s h2.
template <typename T>
struct StepEnd {
    __align__(16) T h2[ck::kMaxRestart + 2];
    __align__(16) T u[ck::kMaxRestart + 2];
    T col[ck::kMaxRestart + 1];
    T hr[ck::kMaxRestart * (ck::kMaxRestart + 1)];   // Hraw columns 0 .. s-1
    T cs[ck::kMaxRestart], sn[ck::kMaxRestart];
    T hn;
};

template <typename T>
__device__ __forceinline__ void step_end(int s, int m, int64_t G, const T *__restrict__ partials,
                                         const GmDev<T> *st, StepEnd<T> &e) {
    const int t = threadIdx.x;
    // loads that do not depend on the sums are issued before them
    const T h1 = t <= s ? st->h1[t] : T(0);
    for (int k = t; k < s * (m + 1); k += ck::kGmThreads)
        e.hr[k] = st->Hraw[k];
    sum_cols(s + 2, G, partials, e.h2);
    __syncthreads();
    if (t <= s)
        e.col[t] = h1 + e.h2[t];
    if (t < 64) {   // s < 64 columns: one wave sums h2^2
        const T h = t <= s ? e.h2[t] : T(0);
        const T proj = ck::wave_sum_last(h * h);   // valid in lane 63
        if (t == 63) {
            const T nrm2 = e.h2[s + 1] - proj;
            e.hn = nrm2 > T(0) ? sqrt(nrm2) : T(0);
        }
    }
    __syncthreads();
    // u_i sums columns c >= i - 1
    for (int i = t; i <= s + 1; i += ck::kGmThreads) {
        T acc = 0;
        for (int c = i > 0 ? i - 1 : 0; c < s; ++c)
            acc += e.hr[c * (m + 1) + i] * e.h2[c];
        e.u[i] = acc + (i <= s ? e.col[i] : e.hn) * e.h2[s];
    }
    __syncthreads();
}

// Givens step s from what step_end formed: Hessenberg column s, previous
// rotations, new rotation, residual estimate and the cycle stop decision.  No
// field that other blocks of the same kernel read is changed, except `halt`
// (a wave that sees it set only leaves out rows nothing will use).
template <typename T>
__device__ __forceinline__ void givens_step(int s, int m, GmDev<T> *st, StepEnd<T> &e) {
    const int t = threadIdx.x;
    T *Rs = st->Hraw + (int64_t)s * (m + 1);
    if (t < s) {
        e.cs[t] = st->cs[t];
        e.sn[t] = st->sn[t];
    }
    if (t <= s)
        Rs[t] = e.col[t];
    __syncthreads();
    if (t != 0)
        return;
    const T hn = e.hn;
    Rs[s + 1] = hn;
    T *Hs = st->H + (int64_t)s * (m + 1);
    // previous rotations applied to (h_0s, ..., h_ss, hn); `a` carries entry i
    T a = e.col[0];
    for (int i = 0; i < s; ++i) {
        const T c2 = e.col[i + 1];
        Hs[i] = e.cs[i] * a + e.sn[i] * c2;
        a = -e.sn[i] * a + e.cs[i] * c2;
    }
    const T d = sqrt(a * a + hn * hn);
    if (d == T(0)) {
        st->final_state = ck::BREAKDOWN;
        st->cycle_stop = ck::BREAKDOWN;
        st->halt = 1;
        return;
    }
    const T cj = a / d, sj = hn / d;
    const T gj = st->res[s], g1 = -sj * gj;
    const int iter = st->iter0 + s + 1;
    st->cs[s] = cj;
    st->sn[s] = sj;
    Hs[s] = d;
    Hs[s + 1] = 0;
    st->g[s] = cj * gj;
    st->res[s + 1] = g1;
    st->j = s + 1;
    st->iter = iter;
    const double relres = fabs((double)g1) / st->bnorm;
    st->relres = relres;
    int stop = ck::RUN;
    if (relres <= st->tol)
        stop = ck::CONVERGED;
    else if (hn == T(0))
        stop = ck::BREAKDOWN;
    else if (iter >= st->max_iter)
        stop = ck::BUDGET;
    else if (s + 1 == m)
        stop = ck::FULL;
    st->cycle_stop = stop;
    st->halt = stop != ck::RUN;
}

}  // namespace

template <typename T, int NC>
__global__ __launch_bounds__(ck::kGmThreads) void gm_pass1(int64_t n, int64_t G, int ncols,
                                                const T *__restrict__ V, int64_t ldv,
                                                const T *__restrict__ w,
                                                T *__restrict__ partials, const GmDev<T> *st) {
    if (st->halt)
        return;
    const int64_t b = blockIdx.x;
    T acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        acc[c] = 0;
    for (int64_t i = b * ck::kGmThreads + threadIdx.x; i < n; i += G * ck::kGmThreads) {
        const T wi = w[i];
        T vv[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
            vv[c] = V[clampc(c, ncols) * ldv + i];
        __builtin_amdgcn_sched_barrier(0);   // every load issued before the first use
#pragma unroll
        for (int c = 0; c < NC; ++c)
            acc[c] += vv[c] * wi;
    }
    block_cols<false, T, NC>(acc, T(0), ncols, partials, b, G);
}

template <typename T, int NC>
__global__ __launch_bounds__(ck::kGmThreads) void gm_pass2(int64_t n, int64_t G, int ncols,
                                                const T *__restrict__ V, int64_t ldv,
                                                T *__restrict__ w,
                                                const T *__restrict__ partials1,
                                                T *__restrict__ partials, GmDev<T> *st,
                                                unsigned long long *progress, unsigned seq) {
    __shared__ __align__(16) T h1[NC];
    // Step seq opens its second sweep: the state is the one the steps before
    // it left.  Reported here, where the store to the host's memory is hidden
    // behind the sweep.
    if (blockIdx.x == 0 && threadIdx.x == 0)
        ck::report(progress, st->relres, seq, seq - 1 - (unsigned)st->iter,
                   st->final_state != ck::RUN ? ck::kReportDone
                   : st->halt ? ck::kReportStopped : ck::kReportRun);
    // A halted solve runs no rows (and leaves zero partials, which no later
    // kernel reads): the flag only sets the loop bound, so the loads of the
    // first pass's partials are issued with it rather than after an early exit.
    const int64_t nl = st->halt ? 0 : n;
    sum_cols(ncols, G, partials1, h1);
    __syncthreads();
    if (blockIdx.x == 0 && (int)threadIdx.x < ncols && nl > 0)
        st->h1[threadIdx.x] = h1[threadIdx.x];
    constexpr bool HREG = NC * sizeof(T) <= 256;   // as in gm_pass31
    if ((int)threadIdx.x >= ncols && threadIdx.x < NC)
        h1[threadIdx.x] = 0;
    __syncthreads();
    T h[HREG ? NC : 1], acc[NC], nn = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if constexpr (HREG)
            h[c] = h1[c];
        acc[c] = 0;
    }
    const int64_t b = blockIdx.x;
    for (int64_t i = b * ck::kGmThreads + threadIdx.x; i < nl; i += G * ck::kGmThreads) {
        T vv[NC];
        T wi = w[i];
#pragma unroll
        for (int c = 0; c < NC; ++c)
            vv[c] = V[clampc(c, ncols) * ldv + i];
        __builtin_amdgcn_sched_barrier(0);   // every load issued before the first use
        int o = 0;
        if constexpr (!HREG)
            asm volatile("" : "+v"(o));
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (HREG)
                wi -= h[c] * vv[c];
            else
                wi -= h1[c + o] * vv[c];
        }
        w[i] = wi;
        nn += wi * wi;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            acc[c] += vv[c] * wi;
    }
    block_cols<true, T, NC>(acc, nn, ncols, partials, b, G);
}

// Step j >= 1 opens here: column j holds w' of step j - 1 (after its first
// projection, not yet corrected by h2 nor normalised) and column j + 1 holds
// z = A w'.  One sweep over V_{j-1} forms, in place, v_j = (w' - V_{j-1} h2)
// * inv and A v_j = (z - V_{j-1} u_{0..j-1} - u_j v_j) * inv, and the
// partials of V_j^T A v_j (columns 0..j).  h2, u and inv = 1 / h_{j,j-1} are step
// j - 1's, formed by every block; block G does that step's Givens work.
template <typename T, int NC>
__global__ __launch_bounds__(ck::kGmThreads) void gm_pass31(int64_t n, int64_t G, int j, int m,
                                                 T *__restrict__ V, int64_t ldv,
                                                 const T *__restrict__ partials2,
                                                 T *__restrict__ partials, GmDev<T> *st) {
    __shared__ StepEnd<T> e;
    const int nold = j;   // finished columns 0 .. j-1, read from memory (NC >= j + 1)
    const int halt = st->halt;
    step_end(j - 1, m, G, partials2, st, e);
    if (blockIdx.x == G) {
        if (!halt)
            givens_step(j - 1, m, st, e);
        return;
    }
    // The coefficients of the swept columns stay in registers where there is
    // room for two waves per SIMD (the grid has no more), else they are read
    // from LDS for every row.
    constexpr bool HREG = NC * sizeof(T) <= 256, UREG = NC * sizeof(T) <= 192;
    const T uj = e.u[j];
    const T inv = e.hn > T(0) ? T(1) / e.hn : T(0);
    __syncthreads();
    if ((int)threadIdx.x >= nold && threadIdx.x < NC)
        e.h2[threadIdx.x] = e.u[threadIdx.x] = 0;
    __syncthreads();
    T h2[HREG ? NC : 1], u[UREG ? NC : 1], acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if constexpr (HREG)
            h2[c] = e.h2[c];
        if constexpr (UREG)
            u[c] = e.u[c];
        acc[c] = 0;
    }
    const int64_t nl = halt ? 0 : n;   // as in gm_pass2: no rows once halted
    const int64_t b = blockIdx.x;
    T *wv = V + (int64_t)j * ldv;         // w' in, v_j out
    T *zw = V + (int64_t)(j + 1) * ldv;   // z in, A v_j out
    T accj = 0;
    for (int64_t i = b * ck::kGmThreads + threadIdx.x; i < nl; i += G * ck::kGmThreads) {
        T a = wv[i], zz = zw[i];
        T vv[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
            vv[c] = V[clampc(c, nold) * ldv + i];
        __builtin_amdgcn_sched_barrier(0);   // every load issued before the first use
        int o = 0;
        if constexpr (!UREG)
            asm volatile("" : "+v"(o));   // read for this row: not kept in registers
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (HREG)
                a -= h2[c] * vv[c];
            else
                a -= e.h2[c + o] * vv[c];
            if constexpr (UREG)
                zz -= u[c] * vv[c];
            else
                zz -= e.u[c + o] * vv[c];
        }
        const T vj = a * inv;
        zz -= uj * vj;
        const T wi = zz * inv;
        wv[i] = vj;
        zw[i] = wi;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            acc[c] += vv[c] * wi;
        accj += vj * wi;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (c == j)
            acc[c] = accj;   // column j is v_j itself (the loop's acc[j] saw a reloaded column)
    block_cols<false, T, NC>(acc, T(0), j + 1, partials, b, G);
}

// Cycle start: partials of ||r||^2 (FP64)
template <typename T>
__global__ __launch_bounds__(256) void gm_start_norm(int64_t n, int64_t G,
                                                     const double *__restrict__ r,
                                                     double *__restrict__ partials,
                                                     const GmDev<T> *st) {
    __shared__ double lds[4];
    if (st->final_state != ck::RUN)
        return;
    const int64_t b = blockIdx.x;
    double s = 0;
    for (int64_t i = b * 256 + threadIdx.x; i < n; i += G * 256)
        s += r[i] * r[i];
    s = ck::block_sum(s, lds);
    if (threadIdx.x == 0)
        partials[b] = s;
}

// beta = ||r||, true-residual convergence test, g = beta e1
template <typename T>
__global__ __launch_bounds__(256) void gm_start_finish(int64_t G,
                                                       const double *__restrict__ partials,
                                                       GmDev<T> *st) {
    __shared__ double lds[4];
    if (st->final_state != ck::RUN)
        return;
    const double tot = ck::sum_partials(partials, G, lds);
    if (threadIdx.x != 0)
        return;
    const double beta = sqrt(tot);
    st->beta = beta;
    st->relres = beta / st->bnorm;
    if (st->relres <= st->tol) {
        st->final_state = ck::CONVERGED;
        st->halt = 1;
        return;
    }
    if (st->iter >= st->max_iter) {
        st->final_state = ck::BUDGET;
        st->halt = 1;
        return;
    }
    st->inv_beta = 1.0 / beta;
    st->j = 0;
    st->cycle_stop = ck::RUN;
    st->halt = 0;
    st->cycles += 1;
    st->iter0 = st->iter;
    st->res[0] = (T)beta;
}

template <typename T>
__global__ __launch_bounds__(256) void gm_start_v0(int64_t n, T *__restrict__ v0,
                                                   const double *__restrict__ r,
                                                   const GmDev<T> *st) {
    if (st->halt)
        return;
    const double inv = st->inv_beta;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * 256)
        v0[i] = (T)(r[i] * inv);
}

// Cycle end: the Givens work of the last step, unless the cycle has stopped
// before (its work was done by the next step's pass 3+1 then), and the back
// substitution R y = g over the k = j columns formed.  The columns are copied to LDS; lane i of one wave then holds g_i, and for t = k -
// 1 .. 0 the wave takes y_t = g_t / R_tt from lane t and subtracts y_t times
// column t.  A chain of k divisions (one thread reading R from memory took
// 38 us for 30 FP64 columns, each subtraction waiting for its loads; 7 us now).
template <typename T>
__global__ __launch_bounds__(ck::kGmThreads) void gm_solve_y(int64_t G, const T *__restrict__ partials2,
                                                  GmDev<T> *st) {
    __shared__ StepEnd<T> e;
    if (st->final_state != ck::RUN)
        return;
    const int tid = threadIdx.x, m = st->m, ld = m + 1;
    if (!st->halt) {
        const int s = st->j;   // every thread reads it before thread 0 moves it on
        step_end(s, m, G, partials2, st, e);
        givens_step(s, m, st, e);
        __threadfence_block();
        __syncthreads();
        if (st->final_state != ck::RUN)
            return;
    }
    T *R = e.hr;
    const int k = st->j;
    T g = tid < k ? st->g[tid] : T(0);
    for (int t = tid; t < k * ld; t += ck::kGmThreads)
        R[t] = st->H[t];
    __syncthreads();
    if (tid >= 64)
        return;
    T y = 0;
    for (int t = k - 1; t >= 0; --t) {
        const T yt = __shfl(g / R[t * ld + t], t, 64);
        if (tid < t)
            g -= R[t * ld + tid] * yt;
        if (tid == t)
            y = yt;
    }
    if (tid < k)
        st->y[tid] = y;
}

// x += V_k y, accumulated in FP64 (the basis may be FP32).
template <typename T>
__global__ __launch_bounds__(256) void gm_update_x(int64_t n, double *__restrict__ x,
                                                   const T *__restrict__ V, int64_t ldv,
                                                   const GmDev<T> *st) {
    __shared__ double ys[ck::kMaxRestart];
    if (st->final_state != ck::RUN)
        return;
    const int k = st->j;
    for (int c = threadIdx.x; c < k; c += 256)
        ys[c] = (double)st->y[c];
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * 256) {
        double acc = 0;
        for (int c = 0; c < k; ++c)
            acc += ys[c] * (double)V[c * ldv + i];
        x[i] += acc;
    }
}

namespace ck {

// Blocks of the Gram-Schmidt passes: as few rows per thread as kGmMaxBlocks
// allow, the same for every block.
int64_t gm_blocks(int64_t n) {
    const int64_t rows = std::max<int64_t>(ceil_div(n, (int64_t)kGmThreads * kGmMaxBlocks), 1);
    return std::max<int64_t>(ceil_div(n, kGmThreads * rows), 1);
}

// Values of the two partial arrays: one column per basis column and ||w'||^2.
static int64_t gm_partials1() { return (int64_t)(kMaxRestart + 2) * kGmMaxBlocks; }
int64_t gm_partials() { return 2 * gm_partials1(); }

static int64_t gm_stream_grid(int64_t n) {
    int64_t g = ceil_div(n, 1024);
    if (g < 1)
        g = 1;
    return g < 8192 ? g : 8192;
}

template <typename T>
ck_status launch_gm_cycle_start(int64_t n, const double *r64, T *v0, double *partials64,
                                GmDev<T> *st, hipStream_t s) {
    const int64_t G = dot_blocks<double>(n);
    hipLaunchKernelGGL((gm_start_norm<T>), dim3(G), dim3(256), 0, s, n, G, r64, partials64, st);
    hipLaunchKernelGGL((gm_start_finish<T>), dim3(1), dim3(256), 0, s, G, partials64, st);
    hipLaunchKernelGGL((gm_start_v0<T>), dim3(gm_stream_grid(n)), dim3(256), 0, s, n, v0, r64, st);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

template <typename T, int NC>
static void arnoldi_nc(int64_t n, int64_t G, int j, T *V, int64_t ldv, T *w, T *partials,
                       int m, GmDev<T> *st, unsigned long long *progress, unsigned seq,
                       hipStream_t s) {
    const int ncols = j + 1;
    T *partials2 = partials + gm_partials1();
    if (j == 0)
        hipLaunchKernelGGL((gm_pass1<T, NC>), dim3(G), dim3(kGmThreads), 0, s, n, G, ncols, V, ldv, w,
                           partials, st);
    else
        hipLaunchKernelGGL((gm_pass31<T, NC>), dim3(G + 1), dim3(kGmThreads), 0, s, n, G, j, m, V, ldv,
                           partials2, partials, st);
    hipLaunchKernelGGL((gm_pass2<T, NC>), dim3(G), dim3(kGmThreads), 0, s, n, G, ncols, V, ldv, w,
                       partials, partials2, st, progress, seq);
}

// Step j after the SpMV of column j into column j+1 (column j is v_0 for
// j = 0, else the previous step's w', see the file comment): ends with
// w' of step j in column j+1 and the partials of its second pass.  partials:
// gm_partials() values, the first pass's, then the second's.
template <typename T>
ck_status launch_gm_arnoldi(int64_t n, int j, int m, T *V, int64_t ldv, T *partials, GmDev<T> *st,
                            unsigned long long *progress, unsigned seq, hipStream_t s) {
    const int64_t G = gm_blocks(n);
    const int ncols = j + 1;
    T *w = V + (int64_t)(j + 1) * ldv;
    if (ncols <= 8)
        arnoldi_nc<T, 8>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else if (ncols <= 16)
        arnoldi_nc<T, 16>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else if (ncols <= 24)
        arnoldi_nc<T, 24>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else if (ncols <= 32)
        arnoldi_nc<T, 32>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else if (ncols <= 40)
        arnoldi_nc<T, 40>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else if (ncols <= 48)
        arnoldi_nc<T, 48>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else if (ncols <= 56)
        arnoldi_nc<T, 56>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else if (ncols <= 64)
        arnoldi_nc<T, 64>(n, G, j, V, ldv, w, partials, m, st, progress, seq, s);
    else
        return fail(CK_E_INVALID, "restart length above %d", kMaxRestart);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

template <typename T>
ck_status launch_gm_cycle_end(int64_t n, double *x, const T *V, int64_t ldv, const T *partials,
                              GmDev<T> *st, hipStream_t s) {
    hipLaunchKernelGGL((gm_solve_y<T>), dim3(1), dim3(kGmThreads), 0, s, gm_blocks(n),
                       partials + gm_partials1(), st);
    hipLaunchKernelGGL((gm_update_x<T>), dim3(gm_stream_grid(n)), dim3(256), 0, s, n, x, V, ldv,
                       st);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

#define CK_GM_INST(T)                                                                          \
    template ck_status launch_gm_cycle_start<T>(int64_t, const double *, T *, double *,        \
                                                GmDev<T> *, hipStream_t);                      \
    template ck_status launch_gm_arnoldi<T>(int64_t, int, int, T *, int64_t, T *, GmDev<T> *,  \
                                            unsigned long long *, unsigned, hipStream_t);      \
    template ck_status launch_gm_cycle_end<T>(int64_t, double *, const T *, int64_t,           \
                                              const T *, GmDev<T> *, hipStream_t);
CK_GM_INST(double)
CK_GM_INST(float)

}  // namespace ck
