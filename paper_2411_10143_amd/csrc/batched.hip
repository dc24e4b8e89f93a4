// Batched small-system solver for the request loop: one workgroup per system
// ("slot"), a bounded number of iterations per launch.  Between launches the
// host retires finished slots and admits new requests, so requests that
// arrive while others run join the next launch (continuous batching).
//
// Each slot runs FP64 iterative refinement around an FP32 inner solve:
//   outer : r = b - A x (FP64 values, FP64 arithmetic), beta = ||r||, test
//           beta/||b|| <= tol; otherwise the inner system A d = r/beta
//   inner : CG (symmetric) until ||r_in|| <= max(tol ||b||/beta, 1e-5), or
//           one GMRES(m) cycle (classical Gram-Schmidt twice, Givens), on
//           the FP32 values with FP32 vectors and FP32 accumulation
//   update: x += beta * d  (FP64)
// With FP64 inner vectors the same loop is plain CG (inner target
// tol ||b||/beta, then the true-residual check) or plain restarted GMRES(m);
// single solves use it, with 1024 threads, for systems too small to fill the
// GPU, where one workgroup running the whole solve beats a launch per step
// (slotrule.hpp).
// Every reduction stays inside the workgroup in a fixed order, so a slot's
// bits do not depend on which other slots share the launch.
#include <algorithm>

#include "batched.hpp"

namespace {

// sum over the workgroup of BS threads, returned to every thread (fixed order)
template <int BS, typename T>
__device__ __forceinline__ T wg_sum(T v, T *lds) {
    v = ck::wave_sum_last(v);   // valid in lane 63
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63)
        lds[w] = v;
    __syncthreads();
    T r = (lds[0] + lds[1]) + (lds[2] + lds[3]);
#pragma unroll
    for (int t = 4; t < BS / 64; t += 4)
        r += (lds[t] + lds[t + 1]) + (lds[t + 2] + lds[t + 3]);
    __syncthreads();
    return r;
}

// A small system's matrix and vectors sit in L2, so its products and vector
// sweeps are bound by load latency, not bandwidth.  Every loop below issues
// its loads unconditionally (indices clamped into range) and applies the
// bounds test only to the arithmetic and the stores; a scheduling barrier
// after each group of loads stops the compiler from sinking a load next to
// its use (which it does to save registers), so the group is in flight
// together.  The summation order is the plain one.
constexpr int kVec = 4;   // vector elements in flight per thread

// A value or pointer that is the same in every lane, in scalar registers, so
// that a load from p[i] takes a scalar base and a 32-bit lane offset.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T *uni(T *p) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return (T *)(((unsigned long long)hi << 32) | lo);
}

// This thread's index, as a value the compiler cannot trace: what a loop
// derives from it (clamped row indices, LDS addresses, bounds tests) is then
// formed there, instead of being kept for the whole solve in registers that
// at 1024 threads do not suffice.
__device__ __forceinline__ int thread_index() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// rows in flight per thread in the workgroup SpMV
constexpr int kRowsInFlight = 4;

// Sum over the L lanes of a row (L a run-time power of two, uniform over
// the workgroup) by DPP moves, valid in lane L - 1 of each row's lanes.
template <typename T>
__device__ __forceinline__ T lanes_sum(T a, int L) {
    switch (L) {
    case 1: return a;
    case 2: return ck::group_sum_last<2>(a);
    case 4: return ck::group_sum_last<4>(a);
    case 8: return ck::group_sum_last<8>(a);
    case 16: return ck::group_sum_last<16>(a);
    case 32: return ck::group_sum_last<32>(a);
    default: return ck::group_sum_last<64>(a);
    }
}

// y[i] = s1 * (A x)[i] + s0 * z[i] with L lanes per row (runtime power of
// two).  Per row the lanes sum entries start + lane, start + lane + L, ...
// in order, then a DPP sum over the L lanes.
template <int BS, typename TV, typename TX, typename TA>
__device__ __forceinline__ void wg_spmv(int n, int L, const int *__restrict__ rp,
                                        const int *__restrict__ col,
                                        const TV *__restrict__ val, const TX *__restrict__ x,
                                        TA s1, TA s0, const TA *__restrict__ z,
                                        TA *__restrict__ y) {
    constexpr int U = kRowsInFlight;
    rp = uni(rp);
    col = uni(col);
    val = uni(val);
    const int tid = thread_index();
    const int lg = 31 - __clz(L);
    const int lane = tid & (L - 1), sub = tid >> lg;
    const int rpp = BS >> lg;
    for (int r0 = 0; r0 < n; r0 += U * rpp) {
        int kb[U], ke[U];
        TA acc[U];
        int trips = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = min(r0 + u * rpp + sub, n - 1);
            kb[u] = rp[(unsigned)row] + lane;
            ke[u] = r0 + u * rpp + sub < n ? rp[(unsigned)row + 1] : 0;
            acc[u] = 0;
            trips = max(trips, (ke[u] - kb[u] + L - 1) >> lg);
        }
        // trips > 0 means some row here has entries, so entry 0 exists and
        // serves as the in-range index of finished rows
        for (int t = 0; t < trips; ++t) {
            int cc[U];
            TV vv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = kb[u] + (t << lg);
                const int kk = k < ke[u] ? k : 0;
                cc[u] = col[(unsigned)kk];
                vv[u] = val[(unsigned)kk];
            }
            TX xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                xv[u] = x[cc[u]];
            __builtin_amdgcn_sched_barrier(0);   // all gathers in flight before the first use
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (kb[u] + (t << lg) < ke[u])
                    acc[u] += (TA)vv[u] * (TA)xv[u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const TA a = lanes_sum(acc[u], L);   // valid in lane L - 1 of the row's lanes
            const int row = r0 + u * rpp + sub;
            if (lane == L - 1 && row < n)
                y[row] = z ? s1 * a + s0 * z[row] : s1 * a;
        }
    }
}

template <typename T>
__device__ __forceinline__ T *wsp(ck::BSlot *s, int which) {
    return (T *)s->work + (int64_t)which * s->ld;
}

// ---- inner loops of systems whose vectors fit the workgroup -------------------
// Rows per thread of the inner loops below: thread t holds rows t, t + BS, ...
// of the inner vectors in registers, and the vector being multiplied sits in
// LDS, so between products nothing is read from memory but the matrix (and
// the basis).
template <int BS>
constexpr int resident_rows() { return BS >= 1024 ? 8 : 4; }

template <typename T, int BS>
struct SlotLds {
    T p[BS * resident_rows<BS>() + 1];   // the vector multiplied, then one zero
    T q[BS * resident_rows<BS>()];       // its product
    T red[2][BS / 64];
    T wred[BS / 64][ck::kBMaxM + 1];
    T h[ck::kBMaxM + 1], hsum[ck::kBMaxM + 1];
    T cs[ck::kBMaxM], sn[ck::kBMaxM];
    T inv;
    int stop;
    int base[BS * resident_rows<BS>() / 64 + 1];   // slice offsets of the slot copy
};

// wg_sum with one barrier: successive calls alternate between two buffers, so
// a buffer is rewritten only after the barrier of the call in between, which
// every thread reaches after reading it.
template <int BS, typename T>
__device__ __forceinline__ T wg_sum_alt(T v, T (&red)[2][BS / 64], int &parity) {
    T *buf = red[parity];
    parity ^= 1;
    v = ck::wave_sum_last(v);   // valid in lane 63
    if ((threadIdx.x & 63) == 63)
        buf[threadIdx.x >> 6] = v;
    __syncthreads();
    T r = (buf[0] + buf[1]) + (buf[2] + buf[3]);
#pragma unroll
    for (int t = 4; t < BS / 64; t += 4)
        r += (buf[t] + buf[t + 1]) + (buf[t + 2] + buf[t + 3]);
    return r;
}

// lds.q = A lds.p from the slot copy: a wave takes slices w, w + BS / 64, ...,
// a lane one row, its entries summed in ascending order (the bits of wg_spmv
// with one lane per row).  The next eight entries (FP64: four) of the slice,
// or of the wave's next slice, are loaded while those before them are gathered
// and multiplied.  One
// workgroup's products are bound by the instructions it issues: a slot costs
// two loads, an LDS gather and two vector instructions here, where lanes
// sharing CSR rows need about 25 an entry (n = 7,000, 19 entries a row, mixed
// GMRES: 82 us a step before, 45 with the copy).
template <typename T, int BS>
__device__ __forceinline__ void slot_product(int n, const ck::SlotCopy &c, SlotLds<T, BS> &lds) {
    constexpr int U = sizeof(T) == 4 ? 8 : 4, NW = BS / 64;
    const int tid = thread_index(), lane = tid & 63;
    const unsigned short *col = uni(c.col), *perm = uni(c.perm);
    const T *val = uni((const T *)c.val);
    const int slices = (n + 63) / 64;
    T v[U];
    unsigned short cc[U];
    int row = 0, nrow = 0;
    // entries t .. t + 7 (as far as there are) of the lane's row of slots k0 ..
    // k0 + 64 K - 1, K >= 1
    auto fetch = [&](int k0, int K, int t) {
        const unsigned short *cp = col + k0;
        const T *vp = val + k0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (t + u < K) {   // uniform over the wave
                cc[u] = (cp + 64 * (t + u))[(unsigned)lane];
                v[u] = (vp + 64 * (t + u))[(unsigned)lane];
            }
    };
    int sl = uni(tid >> 6);
    int k0 = 0, K = 0;
    auto open = [&](int s) {   // slice s: its extent, the lane's row, its first entries
        k0 = uni(lds.base[s]);
        K = (uni(lds.base[s + 1]) - k0) >> 6;
        nrow = perm[(unsigned)min(s * 64 + lane, n - 1)];
        if (K > 0)
            fetch(k0, K, 0);
    };
    if (sl < slices)
        open(sl);
    while (sl < slices) {
        const int at = sl * 64 + lane, K0 = K, first = k0;
        row = nrow;
        sl += NW;
        T acc = 0;
        if (K0 == 0 && sl < slices)
            open(sl);
        for (int t = 0; t < K0; t += U) {
            T vv[U], g[U];
            const int left = K0 - t;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u < left) {
                    vv[u] = v[u];
                    g[u] = lds.p[cc[u]];
                }
            if (t + U < K0)
                fetch(first, K0, t + U);
            else if (sl < slices)
                open(sl);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u < left)
                    acc += vv[u] * g[u];
        }
        if (at < n)
            lds.q[row] = acc;
    }
}

// lds.q = A lds.p in the inner type, from the slot copy or (also where there was no
// room for it; with one lane the sums are the same) from the CSR arrays.  Each form
// has a loop over the steps of its own: with both in one, steps on the copy took
// 0.75 us more (FP64, registers).
template <bool SELL, typename T, int BS>
__device__ __forceinline__ void inner_product(const ck::BSlot *s, int n, const T *val,
                                              SlotLds<T, BS> &lds) {
    if constexpr (SELL)
        slot_product<T, BS>(n, s->sell, lds);
    else
        wg_spmv<BS, T, T, T>(n, uni(s->inner_lanes), s->rp, s->col, val, lds.p, T(1), T(0),
                             (const T *)nullptr, lds.q);
}

// CG steps of a slot in phase B_INNER until it leaves the phase or `budget`
// steps are done; returns the steps, and the new phase in *phase.
template <bool SELL, typename T, int BS>
__device__ __forceinline__ int slot_cg(ck::BSlot *s, int budget, SlotLds<T, BS> &lds, int *phase) {
    constexpr int R = resident_rows<BS>();
    const int tid = thread_index(), n = uni(s->n);
    T *r = wsp<T>(s, 0), *p = wsp<T>(s, 1), *d = wsp<T>(s, 3);
    const T *val = sizeof(T) == 4 ? (const T *)s->val32 : (const T *)s->val64;
    T rr[R], pr[R], dr[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int i = tid + u * BS, ii = min(i, n - 1);
        rr[u] = r[ii];
        pr[u] = p[ii];
        dr[u] = d[ii];
        if (i >= n)
            rr[u] = pr[u] = dr[u] = 0;
        else
            lds.p[i] = pr[u];
    }
    if (tid == 0)
        lds.p[n] = 0;
    if (SELL && tid <= (n + 63) / 64)
        lds.base[tid] = s->sell.base[tid];
    T rho = (T)s->rho;
    int inner = s->inner_iter, iter = s->iter, parity = 0, steps = 0, next = ck::B_INNER;
    const int inner_cap = s->inner_cap, max_iter = s->max_iter;
    const double tol2 = s->inner_tol * s->inner_tol;
    bool broken = false;
    while (steps < budget && next == ck::B_INNER) {
        const int tid = thread_index();
        ++steps;
        __syncthreads();   // lds.p is complete
        inner_product<SELL, T, BS>(s, n, val, lds);
        __syncthreads();
        T q[R], pq = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int i = tid + u * BS;
            q[u] = i < n ? lds.q[i] : T(0);
            pq += pr[u] * q[u];
        }
        const T sigma = wg_sum_alt<BS>(pq, lds.red, parity);
        if (!(sigma > T(0))) {
            broken = inner == 0;
            next = broken ? ck::B_DONE : ck::B_UPDATE;
            break;
        }
        const T alpha = rho / sigma;
        T rn = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) {
            dr[u] += alpha * pr[u];
            rr[u] -= alpha * q[u];
            rn += rr[u] * rr[u];
        }
        const T rho_new = wg_sum_alt<BS>(rn, lds.red, parity);
        ++inner;
        const bool stop = (double)rho_new <= tol2 || inner >= inner_cap ||
                          iter + 1 >= max_iter;
        ++iter;
        const T beta = rho_new / rho;
        rho = rho_new;
        if (stop) {
            next = ck::B_UPDATE;
        } else {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int i = tid + u * BS;
                pr[u] = rr[u] + beta * pr[u];
                if (i < n)
                    lds.p[i] = pr[u];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int i = tid + u * BS;
        if (i < n) {
            r[i] = rr[u];
            p[i] = pr[u];
            d[i] = dr[u];
        }
    }
    if (tid == 0) {
        s->rho = (double)rho;
        s->inner_iter = inner;
        s->iter = iter;
        if (broken)
            s->status = ck::BREAKDOWN;
    }
    *phase = next;
    __syncthreads();
    return steps;
}

// C basis columns g .. g + C - 1 of the thread's rows: DOT adds V_c . w to
// lds.wred, else w -= h_c V_c.  The columns of U rows are in flight together.
template <int C, bool DOT, typename T, int BS>
__device__ __forceinline__ void basis_columns(int n, int g, const T *__restrict__ V, int64_t ld,
                                              T (&w)[resident_rows<BS>()], SlotLds<T, BS> &lds) {
    constexpr int R = resident_rows<BS>();
    constexpr int most = sizeof(T) == 4 ? 32 : 16;   // loads in flight
    constexpr int U = most / C < R ? most / C : R;
    const int tid = thread_index();
    T acc[C], h[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        acc[c] = 0;
        h[c] = DOT ? T(0) : lds.h[g + c];
    }
#pragma unroll
    for (int u0 = 0; u0 < R; u0 += U) {
        if (u0 * BS < n) {
            T vv[U][C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T *Vc = V + (int64_t)(g + c) * ld;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    vv[u][c] = Vc[(unsigned)min(tid + (u0 + u) * BS, n - 1)];
            }
            __builtin_amdgcn_sched_barrier(0);   // the loads are in flight together
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if (DOT)
                        acc[c] += vv[u][c] * w[u0 + u];   // w is 0 past the last row
                    else
                        w[u0 + u] -= h[c] * vv[u][c];
                }
        }
    }
    if (DOT) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const T v = ck::wave_sum_last(acc[c]);   // valid in lane 63
            if ((tid & 63) == 63)
                lds.wred[tid >> 6][g + c] = v;
        }
    }
}

// One sweep over basis columns 0 .. j: groups of eight, then four, two, one.
template <bool DOT, typename T, int BS>
__device__ __forceinline__ void basis_sweep(int n, int j, const T *__restrict__ V, int64_t ld,
                                            T (&w)[resident_rows<BS>()], SlotLds<T, BS> &lds) {
    constexpr int R = resident_rows<BS>();
    const int cols = j + 1;
    int g = 0;
    for (; g + 8 <= cols; g += 8)
        basis_columns<8, DOT, T, BS>(n, g, V, ld, w, lds);
    if (cols & 4) {
        basis_columns<4, DOT, T, BS>(n, g, V, ld, w, lds);
        g += 4;
    }
    if (cols & 2) {
        basis_columns<2, DOT, T, BS>(n, g, V, ld, w, lds);
        g += 2;
    }
    if (cols & 1)
        basis_columns<1, DOT, T, BS>(n, g, V, ld, w, lds);
    if (!DOT) {
        const int tid = thread_index();
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (tid + u * BS >= n)
                w[u] = 0;
    }
}

// Arnoldi steps (classical Gram-Schmidt twice, Givens) of a slot in phase
// B_INNER, as slot_cg.
template <bool SELL, typename T, int BS>
__device__ __forceinline__ int slot_gmres(ck::BSlot *s, int budget, SlotLds<T, BS> &lds, int *phase) {
    constexpr int R = resident_rows<BS>(), NW = BS / 64;
    const int tid = thread_index(), n = uni(s->n), m = uni(s->m);
    const int64_t ld = uni((int)s->ld);
    T *V = uni(wsp<T>(s, 0));
    const T *val = sizeof(T) == 4 ? (const T *)s->val32 : (const T *)s->val64;
    int j = uni(s->j), iter = s->iter, parity = 0, steps = 0, next = ck::B_INNER;
    const int max_iter = s->max_iter;
    const double beta = s->beta, bnorm = s->bnorm, tol = s->tol;
    for (int u = 0; u < R; ++u) {
        const int i = tid + u * BS;
        if (i < n)
            lds.p[i] = V[(int64_t)j * ld + i];
    }
    if (tid == 0)
        lds.p[n] = 0;
    if (SELL && tid <= (n + 63) / 64)
        lds.base[tid] = s->sell.base[tid];
    if (tid < j) {
        lds.cs[tid] = (T)s->cs[tid];
        lds.sn[tid] = (T)s->sn[tid];
    }
    T gj = (T)s->g[j];   // every thread; thread 0 uses it
    while (steps < budget && next == ck::B_INNER) {
        const int tid = thread_index();
        ++steps;
        __syncthreads();   // lds.p is complete
        inner_product<SELL, T, BS>(s, n, val, lds);
        __syncthreads();
        T w[R];
#pragma unroll
        for (int u = 0; u < R; ++u)
            w[u] = tid + u * BS < n ? lds.q[tid + u * BS] : T(0);
        for (int pass = 0; pass < 2; ++pass) {
            basis_sweep<true, T, BS>(n, j, V, ld, w, lds);
            __syncthreads();
            if (tid <= j) {
                T h = 0;
#pragma unroll
                for (int t = 0; t < NW; t += 4)
                    h += (lds.wred[t][tid] + lds.wred[t + 1][tid]) +
                         (lds.wred[t + 2][tid] + lds.wred[t + 3][tid]);
                lds.h[tid] = h;
                lds.hsum[tid] = pass == 0 ? h : lds.hsum[tid] + h;
            }
            __syncthreads();
            basis_sweep<false, T, BS>(n, j, V, ld, w, lds);
        }
        T nn = 0;
#pragma unroll
        for (int u = 0; u < R; ++u)
            nn += w[u] * w[u];
        const T hn = sqrt(wg_sum_alt<BS>(nn, lds.red, parity));
        if (tid == 0) {
            // Hessenberg column j in the inner precision (stored as double)
            double *Hj = s->H + j * (m + 1);
            T a = lds.hsum[0];
            for (int i = 0; i < j; ++i) {
                const T c2 = lds.hsum[i + 1], ci = lds.cs[i], si = lds.sn[i];
                Hj[i] = (double)(ci * a + si * c2);
                a = -si * a + ci * c2;
            }
            const T dd = sqrt(a * a + hn * hn);
            int stop = 0;
            if (dd == T(0)) {
                stop = 2;           // singular least-squares problem
            } else {
                const T cj = a / dd, sj = hn / dd, g1 = -sj * gj;
                lds.cs[j] = cj;
                lds.sn[j] = sj;
                s->cs[j] = (double)cj;
                s->sn[j] = (double)sj;
                Hj[j] = (double)dd;
                Hj[j + 1] = 0;
                s->g[j + 1] = (double)g1;
                s->g[j] = (double)(cj * gj);
                gj = g1;
                const double est = fabs((double)g1) * beta / bnorm;
                if (est <= tol || hn == T(0) || j + 1 == m || iter + 1 >= max_iter)
                    stop = 1;
            }
            lds.stop = stop;
            lds.inv = hn > T(0) ? T(1) / hn : T(0);
        }
        __syncthreads();
        const int stop = uni(lds.stop);
        if (stop == 2) {
            next = j == 0 ? ck::B_DONE : ck::B_UPDATE;
        } else {
            ++j;
            ++iter;
            if (stop == 1) {
                next = ck::B_UPDATE;
            } else {
                const T inv = lds.inv;
                T *v = V + (int64_t)j * ld;
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    const int i = tid + u * BS;
                    if (i < n) {
                        v[i] = w[u] * inv;
                        lds.p[i] = w[u] * inv;
                    }
                }
            }
        }
    }
    if (tid == 0) {
        s->j = j;
        s->iter = iter;
        if (next == ck::B_DONE)
            s->status = ck::BREAKDOWN;
    }
    *phase = next;
    __syncthreads();
    return steps;
}

}  // namespace

// Slot `which` advances by up to `budget` steps on BS threads.
template <typename T, int BS>
__device__ __forceinline__ void run_slot(ck::BSlot *slots, ck::BStat *stat, int which,
                                         int budget, SlotLds<T, BS> &resident) {
    constexpr int NW = BS / 64;
    auto &hcol = resident.h, &hacc = resident.hsum;
    auto &wred = resident.wred;
    __shared__ T lds[NW];
    __shared__ double lds64[NW];
    ck::BSlot *s = slots + which;
    const int tid = threadIdx.x;
    const int n = uni(s->n), L = uni(s->lanes);
    const bool fits = n <= BS * resident_rows<BS>();
    int phase = s->phase;
    if (phase == ck::B_DONE)
        return;
    if (s->bnorm < 0) {   // first launch of this request: ||b||, x0 = 0
        double q = 0;
        for (int i = tid; i < n; i += BS) {
            q += s->b[i] * s->b[i];
            if (!s->keep_x0)
                s->x[i] = 0.0;
        }
        const double bn = sqrt(wg_sum<BS>(q, lds64));
        if (tid == 0)
            s->bnorm = bn;
        __syncthreads();
        if (bn == 0.0) {   // b = 0: x = 0 is the solution
            for (int i = tid; i < n; i += BS)
                s->x[i] = 0.0;
            phase = ck::B_DONE;
            if (tid == 0) {
                s->status = ck::CONVERGED;
                s->relres = 0.0;
            }
        }
    }
    int steps = 0;
    while (steps < budget && phase != ck::B_DONE) {
        const int tid = thread_index();
        if (phase == ck::B_INNER && fits) {
            const int left = budget - steps;
            const bool sell = s->sell.base != nullptr;
            if (s->kind == ck::B_CG)
                steps += sell ? slot_cg<true, T, BS>(s, left, resident, &phase)
                              : slot_cg<false, T, BS>(s, left, resident, &phase);
            else
                steps += sell ? slot_gmres<true, T, BS>(s, left, resident, &phase)
                              : slot_gmres<false, T, BS>(s, left, resident, &phase);
            continue;
        }
        ++steps;
        if (phase == ck::B_OUTER) {
            // r = b - A x in FP64; beta = ||r||
            wg_spmv<BS, double, double, double>(n, L, s->rp, s->col, s->val64, s->x, -1.0, 1.0, s->b,
                                            s->r64);
            __syncthreads();
            double q = 0;
            const double *r64 = s->r64;
            for (int i0 = tid; i0 < n; i0 += kVec * BS) {
                double rv[kVec];
#pragma unroll
                for (int u = 0; u < kVec; ++u)
                    rv[u] = r64[min(i0 + u * BS, n - 1)];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kVec; ++u)
                    if (i0 + u * BS < n)
                        q += rv[u] * rv[u];
            }
            const double beta = sqrt(wg_sum<BS>(q, lds64));
            const double rel = beta / s->bnorm;
            if (tid == 0) {
                s->relres = rel;
                s->beta = beta;
            }
            if (rel <= s->tol) {
                phase = ck::B_DONE;
                if (tid == 0)
                    s->status = ck::CONVERGED;
                break;
            }
            if (s->iter >= s->max_iter) {
                phase = ck::B_DONE;
                if (tid == 0)
                    s->status = ck::BUDGET;
                break;
            }
            const double inv = 1.0 / beta;
            if (s->kind == ck::B_CG) {
                T *r = wsp<T>(s, 0), *p = wsp<T>(s, 1), *d = wsp<T>(s, 3);
                T rr = 0;
                for (int i = tid; i < n; i += BS) {
                    const T ri = (T)(s->r64[i] * inv);
                    r[i] = ri;
                    p[i] = ri;
                    d[i] = 0;
                    rr += ri * ri;
                }
                rr = wg_sum<BS>(rr, lds);
                if (tid == 0) {
                    s->rho = (double)rr;
                    // FP32 inner solves stop at 1e-5 (their attainable
                    // accuracy); FP64 inner solves go to the outer target
                    s->inner_tol = fmax(s->tol * s->bnorm / beta, sizeof(T) == 4 ? 1e-5 : 0.0);
                    s->inner_iter = 0;
                }
            } else {
                T *v0 = wsp<T>(s, 0);
                for (int i = tid; i < n; i += BS)
                    v0[i] = (T)(s->r64[i] * inv);
                if (tid == 0) {
                    s->j = 0;
                    s->g[0] = 1;
                    for (int t = 1; t <= s->m; ++t)
                        s->g[t] = 0;
                }
            }
            if (tid == 0)
                s->outer += 1;
            phase = ck::B_INNER;
            __syncthreads();
            continue;
        }
        if (phase == ck::B_INNER && s->kind == ck::B_CG) {
            T *r = wsp<T>(s, 0), *p = wsp<T>(s, 1), *q = wsp<T>(s, 2), *d = wsp<T>(s, 3);
            const T *val = sizeof(T) == 4 ? (const T *)s->val32 : (const T *)s->val64;
            wg_spmv<BS, T, T, T>(n, L, s->rp, s->col, val, p, T(1), T(0), (const T *)nullptr, q);
            __syncthreads();
            T pq = 0;
            for (int i0 = tid; i0 < n; i0 += kVec * BS) {
                T pv[kVec], qv[kVec];
#pragma unroll
                for (int u = 0; u < kVec; ++u) {
                    const int i = min(i0 + u * BS, n - 1);
                    pv[u] = p[i];
                    qv[u] = q[i];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kVec; ++u)
                    if (i0 + u * BS < n)
                        pq += pv[u] * qv[u];
            }
            const T sigma = wg_sum<BS>(pq, lds);
            if (!(sigma > T(0))) {
                phase = s->inner_iter == 0 ? ck::B_DONE : ck::B_UPDATE;
                if (phase == ck::B_DONE && tid == 0)
                    s->status = ck::BREAKDOWN;
                __syncthreads();
                continue;
            }
            const T rho = (T)s->rho;
            const T alpha = rho / sigma;
            T rr = 0;
            for (int i0 = tid; i0 < n; i0 += kVec * BS) {
                T dv[kVec], pv[kVec], rv[kVec], qv[kVec];
#pragma unroll
                for (int u = 0; u < kVec; ++u) {
                    const int i = min(i0 + u * BS, n - 1);
                    dv[u] = d[i];
                    pv[u] = p[i];
                    rv[u] = r[i];
                    qv[u] = q[i];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kVec; ++u) {
                    const int i = i0 + u * BS;
                    if (i < n) {
                        d[i] = dv[u] + alpha * pv[u];
                        const T ri = rv[u] - alpha * qv[u];
                        r[i] = ri;
                        rr += ri * ri;
                    }
                }
            }
            const T rho_new = wg_sum<BS>(rr, lds);
            const int it = s->inner_iter + 1;
            const bool stop = sqrt((double)rho_new) <= s->inner_tol || it >= s->inner_cap ||
                              s->iter + 1 >= s->max_iter;
            const T bcg = rho_new / rho;
            if (!stop)
                for (int i0 = tid; i0 < n; i0 += kVec * BS) {
                    T rv[kVec], pv[kVec];
#pragma unroll
                    for (int u = 0; u < kVec; ++u) {
                        const int i = min(i0 + u * BS, n - 1);
                        rv[u] = r[i];
                        pv[u] = p[i];
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < kVec; ++u)
                        if (i0 + u * BS < n)
                            p[i0 + u * BS] = rv[u] + bcg * pv[u];
                }
            __syncthreads();
            if (tid == 0) {
                s->rho = (double)rho_new;
                s->inner_iter = it;
                s->iter += 1;
            }
            if (stop)
                phase = ck::B_UPDATE;
            __syncthreads();
            continue;
        }
        if (phase == ck::B_INNER) {   // GMRES: one Arnoldi step (CGS2) + Givens
            const int j = s->j, m = s->m;
            const int64_t ld = s->ld;
            T *V = wsp<T>(s, 0);
            T *w = V + (int64_t)(j + 1) * s->ld;
            const T *val = sizeof(T) == 4 ? (const T *)s->val32 : (const T *)s->val64;
            wg_spmv<BS, T, T, T>(n, L, s->rp, s->col, val, V + (int64_t)j * s->ld, T(1), T(0),
                             (const T *)nullptr, w);
            __syncthreads();
            for (int pass = 0; pass < 2; ++pass) {
                for (int g = 0; g <= j; g += 8) {   // eight columns at a time
                    T acc[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        acc[c] = 0;
                    for (int i = tid; i < n; i += BS) {
                        const T wi = w[i];
                        T vv[8];
#pragma unroll
                        for (int c = 0; c < 8; ++c)
                            vv[c] = V[(int64_t)min(g + c, j) * ld + i];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int c = 0; c < 8; ++c)
                            acc[c] += vv[c] * wi;
                    }
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        if (g + c <= j) {
                            const T v = ck::wave_sum_last(acc[c]);   // valid in lane 63
                            if ((tid & 63) == 63)
                                wred[tid >> 6][g + c] = v;
                        }
                }
                __syncthreads();
                if (tid <= j) {
                    T h = (wred[0][tid] + wred[1][tid]) + (wred[2][tid] + wred[3][tid]);
                    for (int t = 4; t < NW; t += 4)
                        h += (wred[t][tid] + wred[t + 1][tid]) + (wred[t + 2][tid] + wred[t + 3][tid]);
                    hcol[tid] = h;
                    hacc[tid] = pass == 0 ? h : hacc[tid] + h;
                }
                __syncthreads();
                for (int i = tid; i < n; i += BS) {
                    T wi = w[i];
                    for (int g = 0; g <= j; g += 8) {
                        T vv[8];
#pragma unroll
                        for (int c = 0; c < 8; ++c)
                            vv[c] = V[(int64_t)min(g + c, j) * ld + i];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int c = 0; c < 8; ++c)
                            if (g + c <= j)
                                wi -= hcol[min(g + c, j)] * vv[c];
                    }
                    w[i] = wi;
                }
                __syncthreads();
            }
            T nn = 0;
            for (int i0 = tid; i0 < n; i0 += kVec * BS) {
                T wv[kVec];
#pragma unroll
                for (int u = 0; u < kVec; ++u)
                    wv[u] = w[min(i0 + u * BS, n - 1)];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kVec; ++u)
                    if (i0 + u * BS < n)
                        nn += wv[u] * wv[u];
            }
            const T hn = sqrt(wg_sum<BS>(nn, lds));
            __shared__ int stop_sh;
            __shared__ T inv_sh;
            if (tid == 0) {
                // Hessenberg column j in the inner precision (stored as double)
                double *Hj = s->H + j * (m + 1);
                for (int c = 0; c <= j; ++c)
                    Hj[c] = (double)hacc[c];
                Hj[j + 1] = (double)hn;
                for (int i = 0; i < j; ++i) {
                    const T a = (T)Hj[i], c2 = (T)Hj[i + 1];
                    const T ci = (T)s->cs[i], si = (T)s->sn[i];
                    Hj[i] = (double)(ci * a + si * c2);
                    Hj[i + 1] = (double)(-si * a + ci * c2);
                }
                const T a = (T)Hj[j], c2 = (T)Hj[j + 1];
                const T dd = sqrt(a * a + c2 * c2);
                int stop = 0;
                if (dd == T(0)) {
                    stop = 2;           // singular least-squares problem
                } else {
                    const T cj = a / dd, sj = c2 / dd, gj = (T)s->g[j];
                    s->cs[j] = (double)cj;
                    s->sn[j] = (double)sj;
                    Hj[j] = (double)dd;
                    Hj[j + 1] = 0;
                    s->g[j + 1] = (double)(-sj * gj);
                    s->g[j] = (double)(cj * gj);
                    s->j = j + 1;
                    s->iter += 1;
                    const double est = fabs((double)s->g[j + 1]) * s->beta / s->bnorm;
                    if (est <= s->tol || hn == T(0) || j + 1 == m || s->iter >= s->max_iter)
                        stop = 1;
                }
                stop_sh = stop;
                inv_sh = hn > T(0) ? T(1) / hn : T(0);
            }
            __syncthreads();
            const int stop = stop_sh;
            if (stop == 2) {
                phase = s->j == 0 ? ck::B_DONE : ck::B_UPDATE;
                if (phase == ck::B_DONE && tid == 0)
                    s->status = ck::BREAKDOWN;
            } else if (stop == 1) {
                phase = ck::B_UPDATE;
            } else {
                const T inv = inv_sh;
                for (int i = tid; i < n; i += BS)
                    w[i] *= inv;
            }
            __syncthreads();
            continue;
        }
        // B_UPDATE: x += beta * d
        const double beta = s->beta;
        if (s->kind == ck::B_CG) {
            const T *d = wsp<T>(s, 3);
            for (int i = tid; i < n; i += BS)
                s->x[i] += beta * (double)d[i];
        } else {
            const int k = s->j, m = s->m;
            if (tid == 0) {
                for (int i = k - 1; i >= 0; --i) {
                    T acc = (T)s->g[i];
                    for (int t = i + 1; t < k; ++t)
                        acc -= (T)s->H[t * (m + 1) + i] * (T)s->y[t];
                    s->y[i] = (double)(acc / (T)s->H[i * (m + 1) + i]);
                }
            }
            __syncthreads();
            const T *V = uni(wsp<T>(s, 0));
            const double *y = uni(s->y);
            const int64_t ld = uni((int)s->ld);
            for (int i = tid; i < n; i += BS) {
                double acc = 0;
                for (int c0 = 0; c0 < k; c0 += 8) {
                    T vv[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        vv[c] = (V + (int64_t)min(c0 + c, k - 1) * ld)[(unsigned)i];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        if (c0 + c < k)
                            acc += y[c0 + c] * (double)vv[c];
                }
                s->x[i] += beta * acc;
            }
        }
        phase = ck::B_OUTER;
        __syncthreads();
    }
    __syncthreads();
    if (tid == 0) {
        s->phase = phase;
        s->launches += 1;
        ck::BStat &o = stat[which];
        o.phase = phase;
        o.status = s->status;
        o.iter = s->iter;
        o.outer = s->outer;
        o.relres = s->relres;
    }
}

// One launch: every listed slot advances by up to `budget` steps.  A slot of
// at most narrow_n rows runs on 256 threads, a larger one on 1024: a slot's
// step is a chain of L2 round trips, so more threads shorten it (n = 7,000,
// FP32 CG: 103 us a step with 256 threads and the vectors in memory, 8 us
// now), while a system of a thousand rows gains nothing from more than 256
// and, where no slot of the launch is wider, leaves the rest of the compute
// unit to other slots (the wide kernel's LDS fills it).  The width follows
// from n alone, so a slot's bits do not depend on the launch it is in.
template <typename T, int BS>
__global__ __launch_bounds__(BS) void batched_chunk(ck::BSlot *slots, ck::BStat *stat,
                                                    const int *active, int budget, int narrow_n) {
    __shared__ __align__(16) char raw[sizeof(SlotLds<T, BS>)];
    const int which = active[blockIdx.x];
    if constexpr (BS > 256) {
        if (slots[which].n > narrow_n) {
            run_slot<T, BS>(slots, stat, which, budget, *(SlotLds<T, BS> *)raw);
            return;
        }
        if (threadIdx.x >= 256)
            return;   // whole waves; barriers count the waves that remain
    }
    run_slot<T, 256>(slots, stat, which, budget, *(SlotLds<T, 256> *)raw);
}

// Builds a slot copy in one workgroup: the rows sorted by length with a bitonic
// sort of (8192 - length, row) in LDS, the slice offsets, then the entries,
// slice by slice and slot-major (coalesced stores).
template <typename T>
__global__ __launch_bounds__(1024) void slot_sell(int n, const int *__restrict__ rp,
                                                  const int *__restrict__ col,
                                                  const T *__restrict__ val,
                                                  int *__restrict__ base,
                                                  unsigned short *__restrict__ perm,
                                                  unsigned short *__restrict__ scol,
                                                  T *__restrict__ sval) {
    static_assert(ck::kSlotRows == 8192, "13 bits of row in a key");
    __shared__ unsigned key[ck::kSlotRows];
    __shared__ int sb[ck::kSlotRows / 64 + 1];
    const int tid = threadIdx.x;
    int n2 = 64;
    while (n2 < n)
        n2 <<= 1;
    for (int i = tid; i < n2; i += 1024)   // a row has at most n <= 8192 entries
        key[i] = i < n ? (unsigned)(ck::kSlotRows - (rp[i + 1] - rp[i])) << 13 | i : ~0u;
    __syncthreads();
    for (int k = 2; k <= n2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = tid; t < n2 / 2; t += 1024) {
                const int a = 2 * t - (t & (j - 1)), b = a + j;
                const unsigned x = key[a], y = key[b];
                if ((x > y) == ((a & k) == 0)) {
                    key[a] = y;
                    key[b] = x;
                }
            }
            __syncthreads();
        }
    const int slices = (n + 63) / 64;
    if (tid == 0) {
        int at = 0;
        for (int sl = 0; sl < slices; ++sl) {
            sb[sl] = at;
            at += 64 * (ck::kSlotRows - (int)(key[64 * sl] >> 13));
        }
        sb[slices] = at;
    }
    __syncthreads();
    for (int i = tid; i <= slices; i += 1024)
        base[i] = sb[i];
    for (int i = tid; i < n; i += 1024)
        perm[i] = (unsigned short)(key[i] & (ck::kSlotRows - 1));
    const int lane = tid & 63;
    for (int sl = tid >> 6; sl < slices; sl += 16) {
        const int at = 64 * sl + lane;
        const int row = at < n ? (int)(key[at] & (ck::kSlotRows - 1)) : 0;
        const int k0 = at < n ? rp[row] : 0, len = at < n ? rp[row + 1] - k0 : 0;
        const int K = (sb[sl + 1] - sb[sl]) / 64;
        for (int t = 0; t < K; ++t) {
            const bool in = t < len;
            scol[sb[sl] + 64 * t + lane] = (unsigned short)(in ? col[k0 + t] : n);
            sval[sb[sl] + 64 * t + lane] = in ? val[k0 + t] : T(0);
        }
    }
}

namespace ck {

static int64_t slot_capacity(int64_t nnz, int64_t max_row) { return nnz + 64 * max_row; }
static int64_t up256(int64_t b) { return (b + 255) / 256 * 256; }

int64_t slot_copy_bytes(int64_t n, int64_t nnz, int64_t max_row, int value_bytes) {
    const int64_t cap = slot_capacity(nnz, max_row);
    return up256(4 * (n / 64 + 2)) + up256(2 * n) + up256(2 * cap) + cap * value_bytes;
}

SlotCopy slot_copy_at(void *mem, int64_t n, int64_t nnz, int64_t max_row, int value_bytes) {
    char *p = (char *)mem;
    SlotCopy c;
    c.base = (const int *)p;
    p += up256(4 * (n / 64 + 2));
    c.perm = (const unsigned short *)p;
    p += up256(2 * n);
    c.col = (const unsigned short *)p;
    p += up256(2 * slot_capacity(nnz, max_row));
    c.val = p;
    return c;
}

ck_status launch_slot_copy(int64_t n, const int *rp, const int *col, const double *val64,
                           const float *val32, const SlotCopy &c, hipStream_t s) {
    if (n < 1 || n > kSlotRows)
        return fail(CK_E_INVALID, "a slot copy takes 1..%d rows", kSlotRows);
    auto go = [&](auto *val) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(val)>>;
        hipLaunchKernelGGL((slot_sell<T>), dim3(1), dim3(1024), 0, s, (int)n, rp, col, val,
                           (int *)c.base, (unsigned short *)c.perm, (unsigned short *)c.col,
                           (T *)c.val);
    };
    if (val32)
        go(val32);
    else
        go(val64);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

int64_t bslot_work_elems(int kind, int64_t n, int m) {
    const int64_t ld = ceil_div(std::max<int64_t>(n, 1), 64) * 64;
    return kind == B_CG ? 4 * ld : (int64_t)(m + 1) * ld;
}

ck_status launch_batched_chunk(BSlot *slots, BStat *stat, const int *active, int nactive,
                               int budget, bool fp32, hipStream_t s, int64_t max_n,
                               int narrow_n) {
    if (nactive <= 0)
        return CK_OK;
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(nactive), dim3(threads), 0, s, slots, stat, active, budget,
                           narrow_n);
    };
    if (max_n > narrow_n) {
        if (fp32)
            go(batched_chunk<float, kWideThreads>, kWideThreads);
        else
            go(batched_chunk<double, kWideThreads>, kWideThreads);
    } else if (fp32) {
        go(batched_chunk<float, kNarrowThreads>, kNarrowThreads);
    } else {
        go(batched_chunk<double, kNarrowThreads>, kNarrowThreads);
    }
    CK_HIP(hipGetLastError());
    return CK_OK;
}

}  // namespace ck
