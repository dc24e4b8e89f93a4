// Single-workgroup FP64 conjugate gradient for small systems (n <= 4096).
//
// A system this small cannot fill the GPU, and a launch per CG step would
// make launch latency the bound.  One workgroup of T threads runs the whole
// solve in one launch: thread t owns rows t, t + T, ... (R <= 8 of them);
// x, r, p and q of its rows live in registers, p also in LDS (the product
// gathers it from there), and only the matrix (L2-resident after the first
// step) and, at the rare residual steps, b are read from memory.  When no
// row has more than 5 entries (1D and 2D stencils, convection-diffusion) the
// matrix itself is loaded into registers once per solve and every product
// only gathers p from LDS.  Otherwise, when no
// row has more than 16 entries, the matrix is first copied column-major into
// a scratch buffer, so that each product reads it in whole cache lines (the
// row-major arrays, read one entry per lane per step, re-fetched partly used
// lines at every step).  The product sums each row with one lane in
// ascending entry order, many entries' loads issued together.  Dot products reduce in a fixed
// order (wave butterfly, then the wave sums by halves), so the result is
// deterministic.
//
// Every wave repeats the sums' ends, the divisions and the stop test, so few waves
// with many rows each are faster, until too little is in flight: us per iteration on
// 2D Laplacians with 1024 threads (R = 1 .. 4), 512 and 256: n = 1,024 1.91, 1.26, 1.29;
// n = 2,025 2.01, 1.37, 2.05; n = 4,096 2.43 (2.21 with all but the threads as now),
// 1.75; n = 256 2.25, 1.49, 1.36.  What bounds it now is the chain of an iteration (4,200
// clocks at n = 4,096): two workgroup sums, two divisions and two rounds of gathers.
//
// The iteration is the same Hestenes-Stiefel CG as the multi-kernel path:
// r = b - A x, p = r; then q = A p, alpha = rho / p.q, x += alpha p,
// r -= alpha q, stop when ||r|| / ||b|| <= tol; at a stop the true residual
// b - A x is recomputed and CG restarts from the current x (at most three
// times) if it is above tol.
#include "batched.hpp"

namespace {

constexpr int kWgCgRegK = 5;   // longest row kept in registers

// sum over the workgroup, returned to every thread (fixed order).  Successive
// calls alternate between the two halves of `red` (2 x kWgWaves doubles), so
// one barrier per call suffices: a half is rewritten only two calls later,
// after every thread has passed the barrier of the call in between, and so
// has finished reading it.
template <int T>
__device__ __forceinline__ double wg_sum(double v, double *red, int &parity) {
    constexpr int kWgWaves = T / 64;
    double *buf = red + parity * kWgWaves;
    parity ^= 1;
    v = ck::wave_sum_last(v);   // valid in lane 63
    if ((threadIdx.x & 63) == 63)
        buf[threadIdx.x >> 6] = v;
    __syncthreads();
    double s[kWgWaves];
#pragma unroll
    for (int w = 0; w < kWgWaves; ++w)
        s[w] = buf[w];
#pragma unroll
    for (int half = kWgWaves / 2; half > 0; half >>= 1)
#pragma unroll
        for (int w = 0; w < half; ++w)
            s[w] += s[w + half];
    return s[0];
}

// sqrt(rho) / bnorm <= tol, decided by one comparison: the left side does not
// decrease with rho, so there is a largest rho that passes, next to
// (tol * bnorm)^2.  It is searched for once a solve; where it is not found
// within a few steps (values that overflow or vanish) the test is as written.
struct StopTest {
    double bnorm, tol, largest;
    bool found;
    __device__ __forceinline__ bool direct(double rho) const { return sqrt(rho) / bnorm <= tol; }
    __device__ StopTest(double bnorm_, double tol_) : bnorm(bnorm_), tol(tol_), found(false) {
        const double t = tol * bnorm;
        largest = t * t;
        if (!(largest > 0.0 && largest < 1.0e300))
            return;
        // neighbours of a positive double are its bits plus and minus one
        long long at = __double_as_longlong(largest);
        for (int k = 0; k < 32 && at > 0 && !direct(__longlong_as_double(at)); ++k)
            --at;
        for (int k = 0; k < 32 && direct(__longlong_as_double(at + 1)); ++k)
            ++at;
        largest = __longlong_as_double(at);
        found = direct(largest) && !direct(__longlong_as_double(at + 1));
    }
    __device__ __forceinline__ bool operator()(double rho) const {
        return found ? rho <= largest : direct(rho);
    }
};

// q += entries k .. k + E - 1 (to `last` at most) of a row times v, in their order.
template <int E>
__device__ __forceinline__ void wg_row(int k, int last, const int *__restrict__ col,
                                       const double *__restrict__ val, const double *v,
                                       double &q) {
    int cc[E];
    double vv[E], g[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int kk = min(k + e, last);
        cc[e] = col[kk];
        vv[e] = val[kk];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < E; ++e)
        g[e] = v[cc[e]];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (k + e <= last)
            q += vv[e] * g[e];
}

// q[u] = (A v)[row u of this thread], v in LDS.  One row after the other, its next
// sixteen entries in flight together: they share cache lines, and a lane with a long
// row does not take its other rows through as many steps.  Stepping all rows together,
// an entry each, took (us per iteration, 1024 threads of at most 4 rows; 512 of at most
// 8; now): n = 4,000, rows of 17 on average 51.6, 53.8, 34.5; of 51 181, 185, 91; one
// row of 4,000 863, 1,373, 112; power-law rows up to 1,407 543, 635, 188.  Thirty-two
// entries at a time gain more on long rows (one of 4,000: 81) but leave rows of 17 no
// faster than they were (49).
template <int R>
__device__ __forceinline__ void wg_matvec(const int (&kb)[R], const int (&ke)[R],
                                          const int *__restrict__ col,
                                          const double *__restrict__ val, const double *v,
                                          double (&q)[R]) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
        q[u] = 0;
        int k = kb[u];
        for (; k + 8 < ke[u]; k += 16)
            wg_row<16>(k, ke[u] - 1, col, val, v, q[u]);
        for (; k < ke[u]; k += 8)
            wg_row<8>(k, ke[u] - 1, col, val, v, q[u]);
    }
}

// The same product from the column-major copy, slots in pairs: slots 2q and
// 2q + 1 of local row i are the int2 / double2 at q * RW + i.  A step's loads
// are consecutive across the lanes and bring two slots of every row, so each
// product reads the matrix once, in whole cache lines, in ceil(K / 2) rounds
// (the row-major arrays, read one entry per lane per step, re-fetched partly
// used lines at every step).  Entries are summed in the same order, so the
// result is the same.
template <int T, int R>
__device__ __forceinline__ void wg_matvec_cm(const int (&len)[R], int K,
                                             const int2 *__restrict__ ccol,
                                             const double2 *__restrict__ cval, const double *v,
                                             double (&q)[R]) {
    constexpr int RW = R * T;
#pragma unroll
    for (int u = 0; u < R; ++u)
        q[u] = 0;
    for (int s = 0; s < K; s += 2) {
        int2 cc[R];
        double2 vv[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int i = threadIdx.x + u * T;
            cc[u] = ccol[(s >> 1) * RW + i];
            vv[u] = cval[(s >> 1) * RW + i];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            if (s < len[u])
                q[u] += vv[u].x * v[cc[u].x];
            if (s + 1 < len[u])
                q[u] += vv[u].y * v[cc[u].y];
        }
    }
}

// The product with the matrix in registers: slot k of local row u holds
// rv[k][u] and its column, the 16-bit half k % 2 of rcp[k / 2][u], loaded
// once per solve.  Slots past the row's length hold
// value 0 and column 0 (columns are stored as their byte offsets in v, below
// 32,768): p[0] is finite while the solve runs (a non-finite
// p.q ends it first) and q starts at +0, so adding 0 * p[0] leaves q's bits
// unchanged, and every row's sum equals, bit for bit, the other forms' sum
// of its entries in the same order.
constexpr int kWgRegPairs = (kWgCgRegK + 1) / 2;

// v at slot k's column.  An empty statement that claims to change w: the columns
// are unpacked here, at each use, instead of being hoisted out of the CG loop as
// 20 loop-invariant registers.
__device__ __forceinline__ double wg_gather(unsigned w, int k, const double *v) {
    asm volatile("" : "+v"(w));
    return *(const double *)((const char *)v + ((k & 1) ? (w >> 16) : (w & 0xffffu)));
}

template <int R>
__device__ __forceinline__ void wg_matvec_reg(const unsigned (&rcp)[kWgRegPairs][R],
                                              const double (&rv)[kWgCgRegK][R], const double *v,
                                              double (&q)[R]) {
#pragma unroll
    for (int u = 0; u < R; ++u)
        q[u] = 0;
    // gathers in rounds of G slots, all rows' loads of a round in flight together
    // (more at once would spill registers at eight rows per lane; one slot a round
    // 2.27 us per iteration at n = 4096, three 2.15)
    constexpr int G = R >= 8 ? 3 : kWgCgRegK;
#pragma unroll
    for (int k0 = 0; k0 < kWgCgRegK; k0 += G) {
        double g[G][R];
#pragma unroll
        for (int k = k0; k < k0 + G && k < kWgCgRegK; ++k)
#pragma unroll
            for (int u = 0; u < R; ++u)
                g[k - k0][u] = wg_gather(rcp[k >> 1][u], k, v);
#pragma unroll
        for (int k = k0; k < k0 + G && k < kWgCgRegK; ++k)
#pragma unroll
            for (int u = 0; u < R; ++u)
                q[u] += rv[k][u] * g[k - k0][u];
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The same where every row has at most two entries on either side of its diagonal
// entry (1D and 2D stencils): that one is slot 2 of every row, the entries before it
// end at slot 1, and its factor is the lane's own entry of v, in a register.  Four
// gathers a row instead of five: 2.15 us per iteration at n = 4096, 1.75 this way.
template <int R>
__device__ __forceinline__ void wg_matvec_centre(const unsigned (&rcp)[kWgRegPairs][R],
                                                 const double (&rv)[kWgCgRegK][R],
                                                 const double *v, const double (&own)[R],
                                                 double (&q)[R]) {
    double g[2][R];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int u = 0; u < R; ++u)
            g[k][u] = wg_gather(rcp[0][u], k, v);
#pragma unroll
    for (int u = 0; u < R; ++u) {
        q[u] = 0;
        q[u] += rv[0][u] * g[0][u];
        q[u] += rv[1][u] * g[1][u];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int u = 0; u < R; ++u)
            g[k][u] = wg_gather(rcp[1][u], k, v);
#pragma unroll
    for (int u = 0; u < R; ++u)
        q[u] += rv[2][u] * own[u];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        q[u] += rv[3][u] * g[0][u];
        q[u] += rv[4][u] * g[1][u];
    }
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace

// The solve after the prologue, one instantiation per product form (the
// form is fixed for the whole solve, so each keeps only its own state live):
// the matrix in registers (with or without its diagonal apart), the column-major
// copy, or the row-major arrays.
enum { kWgRows = 0, kWgColMajor = 1, kWgReg = 2, kWgCentre = 3 };
template <int T, int R, int MODE>
__device__ __forceinline__ void cg_wg_run(int n, const int (&kb)[R], const int (&ke)[R],
                                          const int (&len)[R], int K,
                                          double (&xr)[R], double bb,
                                          const int *__restrict__ col,
                                          const double *__restrict__ val,
                                          const double *__restrict__ b, double *__restrict__ x,
                                          double tol, int max_iter, int2 *__restrict__ ccol,
                                          double2 *__restrict__ cval, ck::WgCgOut *out,
                                          double *v, double *red, int parity) {
    constexpr int RW = R * T;
    const int t = threadIdx.x;
    double rr[R], pr[R], q[R];
    constexpr bool reg = MODE == kWgReg, cm = MODE == kWgColMajor, centre = MODE == kWgCentre;
    unsigned rcp[kWgRegPairs][R];
    double rv[kWgCgRegK][R];
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
        for (int k = 0; k < kWgRegPairs; ++k)
            rcp[k][u] = 0;
#pragma unroll
    for (int k = 0; k < kWgCgRegK; ++k)
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const bool in = reg && k < len[u];
            rcp[k >> 1][u] |= (in ? 8u * (unsigned)col[kb[u] + k] : 0u) << (16 * (k & 1));
            rv[k][u] = in ? val[kb[u] + k] : 0.0;
        }
    if constexpr (centre) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int i = t + u * T;
            int before = 0;   // entries left of the diagonal
            while (before < len[u] && col[kb[u] + before] < i)
                ++before;
            const bool diag = before < len[u] && col[kb[u] + before] == i;
            rv[2][u] = diag ? val[kb[u] + before] : 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = k < 2 ? before - 2 + k : before + (diag ? 1 : 0) + k - 2;
                const bool in = k < 2 ? e >= 0 : e < len[u];
                rcp[k >> 1][u] |= (in ? 8u * (unsigned)col[kb[u] + e] : 0u) << (16 * (k & 1));
                rv[k < 2 ? k : k + 1][u] = in ? val[kb[u] + e] : 0.0;
            }
        }
    }
    auto matvec = [&](const double (&own)[R]) {
        if constexpr (centre)
            wg_matvec_centre<R>(rcp, rv, v, own, q);
        else if constexpr (reg)
            wg_matvec_reg<R>(rcp, rv, v, q);
        else if constexpr (cm)
            wg_matvec_cm<T, R>(len, K, ccol, cval, v, q);
        else
            wg_matvec<R>(kb, ke, col, val, v, q);
    };
    if constexpr (cm) {
        for (int s = 0; s < K; s += 2) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int i = t + u * T;
                const bool in0 = s < len[u], in1 = s + 1 < len[u];   // rows past n: len 0
                ccol[(s >> 1) * RW + i] = make_int2(in0 ? col[kb[u] + s] : 0,
                                                    in1 ? col[kb[u] + s + 1] : 0);
                cval[(s >> 1) * RW + i] = make_double2(in0 ? val[kb[u] + s] : 0.0,
                                                       in1 ? val[kb[u] + s + 1] : 0.0);
            }
        }
        // the copy is read by other waves of this workgroup: the barrier
        // below (in the first workgroup sum) orders it
        __threadfence_block();
    }
    const double bnorm = sqrt(wg_sum<T>(bb, red, parity));
    const StopTest stop(bnorm, tol);
    int status = ck::BUDGET, iters = 0, restarts = 0;
    double relres = 0;
    if (bnorm == 0.0) {
#pragma unroll
        for (int u = 0; u < R; ++u)
            xr[u] = 0;
        status = ck::CONVERGED;
    } else {
        for (restarts = 0; restarts <= 3; ++restarts) {
            // r = b - A x
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (t + u * T < n)
                    v[t + u * T] = xr[u];
            __syncthreads();
            matvec(xr);
            double rho = 0;
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int i = t + u * T;
                rr[u] = (i < n ? b[i] : 0.0) - q[u];
                pr[u] = rr[u];
                rho += rr[u] * rr[u];
            }
            rho = wg_sum<T>(rho, red, parity);   // its barrier also retires the reads of v
            relres = sqrt(rho) / bnorm;
            if (relres <= tol) {
                status = ck::CONVERGED;
                break;
            }
            int state = ck::RUN;
            while (state == ck::RUN) {
                if (iters >= max_iter) {
                    state = ck::BUDGET;
                    break;
                }
#pragma unroll
                for (int u = 0; u < R; ++u)
                    if (t + u * T < n)
                        v[t + u * T] = pr[u];
                __syncthreads();
                matvec(pr);
                double pq = 0;
#pragma unroll
                for (int u = 0; u < R; ++u)
                    pq += pr[u] * q[u];
                const double sigma = wg_sum<T>(pq, red, parity);
                if (!(sigma > 0.0)) {
                    state = ck::BREAKDOWN;
                    break;
                }
                const double alpha = rho / sigma;
                double rn = 0;
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    xr[u] += alpha * pr[u];
                    rr[u] -= alpha * q[u];
                    rn += rr[u] * rr[u];
                }
                const double rho_new = wg_sum<T>(rn, red, parity);
                ++iters;
                if (stop(rho_new)) {
                    state = ck::CONVERGED;
                    break;
                }
                const double beta = rho_new / rho;
#pragma unroll
                for (int u = 0; u < R; ++u)
                    pr[u] = rr[u] + beta * pr[u];
                rho = rho_new;
            }
            if (state == ck::BREAKDOWN) {
                status = ck::BREAKDOWN;
                break;
            }
            // true residual of the current x
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (t + u * T < n)
                    v[t + u * T] = xr[u];
            __syncthreads();
            matvec(xr);
            double tr = 0;
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int i = t + u * T;
                const double d = (i < n ? b[i] : 0.0) - q[u];
                tr += d * d;
            }
            relres = sqrt(wg_sum<T>(tr, red, parity)) / bnorm;
            if (relres <= tol) {
                status = ck::CONVERGED;
                break;
            }
            if (state == ck::BUDGET) {
                status = ck::BUDGET;
                break;
            }
        }
        if (restarts > 3)
            restarts = 3;
    }
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (t + u * T < n)
            x[t + u * T] = xr[u];
    if (t == 0) {
        out->status = status;
        out->iter = iters;
        out->restarts = restarts;
        out->relres = relres;
    }
}

// ccol / cval: scratch of kWgCgColMajorK / 2 * T * R pairs for the
// column-major copy, used when no row has more than kWgCgColMajorK entries.
template <int T, int R>
__global__ __launch_bounds__(T) void cg_wg(int n, const int *__restrict__ rp,
                                                    const int *__restrict__ col,
                                                    const double *__restrict__ val,
                                                    const double *__restrict__ b,
                                                    double *__restrict__ x, double tol,
                                                    int max_iter, int2 *__restrict__ ccol,
                                                    double2 *__restrict__ cval,
                                                    ck::WgCgOut *out) {
    constexpr int kWgWaves = T / 64;
    __shared__ double v[T * R];   // p (or x while forming the residual)
    __shared__ double red[2 * kWgWaves];
    __shared__ int kmax[kWgWaves];
    int parity = 0;
    const int t = threadIdx.x;
    int kb[R], ke[R], len[R];
    double xr[R];
    int trips = 0;
    double bb = 0;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int i = t + u * T;
        const bool in = i < n;
        kb[u] = in ? rp[i] : 0;
        ke[u] = in ? rp[i + 1] : 0;
        len[u] = ke[u] - kb[u];
        const double bi = in ? b[i] : 0.0;
        xr[u] = in ? x[i] : 0.0;
        trips = max(trips, ke[u] - kb[u]);
        bb += bi * bi;
    }
    // longest row of the system: it picks the product form for the solve
    int K = trips;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        K = max(K, __shfl_xor(K, off, 64));
    if ((t & 63) == 0)
        kmax[t >> 6] = K;
    __syncthreads();
    K = 0;
#pragma unroll
    for (int w = 0; w < kWgWaves; ++w)
        K = max(K, kmax[w]);
    bool apart = K <= kWgCgRegK;   // the diagonal can be slot 2 of every row
    if (apart) {                   // uniform
#pragma unroll
        for (int u = 0; u < R; ++u) {   // the third entry is on neither outer side
            const int i = t + u * T;
            if (len[u] > 2)
                apart = apart && col[kb[u] + 2] >= i && col[ke[u] - 3] <= i;
        }
        apart = __syncthreads_and(apart) != 0;
    }
    if (apart)
        cg_wg_run<T, R, kWgCentre>(n, kb, ke, len, K, xr, bb, col, val, b, x, tol, max_iter,
                                   ccol, cval, out, v, red, parity);
    else if (K <= kWgCgRegK)
        cg_wg_run<T, R, kWgReg>(n, kb, ke, len, K, xr, bb, col, val, b, x, tol, max_iter,
                             ccol, cval, out, v, red, parity);
    else if (K <= ck::kWgCgColMajorK)
        cg_wg_run<T, R, kWgColMajor>(n, kb, ke, len, K, xr, bb, col, val, b, x, tol,
                                  max_iter, ccol, cval, out, v, red, parity);
    else
        cg_wg_run<T, R, kWgRows>(n, kb, ke, len, K, xr, bb, col, val, b, x, tol, max_iter,
                              ccol, cval, out, v, red, parity);
}

namespace ck {

ck_status launch_cg_wg(int n, const int *rp, const int *col, const double *val, const double *b,
                       double *x, double tol, int max_iter, void *cm_col, void *cm_val,
                       WgCgOut *out, hipStream_t s) {
    int2 *ccol = (int2 *)cm_col;
    double2 *cval = (double2 *)cm_val;
    if (n < 1 || n > kWgCgMaxN)
        return fail(CK_E_INVALID, "single-workgroup CG takes 1..%d rows, got %d", kWgCgMaxN, n);
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(threads), 0, s, n, rp, col, val, b, x, tol,
                           max_iter, ccol, cval, out);
    };
    if (n <= 256)
        go(cg_wg<256, 1>, 256);
    else if (n <= 512)
        go(cg_wg<512, 1>, 512);
    else if (n <= 1024)
        go(cg_wg<512, 2>, 512);
    else if (n <= 2048)
        go(cg_wg<512, 4>, 512);
    else
        go(cg_wg<512, 8>, 512);
    CK_HIP(hipGetLastError());
    return CK_OK;
}

}  // namespace ck
