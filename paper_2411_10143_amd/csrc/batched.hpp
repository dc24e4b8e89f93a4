// Slot record of the batched small-system solver (device memory, one per slot).
#pragma once

#include "krylov.hpp"
#include "slotrule.hpp"

namespace ck {

constexpr int kBMaxM = 32;            // largest GMRES restart in the batched path
enum : int { B_CG = 0, B_GMRES = 1 };
enum : int { B_OUTER = 0, B_INNER = 1, B_UPDATE = 2, B_DONE = 3 };

// Slot copy of a small matrix (at most kSlotRows rows), read by the inner
// products: sliced ELLPACK (Monakov, Lokhmotov and Avetisyan, 2010) with the rows
// sorted by length as in SELL-C-sigma (Kreutzer et al., 2014), longest first (ties
// by row), 64 to a slice, one lane per row.  Slice s holds slots base[s] ..
// base[s + 1] - 1, slot-major (64 lanes of entry 0, of entry 1, ...), K_s = its
// first row's length; columns are 16 bits, padding has column n (a zero kept
// behind the vector in LDS) and value 0; perm[64 s + lane] = the row.  The
// entries and their padding take at most nnz + 64 * (longest row) slots.
constexpr int kSlotRows = 8192;
struct SlotCopy {
    const int *base = nullptr;              // ceil(n / 64) + 1; null: no copy
    const unsigned short *perm = nullptr;   // n, in slice order
    const unsigned short *col = nullptr;
    const void *val = nullptr;              // inner type
};
// Bytes of a copy, its pieces within a block, and building it on s.
int64_t slot_copy_bytes(int64_t n, int64_t nnz, int64_t max_row, int value_bytes);
SlotCopy slot_copy_at(void *mem, int64_t n, int64_t nnz, int64_t max_row, int value_bytes);
ck_status launch_slot_copy(int64_t n, const int *rp, const int *col, const double *val64,
                           const float *val32, const SlotCopy &c, hipStream_t s);

struct BSlot {
    // problem, set at admission
    int kind, n, lanes, m;
    const int *rp;
    const int *col;
    const double *val64;
    const float *val32;
    SlotCopy sell;        // of val32 (FP32 inner solves) or val64; base null: none
    const double *b;
    double *x;            // caller's solution vector (holds x0 on admission)
    double *r64;          // FP64 residual
    void *work;           // inner vectors: CG r,p,q,d; GMRES basis (m+1 columns)
    int64_t ld;           // length of one inner vector (n rounded up to 64)
    double bnorm, tol;
    int max_iter, inner_cap;
    int keep_x0;          // 1: start from the x given; 0: start from x = 0
    int inner_lanes;      // lanes per row of the inner products, 1 with a slot copy
    // state
    int phase, status, iter, outer, inner_iter, j, launches, pad;
    double beta, relres, inner_tol, rho;
    // Hessenberg least squares (values held in the inner precision)
    double H[(kBMaxM + 1) * kBMaxM];
    double cs[kBMaxM], sn[kBMaxM], g[kBMaxM + 1], y[kBMaxM];
};

// Compact per-slot status written at the end of every launch (read by the host)
struct BStat {
    int phase, status, iter, outer;
    double relres;
};

// Single-workgroup FP64 CG (one launch per solve) for at most kWgCgMaxN rows.
constexpr int kWgCgMaxN = 4096;
struct WgCgOut {
    int status, iter, restarts, pad;
    double relres;   // true relative residual at exit
};
// When the longest row has 6 to this many entries (even), the matrix is
// copied column-major once per solve into cm_col / cm_val: kWgCgColMajorK *
// kWgCgMaxN ints and doubles, 16-byte aligned (rows of at most 5 entries are
// held in registers instead, and longer ones read in place).
constexpr int kWgCgColMajorK = 16;
ck_status launch_cg_wg(int n, const int *rp, const int *col, const double *val, const double *b,
                       double *x, double tol, int max_iter, void *cm_col, void *cm_val,
                       WgCgOut *out, hipStream_t s);

// elements (of the inner type) of a slot's `work`
int64_t bslot_work_elems(int kind, int64_t n, int m);
// max_n = the most rows of a listed slot; slots of at most narrow_n rows run on
// 256 threads, the others on 1024.  `stat` and `active` may be pinned host memory.
constexpr int kNarrowN = 1024;   // the request loop's narrow_n
constexpr int kNarrowThreads = 256, kWideThreads = 1024;
ck_status launch_batched_chunk(BSlot *slots, BStat *stat, const int *active, int nactive,
                               int budget, bool fp32, hipStream_t s, int64_t max_n,
                               int narrow_n);

}  // namespace ck
