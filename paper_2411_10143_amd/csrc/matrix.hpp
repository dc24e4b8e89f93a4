// Device-resident matrix store and the internal launch interface of the SpMV
// kernel family.
#pragma once

#include <atomic>
#include <map>
#include <mutex>

#include "devcache.hpp"
#include "krylov.hpp"

struct ck_matrix {
    int64_t n = 0, ncols = 0, nnz = 0;
    int device = 0;
    uint32_t flags = 0;
    // CSR (always present)
    int32_t *rp = nullptr;
    int32_t *col = nullptr;
    double *val = nullptr;
    float *val32 = nullptr;           // CK_KEEP_FP32
    // ELL (after conversion): column-major, slot s of row i at s*pitch + i
    int32_t *ell_col = nullptr;
    double *ell_val = nullptr;
    float *ell_val32 = nullptr;
    int64_t ell_K = 0, ell_pitch = 0;
    std::atomic<bool> has_ell{false};
    // COO (after conversion): row index per stored entry; col/val shared with CSR
    int32_t *coo_row = nullptr;
    std::atomic<bool> has_coo{false};
    // CSR-panel (after conversion): P column panels of width W, panel-major.
    // Dense layout (panel_row == nullptr): panel_rows = P*n, panel_rp[p*n + i]
    // = start of row i in panel p.  Row-list layout: only the panel_rows
    // non-empty panel rows, in panel-major order; panel_row[k] = the matrix
    // row of panel row k, panel_rp[k] its start, and panel_boff[p*(B+1) + j]
    // = the first panel row of panel p whose row is >= 256 j (B = ceil(n/256))
    int panel_P = 0;
    int64_t panel_W = 0;
    int64_t panel_rows = 0;
    int64_t panel_B = 0;
    int32_t *panel_row = nullptr;
    int32_t *panel_boff = nullptr;
    int32_t *panel_rp = nullptr;
    int32_t *panel_col = nullptr;
    double *panel_val = nullptr;
    float *panel_val32 = nullptr;
    std::atomic<bool> has_panel{false};
    // merge-path plan of the panel-major arrays read as one CSR of panel_rows rows
    int32_t *panel_plan = nullptr;
    bool panel_cut = true;            // a workgroup may start inside a panel row
    // merge-path plan (after conversion to CSR-merge): where every workgroup
    // starts and which merged items are row ends (merge_plan_ints); cut =
    // a workgroup may start inside a row
    int32_t *merge_plan = nullptr;
    bool merge_cut = true;
    std::atomic<bool> has_merge_plan{false};
    // DIA (after conversion): dia_nd offsets (col - row, ascending), values
    // diagonal-major: diagonal k of row i at k*dia_pitch + i, absent = +0.0
    int32_t *dia_off = nullptr;
    double *dia_val = nullptr;
    float *dia_val32 = nullptr;
    int64_t dia_nd = 0, dia_pitch = 0;
    // Constant form (dia_coef != nullptr, dia_val not kept): the entries of
    // every diagonal have the same bits; dia_coef[k] is diagonal k's value and
    // bit k of dia_mask's row i says whether row i stores it (one byte a row
    // for at most 8 diagonals, else four, for at most 32)
    double *dia_coef = nullptr;
    float *dia_coef32 = nullptr;
    void *dia_mask = nullptr;
    std::atomic<bool> has_dia{false};
    // HYB (after conversion): ELL part of width hyb_K (layout as ELL) and the
    // hyb_nt rows longer than hyb_K, ascending; their entries hyb_K.. stay in
    // the CSR arrays and are summed with hyb_L lanes per row
    int32_t *hyb_col = nullptr;
    double *hyb_val = nullptr;
    float *hyb_val32 = nullptr;
    int32_t *hyb_rows = nullptr;
    int64_t hyb_K = 0, hyb_pitch = 0, hyb_nt = 0;
    int hyb_L = 1;
    std::atomic<bool> has_hyb{false};
    int64_t max_row = 0;              // longest row
    int64_t span = 0;                 // sum over the rows of last column - first column
    // Slices of x: what CSR-panel makes of a matrix to which slices_of() gives some
    // (none of the panel arrays then; the layout: slices.hip)
    int slice_P = 0;
    int32_t *slice_base = nullptr;       // all in one block, which slice_val starts
    unsigned short *slice_ends = nullptr;
    unsigned short *slice_col = nullptr;
    double *slice_val = nullptr;
    float *slice_val32 = nullptr;
    // slot copies (batched.hpp) of a small matrix, FP64 and FP32 values
    char *slot_mem[2] = {nullptr, nullptr};
    std::atomic<bool> has_slot[2] = {false, false};
    // feature scratch of the device-resident cascade (kept with the handle)
    char *devsel_scratch = nullptr;
    int64_t *devsel_ints = nullptr;
    ck_config active{};
    std::mutex mu;                    // guards conversions, `active` and `carry`
    ck::MemSource mem;                // where every device block of the handle comes from
    // merge-path / COO carry workspace of spmv_apply, one per stream (work on
    // one stream is ordered, so reuse on that stream is safe)
    std::map<hipStream_t, void *> carry;
};

namespace ck {

// A block of `count` T for handle M, allocated for use on stream s.
template <typename T>
ck_status mat_alloc(ck_matrix &M, T **p, int64_t count, hipStream_t s) {
    void *q = nullptr;
    const ck_status st = mem_alloc(M.mem, &q, (size_t)(count > 0 ? count : 1) * sizeof(T), s);
    *p = (T *)q;
    return st;
}
inline void mat_free(ck_matrix &M, void *p) { mem_free(M.mem, p); }

// Arguments of one product y = alpha*A*x + beta*y.
//  skip   : if non-null and *skip != 0 when the launch starts, it does nothing
//           (lets a solver enqueue iterations ahead of its convergence test).
//  cg     : fused CG step (only where spmv_fuses_dot() holds): the launch also
//           leaves every block's part of sigma = y.x (x = p, y = q = A p) in
//           dot_partials, spmv_dot_blocks() entries.
//  carry  : workspace of spmv_carry_bytes() for merge-path and COO carries
//           and CSR-panel partial sums; when null the launch allocates it
//           stream-ordered.
template <typename T>
struct SpmvArgs {
    T alpha = 1, beta = 0;
    const T *x = nullptr;
    T *y = nullptr;
    const int *skip = nullptr;
    CgDev<T> *cg = nullptr;
    T *dot_partials = nullptr;
    void *carry = nullptr;
};

// Counters that every workgroup of a large grid adds to are kept kSpread
// times, kSpreadInts ints apart (one 4,096-workgroup grid adding to a single
// word waits 37 us for it); the host sums them.
constexpr int kSpread = 32, kSpreadInts = 64;

// Builds M's slot copy (of the FP32 values if fp32; M.n <= kSlotRows) if it is
// not there yet; returns when it is built.  Its bytes: slot_bytes_of.
ck_status build_slot_copy(ck_matrix &M, bool fp32, hipStream_t s);

bool config_valid(const ck_config &c);
bool spmv_fuses_dot(const ck_config &c);
// Number of dot partials a fused launch writes (0 if not fused; <= kMaxPartials).
int64_t spmv_dot_blocks(const ck_matrix &M, const ck_config &c);
// Bytes of carry workspace a launch needs (0 if none).
int64_t spmv_carry_bytes(const ck_matrix &M, const ck_config &c, bool fp32);
// The bytes spmv_apply_noalloc admits against its fixed array: the size with
// 2048 merged items per panel-product workgroup.  A launch's carries take up
// to 3.3 % more (its workgroups start up to 64 items early).
int64_t spmv_noalloc_bytes(const ck_matrix &M, const ck_config &c);
// Merge-path plan of a CSR of `rows` rows (the matrix, or the panel-major
// arrays): its size in ints, and the launches that build it.
int64_t merge_plan_ints(int64_t rows, int64_t nnz);
ck_status launch_merge_plan(int64_t rows, int64_t nnz, const int32_t *rp, int32_t *plan,
                            hipStream_t s);
// Whether a workgroup may start inside a row, from the longest row (-1: not known).
bool merge_cuts_rows(int64_t max_row);

template <typename T>
ck_status launch_spmv(const ck_matrix &M, const ck_config &c, const SpmvArgs<T> &a,
                      hipStream_t s);

// Deterministic two-stage reductions (vecops.hip)
template <typename T>
int64_t dot_blocks(int64_t n);
template <typename T>
ck_status launch_dot_partials(int64_t n, const T *x, const T *y, T *partials, hipStream_t s);

const char *kernel_name(const ck_config &c, bool fp32);
ck_config default_config(int64_t n, int64_t nnz);

}  // namespace ck
