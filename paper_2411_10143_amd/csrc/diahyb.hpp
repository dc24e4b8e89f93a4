// DIA and HYB formats: conversions and products (diahyb.hip).
#pragma once

#include "matrix.hpp"

namespace ck {

// Build M.dia_* (CK_E_UNSUPPORTED when ndiag * pitch > 8 * nnz) / M.hyb_*.
// Enqueued on s; both block on s once to read a count back.
ck_status convert_to_dia(ck_matrix &M, hipStream_t s);
ck_status convert_to_hyb(ck_matrix &M, hipStream_t s);
// Device memory the conversions hold at most, their scratch included, for values
// of value_bytes (the FP32 copy counted).
int64_t dia_convert_bytes(int64_t n, int64_t ncols, int64_t ndiag, int value_bytes);
int64_t hyb_convert_bytes(int64_t n, int64_t nnz, int value_bytes);

// Bytes a row's diagonal mask takes in the constant form.
inline int64_t dia_mask_bytes(int64_t nd) { return nd <= 8 ? 1 : 4; }
// The dense values of M's DIA copy (layout of dia_val) into dv.
ck_status export_dia_values(const ck_matrix &M, double *dv, hipStream_t s);

// Workgroups of a DIA product of `groups` row groups: the constant form, whose
// rows take little time, runs them on at most 2048 (eight per compute unit)
// that loop, as the dispatcher issues about one workgroup per nanosecond.
inline int64_t dia_blocks(const ck_matrix &M, int64_t groups) {
    const int64_t most = M.dia_coef != nullptr ? kFoldPartials : kRowBlocks;
    return groups < most ? (groups > 0 ? groups : 1) : most;
}
// DIA product over G logical row blocks (dot partials as the ELL kernel).
template <typename T, bool BETA, bool DOT>
void launch_dia_spmv(const ck_matrix &M, int64_t G, const T *dv, const SpmvArgs<T> &a,
                     hipStream_t s);
// HYB remainder pass: y[i] += alpha * (entries K.. of each long row i).
template <typename T>
void launch_hyb_tail(const ck_matrix &M, const T *val, const SpmvArgs<T> &a, hipStream_t s);

}  // namespace ck
