// CSR-panel products from slices of x in LDS, see slices.hip.  G_dot = dot partials
// for a fused CG step.
#pragma once

#include "matrix.hpp"

namespace ck {

// Partial sums of a product at most: they fit the fixed array of spmv_apply_noalloc.
constexpr int64_t kSliceWorkBytes = int64_t(64) << 20;

// Slices of x of a matrix that takes them, 0 for any other: from its sizes, its
// longest row and the sum over its rows of last column - first column.
int slices_of(int64_t n, int64_t ncols, int64_t nnz, int64_t max_row, int64_t span);
int64_t slices_bytes(int64_t n, int64_t nnz, int P, bool fp32);
int64_t slices_work_bytes(int64_t n, int P, bool fp32);   // a product's partial sums
// Allocates M's slice arrays and builds them on s, P = slices_of(M) (free_slices once s
// has finished, on error).
ck_status build_slices(ck_matrix &M, int P, hipStream_t s);
void free_slices(ck_matrix &M);
template <typename T>
ck_status launch_slices(const ck_matrix &M, const SpmvArgs<T> &a, T *ypart, int64_t G_dot,
                        hipStream_t s);

}  // namespace ck
