// CSR-panel SpMV (XCD-aware column panels), see panel.hip.  G_dot = dot
// partials for a fused CG step.
#pragma once

#include "matrix.hpp"

namespace ck {

// panels for a vector of ncols entries of value_bytes each (x slice <= 2 MB)
int panel_count_for(int64_t ncols, int value_bytes);
int64_t panel_scan_tmp_elems(int64_t N);
int64_t panel_tmp_ints(int64_t N);   // N counts, then their counters or the scan's scratch
// Device memory a conversion to panels holds at most, its scratch included, for
// values of value_bytes (the FP32 copy counted).
int64_t panel_convert_bytes(int64_t n, int64_t ncols, int64_t nnz, int value_bytes);
// The panel count of M's CSR-panel copy: panel_count_for(ncols, 8), or 4
// (see panel.hip).  tmp: panel_tmp_ints(panel_count_for(
// ncols, 8) * n) ints of scratch; on return tmp[0 .. P n) holds the chosen P's per-row panel counts,
// *filled of them nonzero.
ck_status panel_choose_count(const ck_matrix &M, int *tmp, hipStream_t s, int *P_out,
                             int64_t *filled);
// Sets M's panel count, width and rows to those a CSR-panel copy in P panels would
// have, `filled` of whose rows hold entries; false for P = 4 if it would not be made.
bool panel_layout_of(ck_matrix &M, int P, int64_t filled);
// Exclusive scan of N ints into N + 1 outputs (out[N] = total); tmp holds
// panel_scan_tmp_elems(N) ints.
ck_status launch_scan_exclusive(int64_t N, const int *in, int *out, int *tmp, hipStream_t s);
// The panel-major copy, from cnt = the P*n counts that panel_choose_count left.
ck_status launch_to_panel(const ck_matrix &M, int P, int64_t W, int *cnt, int *tmp, int *prp,
                          int *pcol, double *pval, float *pval32, hipStream_t s);
// After launch_to_panel (M.panel_rp = the dense row pointers): switch M to the
// row-list layout when at most 3/4 of the P*n panel rows are filled (cnt is
// overwritten).  Returns when done.
ck_status panel_make_rows(ck_matrix &M, int *cnt, int64_t filled, hipStream_t s);
// y = alpha * (sum of the P partial vectors, in panel order) + beta * y (M's slices'
// where it has them)
template <typename T>
ck_status launch_panel_combine(const ck_matrix &M, const SpmvArgs<T> &a, const T *ypart,
                               int64_t G_dot, hipStream_t s);

}  // namespace ck
