// Which form a small system's inner products take in a one-workgroup solve,
// and which single solves run in one workgroup at all.  Host arithmetic on
// sizes alone, so that a matrix always takes the same form.
//
// A workgroup's product is bound by the instructions it issues, or by its
// longest row, which few lanes walk while the other waves wait; the
// multi-workgroup kernels by their launches, or again by the longest row.
// Nanoseconds, fitted to CG iterations of 500 to 8,192 rows (FP64, mixed):
//   copy, one lane per row   0.18, 0.16 an entry; at least 100, 83 an entry of
//                            the longest row
//   CSR, L lanes per row     0.32, 0.25 an entry, and 270 for every L entries of
//                            the longest row, in each pass over 4 T / L rows
//                            that may hold such a row (T threads)
//   the rest of an iteration 4,500
//   multi-workgroup kernels  11,500, 15,500 and 150, 130 for every L entries
// us per iteration, FP64, (copy, CSR with the L given, multi-workgroup, before
// there was a copy): 17 entries a row, L = 16, n = 1,000 7.7, 13.3, 11.1, 25.1;
// n = 4,000 17.2, 38.7, 12.6, 75; 51 a row, L = 32, n = 4,000 39.8, 76, 12.7, 147;
// one row of n = 4,000, L = 4, 389, 276, 142, 491; eight of 2,000, n = 4,000, L = 8,
// 202, 149, 54, 335; eight of 200, n = 4,000, L = 2, 27, 71, 29, 94; power-law rows up
// to 1,407, L = 16, 148, 116, 21, 264.
#pragma once

#include <algorithm>
#include <cstdint>

namespace ck {

// Nanoseconds of a product from the copy, and from the CSR arrays with L lanes.
inline int64_t slot_copy_ns(int64_t nnz, int64_t max_row, bool fp32) {
    return fp32 ? std::max(nnz * 16 / 100, max_row * 83) : std::max(nnz * 18 / 100, max_row * 100);
}
inline int64_t slot_lanes_ns(int64_t n, int64_t nnz, int64_t max_row, int lanes, int threads,
                             bool fp32) {
    const int64_t per_pass = 4 * threads / lanes;
    const int64_t passes = std::min((n + per_pass - 1) / per_pass,
                                    max_row > 0 ? nnz / max_row : 0);
    return nnz * (fp32 ? 25 : 32) / 100 + 270 * passes * ((max_row + lanes - 1) / lanes);
}

// Whether the inner products of a system whose configuration has `lanes` lanes
// are better taken with one lane per row, in the copy's order.
inline bool slot_one_lane(int64_t n, int64_t nnz, int64_t max_row, int lanes, int threads,
                          bool fp32) {
    return lanes == 1 || slot_copy_ns(nnz, max_row, fp32) <=
                             slot_lanes_ns(n, nnz, max_row, lanes, threads, fp32);
}

// Whether a single CG solve on a CSR-vector configuration of `lanes` lanes runs
// in one workgroup, its inner products with one lane per row or with `lanes`.
inline bool cg_in_one_workgroup(int64_t n, int64_t nnz, int64_t max_row, int lanes, bool one_lane,
                                int threads, bool fp32) {
    const int64_t product = one_lane ? slot_copy_ns(nnz, max_row, fp32)
                                     : slot_lanes_ns(n, nnz, max_row, lanes, threads, fp32);
    const int64_t steps = (max_row + lanes - 1) / lanes;
    return 4500 + product < (fp32 ? 15500 + 130 * steps : 11500 + 150 * steps);
}

// The same for GMRES(m) (at most n steps a cycle).  A cycle's start and end take the
// multi-workgroup kernels a dozen launches, so one workgroup is ahead by about
// 11,000 / m ns a step in FP64, 12,000 / m + 2,000 in mixed precision, before its
// products: the inner one and, once a cycle, the FP64 residual's.  Longer cycles lose
// it in the basis sweeps.  us a step (one workgroup, multi-workgroup, one workgroup
// before the vectors were on the chip): mixed, 4 rows, m = 30 18.8, 25.2, 21.0; 100 rows of
// three, m = 1 11.7, 26.7, 20.4, m = 10 11.1, 14.4, 16.1, m = 20 14.8, 15.2, 18.5; 2,000
// rows of 9, m = 2 21.7, 23.6, 41.3; FP64, 100 rows of three, m = 1 14.4, 26.1, 24.3,
// m = 5 14.4, 16.4, 19.2, m = 10 17.0, 15.9, 20.2; 4,000 rows of 9, m = 1 64.7, 33.3, 119.
inline bool gmres_in_one_workgroup(int64_t n, int64_t nnz, int64_t max_row, int m, int lanes,
                                   bool one_lane, int threads, bool fp32) {
    const int64_t steps = std::min<int64_t>(m, std::max<int64_t>(n, 1));
    if (steps > (fp32 ? 16 : 6))
        return false;
    const int64_t product = one_lane ? slot_copy_ns(nnz, max_row, fp32)
                                     : slot_lanes_ns(n, nnz, max_row, lanes, threads, fp32);
    const int64_t residual = slot_lanes_ns(n, nnz, max_row, lanes, threads, false);
    return product + residual / steps <= (fp32 ? 12000 / steps + 2000 : 11000 / steps);
}

}  // namespace ck
