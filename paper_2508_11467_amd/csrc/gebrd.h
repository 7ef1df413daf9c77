// Householder bidiagonal reduction, merged-rank-(2b) form (k_gebrd.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace bdc {

constexpr int kBrdMaxB = 32;             // panel width, at most (2b <= 64 columns of P, Q)
constexpr int kBrdSlot = 2 * kBrdMaxB + 2;  // values of a sum over the grid, at most
constexpr int kBrdSets = 3;              // sets of exchange places
constexpr int kBrdMaxWg = 512;           // workgroups of a grid, at most
inline int gebrd_max_block() { return kBrdMaxB; }
// exchange places of a panel: the sums' slots and totals, the column and the
// row, P's row and Q's row
inline size_t gebrd_places(int m, int n, int wgs) {
  return (size_t)kBrdSets * ((size_t)kBrdSlot * wgs + kBrdSlot + (size_t)m + n + 4 * kBrdMaxB);
}
// bytes of the panel buffers (P: m x 2b, Q^T: 2b x n) and the exchange places
// of up to max_wg workgroups
inline size_t gebrd_work_bytes(int m, int n, int b, int max_wg) {
  return 8 * ((size_t)m * 2 * b + (size_t)2 * b * n + gebrd_places(m, n, max_wg < kBrdMaxWg ? max_wg : kBrdMaxWg));
}
// A (m x n, lda, m >= n) <- d, e, the column reflectors below the diagonal
// and the row reflectors right of the superdiagonal (LAPACK's gebrd
// storage); tauq, taup (n; taup[n-1] = 0), d (n), e (n-1).  Returns BDC_OK,
// BDC_ERR_TOO_LARGE (work too small) or BDC_ERR_HIP.
int launch_gebrd(int device, int m, int n, double* A, int lda, double* tauq, double* taup, double* d, double* e,
                 int b, void* work, size_t work_bytes, int max_wg, hipStream_t st);

}  // namespace bdc
