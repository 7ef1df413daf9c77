// Householder QR of a tall matrix and its explicit Q (k_qr.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include "backtr.h"

namespace bdc {

// bytes of the exchange places of a panel's sums over up to max_wg workgroups
size_t qr_sync_bytes(int max_wg);
// largest panel width
int qr_max_block();
// workgroups and rows per workgroup of the panel kernel for `rows_below`
// rows under a top block of b columns (at most 10240 / b rows per
// workgroup): 0, or 1 when the rows do not fit the resident grid, -1 on a
// runtime error
int qr_panel_grid(int device, int rows_below, int b, int* grid, int* rows_per_wg);

// A (m x n, lda, m >= n) <- R above the diagonal and the reflectors below it,
// tau (n): LAPACK's geqrf storage, panels of b columns.  sync_buf: memory of
// qr_sync_bytes, whatever it holds (the first launch empties the places); plan
// and bt_scratch: for m rows and n columns, groups of b.  Returns BDC_OK,
// BDC_ERR_TOO_LARGE or BDC_ERR_HIP (launches enqueued on st).
int launch_geqrf(int device, int m, int n, double* A, int lda, double* tau, int b, void* sync_buf, size_t sync_bytes,
                 const BtPlan& plan, void* bt_scratch, hipStream_t st);

// Q (m x ncols, ldq) <- the first ncols columns of H_0 ... H_{k-1} (geqrf
// storage in A), plan.group reflectors at a time; plan and bt_scratch: for m
// rows and ncols columns
void launch_orgqr(int m, int ncols, int k, const double* A, int lda, const double* tau, double* Q, int ldq,
                  const BtPlan& plan, void* bt_scratch, hipStream_t st);

}  // namespace bdc
