// Back-transformation of singular vectors by blocks of Householder
// reflectors in the modified compact WY form (k_backtr.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace bdc {

constexpr int kBtMaxBlock = 64;  // reflectors per block, at most
constexpr int kBtMaxGroup = 128; // reflectors applied together, at most (two blocks of 64)

// the allocation-free entry point: a fixed 32 MiB of device memory per GPU,
// C taken in panels of at most 512 columns
constexpr size_t kBtFixedScratchBytes = size_t(32) << 20;
constexpr int kBtFixedPanel = 512;
constexpr int kBtFixedWidth = 256;  // columns at a time within the fixed scratch
constexpr int kBtMaxDevices = 64;

constexpr int kTB = 64;                // block of the triangular solve
constexpr int kTSlice = 512;           // depth slice of Y^T Y
constexpr int kBtSliceRows = 4096;     // rows of a slice of W, at most
constexpr int kBtChunk = kBtSliceRows; // the fixed scratch: rows of a chunk
constexpr int kBtChunkT = 2 * kTSlice; // and of a chunk of Y^T Y

// Scratch of one back-transformation: offsets in doubles, all bytes.
struct BtPlan {
  int group, panel;  // reflectors applied together; columns of C at a time
  bool fixed;        // rows in chunks whose scratch does not grow with m (the same sums)
  int slices;        // depth slices of a chunk, at most (fixed)
  size_t yp, p, pt, wsum, tsum, ti, di, z;
  size_t bytes;
};
// bytes that bound the allocation-free entry point's problems, and that any
// problem can be run in (group = block, fixed)
size_t backtr_limit_bytes(int m, int panel, int block);
// reflectors applied together for a block size and k reflectors in all: scratch
// and depth slices go with it, so no more whole blocks than there are (with a
// full group a million rows and 4 reflectors took twice the scratch)
inline int backtr_group(int block, int k) {
  if (block < kBtMaxBlock) return block;
  return k <= kBtMaxBlock ? kBtMaxBlock : kBtMaxGroup;
}
BtPlan backtr_plan(int m, int p, int panel, int group, bool fixed);
// rows of a tile of Y^T [C | Y] for K reflectors
constexpr int bt_tile_rows(int K) { return K <= 32 ? 32 : 64; }
// depth slice of W for `rows` rows, p columns and groups of K
int bt_slice(int rows, int p, int K);

// C (m x p, ldc) <- Q C (trans 0) or Q^T C (trans 1), Q = H_0 ... H_{k-1};
// reflector i has its unit pivot at row i + offset, zeros above, and entry r
// below at Y[r * rs + i * cs]; tau[i] = 0 makes H_i the identity.  Groups of
// plan.group reflectors from a plan made for at least m rows and p columns
// (exactly p when its panel is narrower).  Panels and chunks give the same
// results as one piece, bit for bit.
void launch_backtr(int trans, int m, int p, int k, int offset, const double* Y, int64_t rs, int64_t cs,
                   const double* tau, double* C, int ldc, const BtPlan& plan, void* scratch, hipStream_t st);

// C (rows x N, ldc) -= Y (rows x K, ldy) Z (K x N, ldz), column-major, on the
// FP64 matrix cores
void launch_sub_product(int rows, int N, int K, const double* Y, int ldy, const double* Z, int ldz, double* C,
                        int ldc, hipStream_t st);

// device address of the fixed scratch on `device` (which must be current),
// looked up once per device; nullptr if the lookup failed
void* backtr_fixed_scratch(int device);

}  // namespace bdc
