// Back-transformation of singular vectors (Section 4.3.3): C <- Q C or
// Q^T C for Q = H_0 H_1 ... H_{k-1}, H_i = I - tau_i y_i y_i^T, with the
// reflectors applied a group of K at a time in the modified compact WY form
// of eq. inv_t / larft_update: for a group Y (m' x K, rows from the group's
// first pivot down),
//   T^{-1} = Y^T Y above the diagonal, 1/tau_i on it      (gemm)
//   W      = Y^T C                                        (gemm)
//   Z      = T^{-1} \ W   (Q C)  or  T^{-T} \ W  (Q^T C)  (trsm)
//   C      = C - Y Z                                      (gemm)
// since the group's product is I - Y T Y^T.  Q C takes the groups from the
// last to the first, Q^T C from the first to the last.  All products run on
// FP64 matrix cores (v_mfma_f64_16x16x4f64); the products with the long m'
// dimension as their depth (Y^T Y, Y^T C) split it over several workgroups
// whose partial sums are added in a fixed order (deterministic).
//
// The group.  C crosses HBM three times per group (read for W, read and
// written for the update), 24 bytes per entry against 4 K flops, so K = 64 is
// bound by it and wider groups by the matrix cores; but the error grows with
// the group, as the reflectors of a group see each other through the rounded
// Y^T Y alone.  Against extended precision (rms, relative to blocks of 64 with
// sums over 256 to 512 rows and one back substitution per column; 200 to 40000
// rows): groups of 512 with sums over up to 4096 rows up to 1.9 times for random
// reflectors and up to 4 times for nearly parallel ones; groups of 128 with the
// sums of Y^T [C | Y] in chains of 64 rows 0.45 to 0.9 and 0.65 to 0.95 (groups
// of 256 so up to 1.0 and 1.25).  So two 64-blocks go as one group, the triangular
// solve by 64-row blocks with inverted diagonal blocks, on the matrix cores too.
// 8192 x 8192 with 8192 reflectors: 28.1 ms with groups of 128 (the update 13.8,
// Y^T [C | Y] 12.0), 22.2 with 512, and 70.1 with 64 and one thread per column in
// the solve (113 us a block, whatever its size); 3001 x 3001: 3.00, 2.26 and
// 11.3 ms.
#include <algorithm>
#include <mutex>

#include "bdc_internal.h"
#include "backtr.h"
#include "block_util.h"
#include "gemm128.h"

namespace bdc {
namespace {

constexpr int kSolveCols = 16; // columns of W per workgroup of the solve
constexpr int kChain = 64;     // rows that the sums of Y^T [C | Y] run over at a time

struct PartStore {
  static constexpr bool kReads = false;
  double* P;
  int64_t ld;
  __device__ void operator()(int r, int c, double v) const { P[r + (int64_t)c * ld] = v; }
};
struct SubStore {
  static constexpr bool kReads = true;
  double* C;
  int64_t ld;
  __device__ double at(int r, int c) const { return C[r + (int64_t)c * ld]; }
  __device__ void operator()(int r, int c, double old, double v) const { C[r + (int64_t)c * ld] = old - v; }
};

// Rows [q0, q1) (counted from the group's first pivot r0) of the group's
// reflectors as a dense (q1 - q0) x bw matrix (column c: zeros above its
// pivot, 1 at it, the stored entries below; an all-zero column when tau = 0,
// the identity).
__global__ __launch_bounds__(256) void k_bt_pack(const double* __restrict__ Y, int64_t rs, int64_t cs,
                                                 const double* __restrict__ tau, int i0, int bw, int offset, int q0,
                                                 int q1, double* __restrict__ Yp) {
  const int r0 = i0 + offset, rows = q1 - q0;
  const int64_t total = (int64_t)rows * bw;
  const int64_t step = (int64_t)gridDim.x * 256;
  if (rs <= cs) {
    for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < total; g += step) {
      const int c = (int)(g / rows), rr = (int)(g - (int64_t)c * rows);
      const int r = r0 + q0 + rr, piv = r0 + c;
      double v = 0.0;
      if (tau[i0 + c] != 0.0) v = r < piv ? 0.0 : (r == piv ? 1.0 : Y[(int64_t)r * rs + (int64_t)(i0 + c) * cs]);
      Yp[g] = v;
    }
    return;
  }
  // row-stored reflectors: 32 x 32 tiles turned around in LDS
  __shared__ double tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int tr = (rows + 31) / 32, tc = (bw + 31) / 32;
  for (int b = blockIdx.x; b < tr * tc; b += gridDim.x) {
    const int rb = (b % tr) * 32, cb = (b / tr) * 32;
    __syncthreads();
    for (int j = ty; j < 32; j += 8) {
      const int c = cb + tx, rr = rb + j;
      double v = 0.0;
      if (c < bw && rr < rows && tau[i0 + c] != 0.0) {
        const int r = r0 + q0 + rr, piv = r0 + c;
        v = r < piv ? 0.0 : (r == piv ? 1.0 : Y[(int64_t)r * rs + (int64_t)(i0 + c) * cs]);
      }
      tile[j][tx] = v;
    }
    __syncthreads();
    for (int j = ty; j < 32; j += 8) {
      const int c = cb + j, rr = rb + tx;
      if (c < bw && rr < rows) Yp[rr + (int64_t)c * rows] = tile[tx][j];
    }
  }
}

// Y^T [C | Y] in depth slices, TM x 128 tiles: the first tiles of blockIdx.x
// are C's (slices of `slice` rows), the last ones Y's own (kTSlice
// rows; the tiles on or above the diagonal).  Tile columns 8 apart, so that
// the row tiles of one tile column (which read the same part of C) fall on one
// XCD.  Each sum runs in chains of kChain rows.
template <int TM>
__global__ __launch_bounds__(256, 2) void k_bt_ytx(const double* __restrict__ Yp, const double* __restrict__ C,
                                                   int64_t ldc, int rows, int bw, int N, int slice,
                                                   double* __restrict__ P, int cblocks, double* __restrict__ PT) {
  __shared__ Gemm128Lds sm;
  const int tr = (bw + TM - 1) / TM;
  const bool own = (int)blockIdx.x >= cblocks;  // a tile of Y^T Y
  const int tc = ((own ? bw : N) + 127) / 128;
  int z, r, c;
  if (own) {
    const int b = blockIdx.x - cblocks, per = tr * tc;
    z = b / per, r = (b % per) % tr, c = (b % per) / tr;
    if (r * TM >= (c + 1) * 128) return;
  } else {
    const int band = 8 * tr, per = ((tc + 7) / 8) * band, b = blockIdx.x % per;
    z = blockIdx.x / per, r = (b % band) / 8, c = (b / band) * 8 + b % 8;
    if (c >= tc) return;
  }
  const int len = own ? kTSlice : slice, k0 = z * len, k1 = min(rows, k0 + len);
  gemm128_tile<true, TM, kChain / kG128K>(sm, Yp, rows, own ? Yp : C, own ? (int64_t)rows : ldc, bw, own ? bw : N, k0,
                                          k1, r * TM, c * 128,
                                          PartStore{own ? PT + (int64_t)z * bw * bw : P + (int64_t)z * bw * N, bw});
}

// out += the slices in order (out starts at zero with first)
__global__ __launch_bounds__(256) void k_bt_accumulate(const double* __restrict__ P, int64_t stride, int slices,
                                                       int first, double* __restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= stride) return;
  double s = first ? 0.0 : out[g];
  for (int z = 0; z < slices; ++z) s += P[z * stride + g];
  out[g] = s;
}

// T^{-1} from the slices of Y^T Y (added in order to prev, if any): the
// strictly upper part, 1/tau on the diagonal (1 for a tau = 0 identity).  A
// workgroup per 64 x 64 block on or above the diagonal writes it to Ti (ld
// bw); for a diagonal block it also writes the block's inverse to Di (ld db =
// min(64, bw), db x db each): 16 x 16 diagonal blocks by back substitution, a thread per column,
// then the blocks above them distance by distance.
__global__ __launch_bounds__(1024) void k_bt_tinv(const double* __restrict__ PT, int slices,
                                                 const double* __restrict__ prev, const double* __restrict__ tau,
                                                 int bw, double* __restrict__ Ti, double* __restrict__ Di) {
  constexpr int S = kTB + 1;
  __shared__ double U[kTB * S], X[kTB * S], D[3][16 * 17];
  const int nb = (bw + kTB - 1) / kTB, t = threadIdx.x;
  int bi = 0, bj = blockIdx.x;
  while (bj >= nb - bi) bj -= nb - bi++;
  bj += bi;
  const int64_t stride = (int64_t)bw * bw;
  // 4 entries per thread, the loads of a slice (of several, unrolled) in flight together
  const int lr = t % kTB, r0 = bi * kTB + lr;
  double v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = bj * kTB + t / kTB + 16 * q;
    v[q] = prev && r0 < c && c < bw ? prev[r0 + (int64_t)c * bw] : 0.0;
  }
#pragma unroll 4
  for (int z = 0; z < slices; ++z)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = bj * kTB + t / kTB + 16 * q;
      v[q] += r0 < c && c < bw ? PT[z * stride + r0 + (int64_t)c * bw] : 0.0;
    }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int lc = t / kTB + 16 * q, c = bj * kTB + lc;
    if (r0 == c) v[q] = r0 < bw && tau[r0] != 0.0 ? 1.0 / tau[r0] : 1.0;  // past the group: an identity
    if (r0 > c) v[q] = 0.0;
    if (r0 < bw && c < bw) Ti[r0 + (int64_t)c * bw] = v[q];
    U[lr * S + lc] = v[q];
    X[lr * S + lc] = 0.0;
  }
  if (bi != bj) return;
  __syncthreads();
  if (t < kTB) {
    const int b = t & ~15, c = t & 15;
    double x[16];
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      double s = i == c ? 1.0 : 0.0;
#pragma unroll
      for (int j = i + 1; j < 16; ++j) s -= U[(b + i) * S + b + j] * x[j];
      x[i] = s / U[(b + i) * S + b + i];
      X[(b + i) * S + b + c] = x[i];
    }
  }
  const int r = t & 15, c = (t >> 4) & 15, i = t >> 8;  // 256 threads per block pair
  for (int dist = 1; dist < 4; ++dist) {
    __syncthreads();
    if (i + dist < 4) {
      double s = 0.0;
      for (int k = 16 * (i + 1); k < 16 * (i + dist + 1); ++k)
        s += U[(16 * i + r) * S + k] * X[k * S + 16 * (i + dist) + c];
      D[i][r * 17 + c] = s;
    }
    __syncthreads();
    if (i + dist < 4) {
      double s = 0.0;
      for (int k = 0; k < 16; ++k) s += X[(16 * i + r) * S + 16 * i + k] * D[i][k * 17 + c];
      X[(16 * i + r) * S + 16 * (i + dist) + c] = -s;
    }
  }
  __syncthreads();
  const int db = min(kTB, bw);
  for (int e = t; e < db * db; e += 1024) Di[(int64_t)bi * db * db + e] = X[(e % db) * S + e / db];
}

// Z = T^{-1} \ W (upper, from the last 64-row block up) or T^{-T} \ W (lower,
// from the first block down); W is the sum of prev (if any) and the slices, in
// order.  A chain of block rows, so it is bound by latency: a block's
// operands are read together, 17 us for 128 x 8192 (256 x 8192: 35, and 70 with
// eight loads in flight), and 16 columns to a workgroup keep the chip's CUs
// in it.  kSolveCols columns per workgroup in LDS; for each block row the
// products with the blocks solved before it, then with the inverted diagonal
// block, 16 rows per wavefront.
template <bool TRANS>
__global__ __launch_bounds__(256) void k_bt_solve(const double* __restrict__ P, int slices,
                                                  const double* __restrict__ prev, const double* __restrict__ Ti,
                                                  const double* __restrict__ Di, int bw, int N,
                                                  double* __restrict__ Z) {
  constexpr int S = kBtMaxGroup + 2;
  __shared__ double sw[kSolveCols * S];
  const int t = threadIdx.x, wv = t >> 6, l = t & 63, li = l & 15, lk = l >> 4;
  const int c0 = blockIdx.x * kSolveCols;
  const int nb = (bw + kTB - 1) / kTB, pad = nb * kTB;
  const int64_t stride = (int64_t)bw * N;
  // 8 entries per thread at a time, their loads in flight together (pad is
  // a multiple of 64, so a wavefront stays in a column)
  for (int e0 = t; e0 < pad * kSolveCols; e0 += 8 * 256) {
    double v[8];
    int64_t g[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + 256 * u, r = e % pad, c = e / pad;
      g[u] = c < kSolveCols && r < bw && c0 + c < N ? r + (int64_t)(c0 + c) * bw : -1;
      v[u] = prev && g[u] >= 0 ? prev[g[u]] : 0.0;
    }
#pragma unroll 2
    for (int z = 0; z < slices; ++z)
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] += g[u] >= 0 ? P[z * stride + g[u]] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + 256 * u;
      if (e < pad * kSolveCols) sw[(e / pad) * S + e % pad] = v[u];
    }
  }
  __syncthreads();
  const int db = min(kTB, bw);
  for (int q = 0; q < nb; ++q) {
    const int i = TRANS ? q : nb - 1 - q;
    const int row = i * kTB + wv * 16 + li;
    const int j0 = TRANS ? 0 : i + 1, j1 = TRANS ? i : nb;
    // a block's 16 operands per lane are read together; the inverted
    // diagonal block's before the products that precede it
    double d[16], a[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int kk = 4 * k + lk, rr = wv * 16 + li;
      d[k] = (rr < db && kk < db) ? Di[(int64_t)i * db * db + (TRANS ? kk + rr * db : rr + kk * db)] : 0.0;
    }
    if (j0 < j1) {
      g128_acc acc[kSolveCols / 16] = {};
      for (int j = j0; j < j1; ++j) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const int kk = j * kTB + 4 * k + lk;
          a[k] = (row < bw && kk < bw) ? (TRANS ? Ti[kk + (int64_t)row * bw] : Ti[row + (int64_t)kk * bw]) : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
          for (int b = 0; b < kSolveCols / 16; ++b)
            acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k], sw[(b * 16 + li) * S + j * kTB + 4 * k + lk], acc[b], 0,
                                                          0, 0);
      }
      // this wavefront's 16 rows only; the products above read other blocks
#pragma unroll
      for (int b = 0; b < kSolveCols / 16; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) sw[(b * 16 + li) * S + i * kTB + wv * 16 + lk + 4 * r] -= acc[b][r];
      __syncthreads();
    }
    g128_acc acc[kSolveCols / 16] = {};
#pragma unroll
    for (int k = 0; k < 16; ++k)
#pragma unroll
      for (int b = 0; b < kSolveCols / 16; ++b)
        acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[k], sw[(b * 16 + li) * S + i * kTB + 4 * k + lk], acc[b], 0, 0,
                                                      0);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < kSolveCols / 16; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) sw[(b * 16 + li) * S + i * kTB + wv * 16 + lk + 4 * r] = acc[b][r];
    __syncthreads();
  }
  for (int e = t; e < bw * kSolveCols; e += 256) {
    const int r = e % bw, c = e / bw;
    if (c0 + c < N) Z[r + (int64_t)(c0 + c) * bw] = sw[c * S + r];
  }
}

// C (rows x N) -= Yp (rows x K) Z (K x N, ld ldz).
__global__ __launch_bounds__(256, 2) void k_bt_update(const double* __restrict__ Yp, int ldp,
                                                      const double* __restrict__ Z, int ldz, int K,
                                                      double* __restrict__ C, int64_t ldc, int rows, int N) {
  __shared__ Gemm128Lds sm;
  int tm, tn;
  gemm128_place(blockIdx.x, 8, (rows + 127) / 128, (N + 127) / 128, tm, tn);
  gemm128_tile<false>(sm, Yp, ldp, Z, ldz, rows, N, 0, K, tm * 128, tn * 128, SubStore{C, ldc});
}

}  // namespace

void launch_backtr(int trans, int m, int p, int k, int offset, const double* Y, int64_t rs, int64_t cs,
                   const double* tau, double* C, int ldc, const BtPlan& plan, void* scratch, hipStream_t st) {
  double* base = (double*)scratch;
  double *Yp = base + plan.yp, *P = base + plan.p, *PT = base + plan.pt, *Ti = base + plan.ti, *Di = base + plan.di,
         *Z = base + plan.z;
  const int K = plan.group;
  const int ngrp = (k + K - 1) / K;
  for (int q = 0; q < ngrp; ++q) {
    const int j = trans ? q : ngrp - 1 - q;
    const int i0 = j * K;
    const int r0 = i0 + offset;
    if (r0 >= m) continue;  // reflectors past the last row: identities
    const int rows = m - r0;
    const int bw = std::min({K, k - i0, rows});  // (also within a group)
    const int slice = bt_slice(rows, p, bw);
    // rows of a chunk: whole slices of W and of Y^T Y (both powers of two)
    // rows of a chunk: whole slices of W
    const int chunk = plan.fixed ? slice * std::min(kBtChunk / slice, plan.slices) : rows;
    const int nchunk = (rows + chunk - 1) / chunk;
    const int tm = bt_tile_rows(bw), tr = (bw + tm - 1) / tm, tt = (bw + 127) / 128;
    auto pack = [&](int q0, int q1) {
      const int64_t tot = (int64_t)(q1 - q0) * bw;
      hipLaunchKernelGGL(k_bt_pack, dim3((unsigned)std::min<int64_t>((tot + 255) / 256, 4096)), dim3(256), 0, st, Y,
                         rs, cs, tau, i0, bw, offset, q0, q1, Yp);
    };
    // Y^T [X | Y] over cr packed rows: nz slices of W, nzt of Y^T Y
    auto ytx = [&](const double* X, int pw, int cr, int nz, int nzt) {
      const int cblocks = ((pw + 127) / 128 + 7) / 8 * 8 * tr * nz;
      const dim3 grid(cblocks + tr * tt * nzt);
      hipLaunchKernelGGL(tm == 32 ? k_bt_ytx<32> : k_bt_ytx<64>, grid, dim3(256), 0, st, Yp, X, (int64_t)ldc, cr, bw,
                         pw, slice, P, cblocks, PT);
    };
    auto accumulate = [&](const double* part, int64_t n, int slices, bool first, double* sum) {
      hipLaunchKernelGGL(k_bt_accumulate, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part, n, slices, first,
                         sum);
    };
    int nzt = (rows + kTSlice - 1) / kTSlice;
    const bool tchunks = plan.fixed && (rows > kBtChunkT || nchunk > 1);
    if (nchunk == 1 && !tchunks) pack(0, rows);
    if (tchunks) {
      // Y^T Y by chunks of its own slices (packed over again)
      for (int q0 = 0; q0 < rows; q0 += kBtChunkT) {
        const int q1 = std::min(rows, q0 + kBtChunkT);
        nzt = (q1 - q0 + kTSlice - 1) / kTSlice;
        pack(q0, q1);
        ytx(nullptr, 0, q1 - q0, 0, nzt);
        if (q1 < rows) accumulate(PT, (int64_t)bw * bw, nzt, q0 == 0, base + plan.tsum);
      }
      if (nchunk == 1) pack(0, rows);
    }
    // the columns of C in panels (every column is transformed on its own, so
    // the panels give the same results)
    for (int c0 = 0; c0 < p; c0 += plan.panel) {
      const int pw = std::min(plan.panel, p - c0);
      double* Cb = C + r0 + (int64_t)c0 * ldc;
      int nz = 0;
      for (int q0 = 0; q0 < rows; q0 += chunk) {
        const int q1 = std::min(rows, q0 + chunk);
        nz = (q1 - q0 + slice - 1) / slice;
        if (nchunk > 1) pack(q0, q1);
        ytx(Cb + q0, pw, q1 - q0, nz, !tchunks && q0 == 0 && c0 == 0 ? nzt : 0);
        if (q1 < rows) accumulate(P, (int64_t)bw * pw, nz, q0 == 0, base + plan.wsum);
      }
      const int nb = (bw + kTB - 1) / kTB;
      if (c0 == 0)
        hipLaunchKernelGGL(k_bt_tinv, dim3(nb * (nb + 1) / 2), dim3(1024), 0, st, PT, nzt,
                           tchunks && rows > kBtChunkT ? base + plan.tsum : nullptr, tau + i0, bw, Ti, Di);
      const double* wsum = nchunk > 1 ? base + plan.wsum : nullptr;
      const dim3 sgrid((pw + kSolveCols - 1) / kSolveCols);
      if (trans)
        hipLaunchKernelGGL(k_bt_solve<true>, sgrid, dim3(256), 0, st, P, nz, wsum, Ti, Di, bw, pw, Z);
      else
        hipLaunchKernelGGL(k_bt_solve<false>, sgrid, dim3(256), 0, st, P, nz, wsum, Ti, Di, bw, pw, Z);
      for (int q0 = 0; q0 < rows; q0 += chunk) {
        const int q1 = std::min(rows, q0 + chunk);
        if (nchunk > 1) pack(q0, q1);
        launch_sub_product(q1 - q0, pw, bw, Yp, q1 - q0, Z, bw, Cb + q0, ldc, st);
      }
    }
  }
}

void launch_sub_product(int rows, int N, int K, const double* Y, int ldy, const double* Z, int ldz, double* C,
                        int ldc, hipStream_t st) {
  if (rows <= 0 || N <= 0 || K <= 0) return;
  const int64_t tiles = (int64_t)((rows + 127) / 128) * ((N + 127) / 128);
  hipLaunchKernelGGL(k_bt_update, dim3((unsigned)tiles), dim3(256), 0, st, Y, ldy, Z, ldz, K, C, (int64_t)ldc, rows,
                     N);
}

// ---------------------------------------------------------------- fixed scratch
// Device memory of the allocation-free entry point: one array per GPU, held
// until the process ends.  Host code never passes `scratch` itself to a
// kernel (on the host the name stands for a host-side shadow, not a device
// address); it passes the address hipGetSymbolAddress returns for the
// current device.
static __device__ __align__(256) char scratch[kBtFixedScratchBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kBtMaxDevices] = {};
bool g_scratch_done[kBtMaxDevices] = {};
}  // namespace

void* backtr_fixed_scratch(int device) {
  if (device < 0 || device >= kBtMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_done[device]) {
    // once per device, with that device current (the caller's guard)
    void* ptr = nullptr;
    const hipError_t rc = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    g_scratch_ptr[device] = rc == hipSuccess ? ptr : nullptr;
    g_scratch_done[device] = true;
  }
  return g_scratch_ptr[device];
}

}  // namespace bdc
