// The 128 x 128 FP64 matrix-core tile of the large products (the vector
// update's 128 class, the plain product, the back-transformation).
//
// v_mfma_f64_16x16x4f64 keeps a SIMD's matrix core busy for 64 cycles, so a
// 16-deep slab of the tile is 4096 cycles of products per wavefront against
// 32 KB of operands: the operands are no bound, whatever stops a wavefront
// from issuing its next product is.  So two workgroups share a CU (at most
// 256 registers a lane and 74 KB of LDS each), one's products filling the
// other's barriers and epilogue, and the loop's own work is kept small: a
// slab is eight 16-byte loads per thread whose addresses are a wave-uniform
// base that moves by slab and an offset that does not, with no test of a bound
// (rows and columns past the matrix are clamped to the last one: they only
// feed outputs that are not stored).  The slab that ends K, and matrices too
// small or strides too large for that, take element loads with tests.
// The rule of the plain product below (launch_gemm_plain) has the rates.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bdc {

constexpr int kG128K = 16;    // slab depth
constexpr int kG128A = 144;   // A as [k][m]: row stride (the two k rows of a half-wavefront's read 32 banks apart)
constexpr int kG128B = 18;    // B (and a transposed A) as [n][k]: stride, 16-byte aligned

struct Gemm128Lds {
  double A[2][128 * kG128B];  // 128 * 18 = 16 * 144
  double B[2][128 * kG128B];
};
static_assert(128 * kG128B == kG128K * kG128A, "both layouts of A take the same LDS");

// a pair of doubles of any alignment a double may have
typedef double g128_pair __attribute__((ext_vector_type(2), aligned(8)));
typedef double g128_pair16 __attribute__((ext_vector_type(2)));
typedef double g128_acc __attribute__((ext_vector_type(4)));

// Tile v of a tiles_m x tiles_n product whose workgroups v, v + P, v + 2P, ...
// run on the same XCD (workgroups are dealt to the 8 XCDs in turn): each such
// class takes one contiguous run of the tiles, ordered in bands of eight tile
// rows, column by column, so the workgroups in flight on an XCD (64) share
// eight panels of A and of B in its L2.
__device__ inline void gemm128_place(int v, int P, int tiles_m, int tiles_n, int& tm, int& tn) {
  constexpr int kBand = 8;
  const int T = tiles_m * tiles_n, x = v % P;
  const int idx = x * (T / P) + min(x, T % P) + v / P;
  const int band = idx / (kBand * tiles_n), in = idx - band * kBand * tiles_n;
  const int h = min(kBand, tiles_m - band * kBand);
  tm = band * kBand + in % h;
  tn = in / h;
}

// C tile (tm0.., tn0.., TM x 128) of A (M x K) B (K x N) over k0 <= k < k1,
// all column-major; element (r, k) of A at A[r + k lda], or at A[k + r lda]
// with TRANSA.  store(row, col, value) for the tile's elements inside M x N, or,
// with Store::kReads, store(row, col, store.at(row, col), value).
// Sums run over k ascending in steps of four from k0.  256 threads.  TM = 64
// or 32 (a transposed A only) is for products of so few rows, and for sums over
// a long depth: they run in chains of CHAIN slabs (a power of two; 0: one
// chain), each from zero, which are added up one by one, so that a term passes
// through a chain's roundings and not through the whole depth's.  (A chain's
// sums and the total take two sets of accumulators, for which 128 rows have no
// registers with two workgroups per CU.)
template <bool TRANSA, int TM = 128, int CHAIN = 0, class Store>
__device__ inline void gemm128_tile(Gemm128Lds& sm, const double* __restrict__ A, int64_t lda,
                                    const double* __restrict__ B, int64_t ldb, int M, int N, int k0, int k1, int tm0,
                                    int tn0, const Store& store) {
  constexpr int TK = kG128K;
  constexpr int BA = TM / 32;  // 16 x 16 blocks of a wavefront's rows; lines of a transposed A per thread
  static_assert(TM == 128 || ((TM == 64 || TM == 32) && TRANSA), "tile");
  static_assert(CHAIN == 0 || (TM < 128 && (CHAIN & (CHAIN - 1)) == 0), "chain");
  const int t = threadIdx.x, wv = t >> 6, l = t & 63;
  const int wm = wv & 1, wn = wv >> 1;
  const int li = l & 15, lk = l >> 4;
  g128_acc acc[BA][4];
#pragma unroll
  for (int a = 0; a < BA; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = g128_acc{0.0, 0.0, 0.0, 0.0};

  // This thread's part of a slab: pairs along the contiguous dimension.
  // k-contiguous operands: k pair 2 (t & 7), lines (t >> 3) + 32 q; A as
  // stored: row pair 2 l, k = wave + 4 q.
  const int kp = 2 * (t & 7), line = t >> 3;
  uint32_t offA[4], offB[4];
  bool last_row = false;  // this pair starts at the matrix's last row: it is loaded from the row before
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    offB[q] = (uint32_t)((min(line + 32 * q, N - 1 - tn0) * ldb + kp) * 8);
    if (TRANSA && q < BA) offA[q] = (uint32_t)((min(line + 32 * q, M - 1 - tm0) * lda + kp) * 8);
  }
  if (!TRANSA) {
    const int r = min(2 * l, M - 2 - tm0);
    last_row = 2 * l == M - 1 - tm0;
    offA[0] = (uint32_t)((int64_t)r * 8);
  }
  const bool narrow = (TRANSA ? lda < (1 << 21) && k1 - k0 >= 2 : M >= 2) && ldb < (1 << 21);
  const char* const baseA = reinterpret_cast<const char*>(TRANSA ? A + (int64_t)tm0 * lda : A + tm0);
  const char* const baseB = reinterpret_cast<const char*>(B + (int64_t)tn0 * ldb);

  g128_pair ra[BA], rb[4];
  auto load = [&](int kb) {
#pragma unroll
    for (int q = 0; q < BA; ++q) {
      if (TRANSA) {
        ra[q] = *reinterpret_cast<const g128_pair*>(baseA + (int64_t)kb * 8 + offA[q]);
      } else {
        const int kw = __builtin_amdgcn_readfirstlane(kb + wv + 4 * q);
        ra[q] = *reinterpret_cast<const g128_pair*>(baseA + (int64_t)kw * lda * 8 + (int32_t)offA[0]);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) rb[q] = *reinterpret_cast<const g128_pair*>(baseB + (int64_t)kb * 8 + offB[q]);
  };
  auto load_tested = [&](int kb) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = tm0 + (TRANSA ? line + 32 * q : 2 * l + h), ka = kb + (TRANSA ? kp + h : wv + 4 * q);
        if (q < BA)
          ra[q][h] = (r < M && ka < k1) ? (TRANSA ? A[ka + (int64_t)r * lda] : A[r + (int64_t)ka * lda]) : 0.0;
        const int c = tn0 + line + 32 * q, kc = kb + kp + h;
        rb[q][h] = (c < N && kc < k1) ? B[kc + (int64_t)c * ldb] : 0.0;
      }
    }
  };
  auto stash = [&](int buf, bool shifted) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int ea = TRANSA ? (line + 32 * q) * kG128B + kp : (wv + 4 * q) * kG128A + 2 * l;
      if (q < BA)
        *reinterpret_cast<g128_pair16*>(&sm.A[buf][ea]) = g128_pair16{shifted ? ra[q].y : ra[q].x, ra[q].y};
      *reinterpret_cast<g128_pair16*>(&sm.B[buf][(line + 32 * q) * kG128B + kp]) = g128_pair16{rb[q].x, rb[q].y};
    }
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < TK; kk += 4) {
      double af[BA], bf[4];
#pragma unroll
      for (int a = 0; a < BA; ++a) {
        const int row = wm * (TM / 2) + a * 16 + li;
        af[a] = TRANSA ? sm.A[buf][row * kG128B + kk + lk] : sm.A[buf][(kk + lk) * kG128A + row];
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) bf[b] = sm.B[buf][(wn * 64 + b * 16 + li) * kG128B + kk + lk];
#pragma unroll
      for (int a = 0; a < BA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(bf[b], af[a], acc[a][b], 0, 0, 0);
    }
  };
  g128_acc total[CHAIN ? BA : 1][4];
  int slabs = 0;  // of the chain
  auto chain_end = [&] {
    if constexpr (CHAIN > 0) {
#pragma unroll
      for (int a = 0; a < BA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          total[a][b] += acc[a][b];
          acc[a][b] = g128_acc{0.0, 0.0, 0.0, 0.0};
        }
    }
  };
  auto chain_step = [&] {  // after every slab
    if constexpr (CHAIN > 0)
      if ((++slabs & (CHAIN - 1)) == 0) chain_end();
  };
  if constexpr (CHAIN > 0) {
#pragma unroll
    for (int a = 0; a < BA; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) total[a][b] = g128_acc{0.0, 0.0, 0.0, 0.0};
  }
  int kb = k0, buf = 0;
  __syncthreads();  // the previous tile's readers are done with both buffers
  const int nfull = narrow ? (k1 - k0) / TK : 0;
  if (nfull > 0) {
    load(k0);
    stash(0, last_row);
    __syncthreads();
    for (int sl = 1; sl < nfull; ++sl) {
      load(k0 + sl * TK);
      multiply(buf);
      chain_step();
      buf ^= 1;
      stash(buf, last_row);
      __syncthreads();
    }
    multiply(buf);
    chain_step();
    buf ^= 1;
    kb += nfull * TK;
  }
  for (; kb < k1; kb += TK) {
    load_tested(kb);
    stash(buf, false);
    __syncthreads();
    multiply(buf);
    chain_step();
    buf ^= 1;
  }
  chain_end();
  auto& sum = [&]() -> auto& {
    if constexpr (CHAIN > 0) return total;
    else return acc;
  }();
  // The products are taken as B^T A^T: D[i][j] of a 16x16 block sits in lane
  // j + 16 * (i % 4), register i / 4, so with i the column and j the row a
  // wavefront's access is 16 consecutive rows of four columns (whole 128-byte
  // lines, where A B would give 32 bytes of sixteen).  What the stores replace
  // is read a block row at a time, before any of its stores.
#pragma unroll
  for (int a = 0; a < BA; ++a) {
    const int row = tm0 + wm * (TM / 2) + a * 16 + li, col0 = tn0 + wn * 64 + lk;
    double old[4][4];
    if constexpr (Store::kReads) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int col = col0 + b * 16 + 4 * r;
          old[b][r] = row < M && col < N ? store.at(row, col) : 0.0;
        }
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = col0 + b * 16 + 4 * r;
        if (row >= M || col >= N) continue;
        if constexpr (Store::kReads) store(row, col, old[b][r], sum[a][b][r]);
        else store(row, col, sum[a][b][r]);
      }
  }
}

}  // namespace bdc
