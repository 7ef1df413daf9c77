// Reduction of a dense m x n matrix (m >= n) to upper bidiagonal form
// B = Q^T A P by Householder reflectors (Section 4.1), blocked as the
// merged-rank-(2b) gebrd of Algorithm 1: every panel of b columns and rows
// is reduced by the labrd loop, which keeps the trailing matrix at its
// panel-start value and collects P = [v_1, x_1, ..., v_b, x_b] and
// Q = [y_1, u_1, ..., y_b, u_b] so that the reduced matrix is A - P Q^T
// (eq. bidiag-A-trail3); the trailing matrix is then updated by that one
// product.  Inside labrd (eq. bidiag-y-k3, bidiag-x-k3), column c:
//   (a) column c <- column c - P Q[c, :]^T;
//   (b) the reflector of its part from the diagonal down (Section 4.1:
//       beta = -sign(alpha) ||x||, v = x / (alpha - beta) below the pivot,
//       tau = 2 / v^T v), then y = tau (A^T v - Q (P^T v));
//   (c) row c <- row c - P[c, :] Q^T;
//   (d) the reflector of its part right of the diagonal, u, pi, then
//       x = pi (A u - P (Q^T u)),
// where A is the panel-start trailing matrix (its two matrix-vector
// products are the only passes over it).  One cooperative grid runs the
// whole panel: workgroup g owns a slice of the rows (of A and P) and a slice
// of the columns (of A and Q), and what workgroups need of each other goes
// through single-writer places of device memory (grid_sync.h): the unscaled
// column x and P's row c, the unscaled row and Q's row c + 1, and two sums over
// the grid per column, added in a fixed order (deterministic): after (a)
// ||x||^2, alpha and P^T x together (P^T v is P's pivot row plus the
// reflector's scale times P^T x), after (c) the row's ||x||^2, alpha and Q^T x.
// Everything else a workgroup reads it has written itself, so the caches stay
// valid across the sums (a trailing matrix of a few MB per XCD stays in its
// L2).
//
// What bounds it: the two passes read the trailing matrix twice per column
// (16 bytes per entry, 5 flops), and the exchanges are a chain of four
// round trips through memory per column.  The passes load 16 bytes per lane,
// 16 in flight.  4096 x 4096 (mean per column): see launch_gebrd.
// Storage as LAPACK's gebrd: d and e on the bidiagonal, v below the diagonal
// (unit pivot at row c), u right of the superdiagonal (unit pivot at column
// c + 1), tauq, taup.
#include <algorithm>

#include "bdc_internal.h"
#include "backtr.h"
#include "block_util.h"
#include "gebrd.h"
#include "grid_sync.h"

namespace bdc {
namespace {

constexpr int kSlot = kBrdSlot;
static_assert(kBrdSets == kGridSets && kBrdMaxWg == kGridMaxWg, "exchange places");

struct BrdLds {
  double q[kSlot];              // partial sums, then totals
  double qc[2 * kBrdMaxB];      // Q's row c (column c of Q^T)
  double pc[2 * kBrdMaxB];      // P's row c
  double pv[2 * kBrdMaxB + 2];  // P^T v, then Q^T u
  double xa[16];                // x of 16 rows
  double red[4 * 64];
  double sc[8];
  unsigned bad;
};

// The exchange places of a panel: kGridSets of each, all empty at its start.
struct BrdX {
  double* slots;   // kSlot x G
  double* totals;  // kSlot
  double* x;       // m: column c below its pivot, unscaled
  double* pc;      // 64: P's row c
  double* u;       // n: row c right of its pivot, unscaled
  double* qc;      // 64: Q's row c + 1
};

// a pair of doubles of any alignment a double may have
typedef double pair8 __attribute__((ext_vector_type(2), aligned(8)));

struct Refl {
  double beta, tau, scale;
};

// Householder reflector of (alpha, x) with sigma = ||x||^2 (Section 4.1)
__device__ inline Refl reflector(double alpha, double sigma) {
  Refl r{alpha, 0.0, 0.0};
  if (sigma > 0.0) {
    const double nrm = sqrt(alpha * alpha + sigma);
    r.beta = -copysign(nrm, alpha);
    const double den = alpha - r.beta;
    r.scale = 1.0 / den;
    r.tau = 2.0 / (1.0 + sigma / (den * den));
  }
  return r;
}

__global__ __launch_bounds__(256, 1) void k_brd_panel(double* __restrict__ A, int64_t lda, int m, int n, int j0,
                                                      int bw, double* __restrict__ P, int64_t ldp,
                                                      double* __restrict__ Qt, int ldq, double* __restrict__ tauq,
                                                      double* __restrict__ taup, double* __restrict__ dv,
                                                      double* __restrict__ ev, BrdX X, int rows_per_wg,
                                                      int cols_per_wg) {
  __shared__ BrdLds L;
  const int t = threadIdx.x, G = gridDim.x, g = blockIdx.x;
  const int ln = t & 63, wv = t >> 6;
  const int rlo = j0 + g * rows_per_wg, rhi = min(m, rlo + rows_per_wg);
  const int clo = j0 + g * cols_per_wg, chi = min(n, clo + cols_per_wg);
  bool ok = true;         // no wait of this thread has expired
  int set = 0, last = 0;  // the next sum's set; values of the last one
  double* prev = nullptr;
  // L.q[0, cnt) <- its totals over the grid
  auto grid_reduce = [&](int cnt) -> bool {
    if (!ok) L.bad = 1;
    __syncthreads();
    double* tot = X.totals + set * kSlot;
    const bool done = grid_sum<256>(X.slots + (size_t)set * kSlot * G, tot, prev, last, cnt, L.q, &L.bad);
    prev = tot;
    last = cnt;
    set = set == kGridSets - 1 ? 0 : set + 1;
    return done;
  };
  if (t == 0) L.bad = 0;
  int xs = 0;  // the column's set of x, pc, u and qc
  // with at most 16 owned rows and columns the unscaled entries stay in a
  // thread's register until their scale is known, else in A, P and Q
  const bool held = rows_per_wg <= 16 && cols_per_wg <= 16;
  for (int i = 0; i < bw; ++i, xs = xs == kGridSets - 1 ? 0 : xs + 1) {
    const int c = j0 + i, nP = 2 * i;
    double* const xv = X.x + (size_t)xs * m;
    double* const uv = X.u + (size_t)xs * n;
    double* const xpc = X.pc + xs * 2 * kBrdMaxB;
    double* const xqc = X.qc + xs * 2 * kBrdMaxB;
    // ---- (a) column c from row c down (owned rows): x = A[:, c] - P Q[c, :]^T,
    // unscaled to x's places (L.qc is the last column's)
    if (t == 0) L.q[1] = 0.0;
    grid_settle();
    __syncthreads();
    // 16 rows at a time.  Thread (rr, cg) holds P[r, q] for q = cg + 16 j
    // (registers): first the 2i products of the row, added over the 16
    // groups in a fixed order, then, once x_r is known, its share of P^T x
    // (rows below the pivot), added over the 16 rows
    const int rr = t & 15, cg = t >> 4;
    double sg = 0.0, xheld = 0.0, uheld = 0.0;
    double ptx[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r0 = max(rlo, c); r0 < rhi; r0 += 16) {
      const int r = r0 + rr;
      double pr[4], s = 0.0;
      const double arc = t < 16 && r0 + t < rhi ? A[r0 + t + (int64_t)c * lda] : 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = cg + 16 * j;
        pr[j] = (r < rhi && q < nP) ? P[r + (int64_t)q * ldp] : 0.0;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = cg + 16 * j;
        if (q < nP) s += pr[j] * L.qc[q];
        if (r == c && q < nP) grid_put(xpc + q, pr[j]);
      }
      L.red[cg * 16 + rr] = s;
      __syncthreads();
      if (t < 16) {
        const int rw = r0 + t;
        double xr = 0.0;
        if (rw < rhi) {
          double acc = 0.0;
          for (int p = 0; p < 16; ++p) acc += L.red[p * 16 + t];
          const double a = arc - acc;
          if (rw > c) {
            sg += a * a;
            xr = a;
            grid_put(xv + rw, a);
            xheld = a;
            if (!held) {
              A[rw + (int64_t)c * lda] = a;
              P[rw + (int64_t)nP * ldp] = a;
            }
          } else {
            L.q[1] = a;  // alpha, from the pivot row's owner
            P[rw + (int64_t)nP * ldp] = 1.0;
          }
        }
        L.xa[t] = xr;
      }
      __syncthreads();
      const double xr = L.xa[rr];
#pragma unroll
      for (int j = 0; j < 4; ++j) ptx[j] += pr[j] * xr;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double v = row_sum(ptx[j]);
      const int q = cg + 16 * j;
      if (rr == 0 && q < nP) L.q[2 + q] = v;
    }
    if (wv == 0) {
      sg = wave_sum_last(sg);
      if (ln == 63) L.q[0] = sg;
    }
    if (!grid_reduce(2 + nP)) return;
    const Refl h = reflector(L.q[1], L.q[0]);
    // P's row c is on its way while the pass below runs
    const unsigned long long pcb = t < nP ? grid_peek(xpc + t) : 0ull;
    const double ptv = t < nP ? L.q[2 + t] : 0.0;
    if (t == 0) {
      if (rlo <= c && c < rhi) A[c + (int64_t)c * lda] = h.beta;
      if (g == 0) {
        tauq[c] = h.tau;
        dv[c] = h.beta;
      }
    }
    // v: the owned entries; and the last column's u and qc, which everybody
    // has read (this sum is past)
    if (held) {
      const int r = max(rlo, c) + t;
      if (t < 16 && r > c && r < rhi) {
        P[r + (int64_t)nP * ldp] = xheld * h.scale;
        A[r + (int64_t)c * lda] = xheld * h.scale;
      }
    } else {
      for (int r = max(rlo, c + 1) + t; r < rhi; r += 256) {
        P[r + (int64_t)nP * ldp] *= h.scale;
        A[r + (int64_t)c * lda] *= h.scale;
      }
    }
    if (i > 0) {
      const int ps = xs == 0 ? kGridSets - 1 : xs - 1;
      for (int k = max(clo, c + 1) + t; k < chi; k += 256) grid_clear(X.u + (size_t)ps * n + k);
      if (clo <= c && c < chi && t < 2 * kBrdMaxB) grid_clear(X.qc + ps * 2 * kBrdMaxB + t);
    }
    __syncthreads();
    // ---- (b) y = tau (A^T v - Q (P^T v)) on the owned columns k > c, and
    // (c) row c there: x_k = A[c, k] - y_k - P[c, :] Q[k, :]^T, stored
    // unscaled in A's row c, Q's column nP + 1 (1 at the pivot) and u's places.
    // 16 owned columns at a time: every thread accumulates A^T v over its
    // row pairs for all 16 (16 loads of 16 bytes in flight), added over the
    // waves in a fixed order; then thread (kk, qg) finishes column kk with q =
    // qg + 16 j of Q's row (registers): the products with P^T v and P's row c
    // over the 16 lanes, and its share of Q^T x (q <= nP, Q's column nP being
    // y) for the columns right of the pivot
    const int kk = t >> 4, qg = t & 15;
    double qtx[4] = {0.0, 0.0, 0.0, 0.0};
    double sg2 = 0.0;
    if (t == 0) L.q[1] = 0.0;
    for (int kb = max(clo, c + 1); kb < chi; kb += 16) {
      const int nk = min(16, chi - kb);
      double acc[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] = 0.0;
      // unconditional loads (columns past the owned ones clamped to the last
      // and not used), so all 16 are in flight before the first product; the
      // pair that would start at the last row is loaded from the row before
      const double* Ab = A + (int64_t)kb * lda;
      int64_t col[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) col[j] = (int64_t)min(j, nk - 1) * lda;
      const int k = kb + kk;
      const bool live = kk < nk;  // uniform over each 16-lane group
      double q4[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = qg + 16 * j;
        q4[j] = (live && q < nP) ? Qt[q + (int64_t)k * ldq] : 0.0;
      }
      const double ack = live ? A[c + (int64_t)k * lda] : 0.0;
      for (int r = c + 2 * t; r < m; r += 512) {
        const bool alone = r == m - 1;
        const int rl = alone ? r - 1 : r;
        const unsigned long long x0 = r == c ? 0ull : grid_peek(xv + r);
        const unsigned long long x1 = alone ? 0ull : grid_peek(xv + r + 1);
        pair8 av[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) av[j] = *reinterpret_cast<const pair8*>(Ab + rl + col[j]);
        const double v0 = r == c ? 1.0 : grid_take(xv + r, x0, ok) * h.scale;
        const double v1 = alone ? v0 : grid_take(xv + r + 1, x1, ok) * h.scale;
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = fma(av[j].y, v1, fma(alone ? 0.0 : av[j].x, v0, acc[j]));
      }
      if (t < nP && kb == max(clo, c + 1)) {
        const double pc = grid_take(xpc + t, pcb, ok);
        L.pc[t] = pc;
        L.pv[t] = pc + h.scale * ptv;  // P^T v
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double v = wave_sum_last(acc[j]);
        if (ln == 63) L.red[wv * 16 + j] = v;
      }
      grid_settle();
      __syncthreads();
      double d1 = 0.0, d2 = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = qg + 16 * j;
        if (q < nP) {
          d1 += q4[j] * L.pv[q];
          d2 += L.pc[q] * q4[j];
        }
      }
      d1 = row_sum(d1);
      d2 = row_sum(d2);
      if (live) {
        const double s = (L.red[kk] + L.red[16 + kk]) + (L.red[32 + kk] + L.red[48 + kk]);
        const double y = h.tau * (s - d1);
        const double a = ack - y - d2;
        if (qg == 0) {
          if (k == c + 1) {
            L.q[1] = a;
          } else {
            grid_put(uv + k, a);
            sg2 += a * a;
          }
          Qt[nP + (int64_t)k * ldq] = y;
          uheld = a;
          if (!held || k == c + 1) {
            A[c + (int64_t)k * lda] = a;
            Qt[nP + 1 + (int64_t)k * ldq] = k == c + 1 ? 1.0 : a;
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int q = qg + 16 * j;
          const double v = q == nP ? y : q4[j];
          if (k > c + 1) qtx[j] += v * a;
          else if (q <= nP) grid_put(xqc + q, v);  // Q's row c + 1
        }
      }
      __syncthreads();  // L.red
    }
    if (c + 1 >= n) {  // the last column: no row reflector
      if (g == 0 && t == 0) taup[c] = 0.0;
      return;
    }
    // Q^T x: over the 4 columns of a wave (lanes 16 and 32 apart), then
    // over the waves in a fixed order
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double v = qtx[j];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (ln < 16) L.red[wv * 64 + qg + 16 * j] = v;
    }
    sg2 = wave_sum_last(sg2);
    if (ln == 63) L.sc[wv] = sg2;
    __syncthreads();
    if (t <= nP) L.q[2 + t] = (L.red[t] + L.red[64 + t]) + (L.red[128 + t] + L.red[192 + t]);
    if (t == 0) L.q[0] = (L.sc[0] + L.sc[1]) + (L.sc[2] + L.sc[3]);
    if (!grid_reduce(3 + nP)) return;
    const Refl gr = reflector(L.q[1], L.q[0]);
    const unsigned long long qcb = t <= nP ? grid_peek(xqc + t) : 0ull;
    const double qtu = t <= nP ? L.q[2 + t] : 0.0;
    if (t == 0) {
      if (clo <= c + 1 && c + 1 < chi) A[c + (int64_t)(c + 1) * lda] = gr.beta;
      if (g == 0) {
        taup[c] = gr.tau;
        ev[c] = gr.beta;
      }
    }
    // u: the owned entries; and this column's x and pc, which everybody has
    // read
    if (held) {
      const int k = max(clo, c + 1) + kk;
      if (qg == 0 && k > c + 1 && k < chi) {
        Qt[nP + 1 + (int64_t)k * ldq] = uheld * gr.scale;
        A[c + (int64_t)k * lda] = uheld * gr.scale;
      }
    } else {
      for (int k = max(clo, c + 2) + t; k < chi; k += 256) {
        Qt[nP + 1 + (int64_t)k * ldq] *= gr.scale;
        A[c + (int64_t)k * lda] *= gr.scale;
      }
    }
    for (int r = max(rlo, c + 1) + t; r < rhi; r += 256) grid_clear(xv + r);
    if (rlo <= c && c < rhi && t < 2 * kBrdMaxB) grid_clear(xpc + t);
    __syncthreads();
    // ---- (d) x = pi (A u - P (Q^T u)) on the owned rows r > c: 16 rows at
    // a time, 8 lanes with a row pair each, the columns of A and of P split
    // over 32 groups of lanes, added over a wave's 8 groups and then over the
    // waves in a fixed order
    const int rp = t & 7, kg = t >> 3;
    for (int r0 = max(rlo, c + 1); r0 < rhi; r0 += 16) {
      // rows past the owned ones are clamped to the last pair and not used;
      // the columns go in batches of 16 unconditional loads (past n: clamped)
      const int r = min(r0 + 2 * rp, m - 2);
      double s0 = 0.0, s1 = 0.0;
      double p0[2], p1[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int q = kg + 32 * j;
        p0[j] = q <= nP ? P[r + (int64_t)q * ldp] : 0.0;
        p1[j] = q <= nP ? P[r + 1 + (int64_t)q * ldp] : 0.0;
      }
      for (int k0 = c + 1 + kg; k0 < n; k0 += 512) {
        pair8 av[16];
        unsigned long long ub[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int k = min(k0 + 32 * j, n - 1);
          ub[j] = k == c + 1 ? 0ull : grid_peek(uv + k);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j)
          av[j] = *reinterpret_cast<const pair8*>(A + r + (int64_t)min(k0 + 32 * j, n - 1) * lda);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int k = k0 + 32 * j;
          if (k < n) {
            const double u = k == c + 1 ? 1.0 : grid_take(uv + k, ub[j], ok) * gr.scale;
            s0 += av[j].x * u;
            s1 += av[j].y * u;
          }
        }
      }
      if (r0 == max(rlo, c + 1)) {
        if (t <= nP) {
          const double qc = grid_take(xqc + t, qcb, ok);
          L.qc[t] = qc;
          L.pv[t] = qc + gr.scale * qtu;  // Q^T u
        }
        if (t == 0) L.qc[nP + 1] = 1.0;  // u's pivot
        __syncthreads();
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int q = kg + 32 * j;
        if (q <= nP) {
          s0 -= p0[j] * L.pv[q];
          s1 -= p1[j] * L.pv[q];
        }
      }
#pragma unroll
      for (int off = 8; off < 64; off *= 2) {
        s0 += __shfl_xor(s0, off, 64);
        s1 += __shfl_xor(s1, off, 64);
      }
      if (ln < 8) {
        L.red[wv * 16 + 2 * rp] = s0;
        L.red[wv * 16 + 2 * rp + 1] = s1;
      }
      __syncthreads();
      if (t < 16 && r0 + t < rhi) {
        // where the pair was clamped, its second row is the last one
        const int at = r0 + t == m - 1 && (t & 1) == 0 ? t + 1 : t;
        const double x = (L.red[at] + L.red[16 + at]) + (L.red[32 + at] + L.red[48 + at]);
        P[r0 + t + (int64_t)(nP + 1) * ldp] = gr.tau * x;
      }
      __syncthreads();
    }
  }
}

__global__ __launch_bounds__(256) void k_brd_clear(double* __restrict__ places, int64_t count) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256)
    grid_clear(places + e);
}

}  // namespace

int launch_gebrd(int device, int m, int n, double* A, int lda, double* tauq, double* taup, double* d, double* e,
                 int b, void* work, size_t work_bytes, int max_wg, hipStream_t st) {
  int cus = 0, per = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return BDC_ERR_HIP;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void*>(k_brd_panel), 256, 0) !=
      hipSuccess)
    return BDC_ERR_HIP;
  const int maxg = std::min(std::min(max_wg, kGridMaxWg), std::max(1, cus * std::max(per, 1)));
  if (gebrd_work_bytes(m, n, b, maxg) > work_bytes) return BDC_ERR_TOO_LARGE;
  double* P = reinterpret_cast<double*>(work);
  double* Qt = P + (size_t)m * 2 * b;
  double* places = Qt + (size_t)2 * b * n;
  const int ldq = 2 * b;
  for (int j0 = 0; j0 < n; j0 += b) {
    const int bw = std::min(b, n - j0);
    // at least 16 rows per workgroup: 4096 x 4096 takes 195 ms with 32, 146 with
    // 16 and 205 with 8 (whose passes load half of their 16 columns for
    // nothing), 2000 x 2000 67, 47 and 51
    const int G = std::max(1, std::min(maxg, (m - j0 + 15) / 16));
    int rpw = (m - j0 + G - 1) / G, cpw = (n - j0 + G - 1) / G;
    int64_t lda64 = lda, ldp64 = m;
    int ldq_ = ldq;
    BrdX X;
    X.slots = places;
    X.totals = X.slots + (size_t)kGridSets * kSlot * G;
    X.pc = X.totals + kGridSets * kSlot;
    X.qc = X.pc + kGridSets * 2 * kBrdMaxB;
    X.x = X.qc + kGridSets * 2 * kBrdMaxB;
    X.u = X.x + (size_t)kGridSets * m;
    const int64_t count = (int64_t)gebrd_places(m, n, G);
    hipLaunchKernelGGL(k_brd_clear, dim3((unsigned)std::min<int64_t>((count + 255) / 256, 1024)), dim3(256), 0, st,
                       places, count);
    void* args[] = {&A, &lda64, &m, &n, &j0, const_cast<int*>(&bw), &P, &ldp64, &Qt, &ldq_, &tauq, &taup, &d, &e,
                    &X, &rpw, &cpw};
    if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_brd_panel), dim3(G), dim3(256), args, 0, st) !=
        hipSuccess)
      return BDC_ERR_HIP;
    // trailing matrix: A <- A - P Q^T over rows and columns past the panel
    const int r0 = j0 + bw;
    if (r0 < n)
      launch_sub_product(m - r0, n - r0, 2 * bw, P + r0, m, Qt + (int64_t)r0 * ldq, ldq,
                         A + r0 + (int64_t)r0 * lda, lda, st);
  }
  return BDC_OK;
}

}  // namespace bdc
