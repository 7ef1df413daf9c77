// Householder QR of a tall matrix and the explicit Q (Section 4.3.1-4.3.2,
// the tall-and-skinny path): blocked Householder QR in LAPACK's geqrf storage
// with the panel factored on the GPU and the trailing matrix updated in the
// modified compact WY form (eq. larfb with T^{-1} = Y^T Y of eq.
// larft_update), and Q = prod_k (I - Y_k T_k Y_k^T) I (eq. orgqr-q) with
// T^{-1} recomputed at its own block size.
//
// Panel (b <= 64 columns, rows j0..m-1): one cooperative grid of G
// workgroups.  Every workgroup keeps the panel's top b x b block (the rows of
// its pivots) in LDS and updates it redundantly, and owns a contiguous slice
// of the rows below it, also in LDS.  The columns go in steps of up to 8,
// because a grid all-reduce costs about 10 us whatever it carries:
//   1. one all-reduce per step: M = X_s^T [X_s X_later] over the owned rows of
//      all workgroups (per-workgroup partial sums added by every workgroup in
//      the same order: deterministic);
//   2. the step's reflectors from M and the top block alone (Section 4.1):
//      alpha = the pivot entry, sigma = ||x below the pivot||^2, beta =
//      -sign(alpha) sqrt(alpha^2 + sigma), y = x / (alpha - beta) below the
//      pivot, 1 at it, tau = 2 / y^T y with y^T y = 1 + sigma / (alpha -
//      beta)^2 (tau = 0, the identity, when sigma = 0); w = tau y^T X; then
//      M of the columns after it follows from x <- x - y w as <x_i, x_k> -
//      w_i <y, x_k> - w_k <y, x_i> + w_i w_k <y, y>.  A column whose sum of
//      squares has cancelled by more than a bit so far ends the step before
//      it: the next step's all-reduce forms it anew.  (The sum's error goes
//      into tau and R as it is.  Chebyshev polynomials on 700 points, 200
//      columns: factorisation error 0.9e-15 so and 1e-14 to 3e-14 with 3 bits,
//      1.0e-15 with an all-reduce per column.  Columns of random entries
//      do not cancel, so their steps stay 8 columns long);
//   3. the step's reflectors applied to the owned rows: each row's entries of
//      the step's columns one reflector after the other, then the later
//      columns together.
// Panels of 32 columns of 20000 rows: 525 us with an all-reduce and three
// passes over LDS per column, 114 us so (four all-reduces).
// Every wait of the all-reduce is bounded (the kernel ends after an expired one),
// and the launch is cooperative, so all workgroups are resident.
#include <algorithm>

#include "bdc_internal.h"
#include "backtr.h"
#include "block_util.h"
#include "qr.h"
#include "grid_sync.h"

namespace bdc {
namespace {

constexpr int kQrMaxB = 64;         // panel width, at most
constexpr int kQrBlock = 1024;      // threads of a panel workgroup (16 wavefronts)
constexpr int kQrWaves = kQrBlock / 64;
constexpr int kQrXCap = 160 * kQrMaxB;  // entries of the owned rows: 10240 / b rows
constexpr int kQrStep = 8;          // columns per all-reduce, at most
constexpr int kQrSums = 256;        // sums per all-reduce, at most
constexpr double kQrKeep = 0.5;     // a column of a step keeps this share of its sum of squares
// row stride of the owned rows: odd from 16 columns on, so that a wavefront
// with a row per lane spreads over the LDS banks
__device__ __host__ constexpr int qr_stride(int b) { return b >= 16 ? (b | 1) : b; }
struct PanelLds {
  double X[kQrXCap + kQrXCap / 16];  // owned rows, X[r * stride + k]
  double T[kQrMaxB * (kQrMaxB + 1)];  // top block, T[i * (b + 1) + k] = A(j0 + i, j0 + k)
  double red[kQrWaves * kQrSums];
  double M[kQrSums];                 // M[i * nk + k] = <x_{c+i}, x_{c+k}>
  double W[kQrStep * kQrMaxB];       // W[i * 64 + k]: w of reflector i, column k of the panel
  double P[kQrMaxB];                 // the top block's part of M's row i
  double big[kQrStep];               // sum of the terms' sizes in M[i][i]
  unsigned bad;                      // a wait of an all-reduce has expired
};

// grid: G workgroups (cooperative), kQrBlock threads.  slots: kGridSets x
// kQrSums x G places; totals: two regions of kGridSets x kQrSums, this launch's
// (`region`) all empty, the other, which the last launch used and did not
// clear, emptied here for the next one.
__global__ __launch_bounds__(kQrBlock, 1) void k_qr_panel(double* __restrict__ A, int64_t lda, int m, int j0, int b,
                                                     int rows_per_wg, double* __restrict__ tau,
                                                     double* __restrict__ slots, double* __restrict__ totals,
                                                     int region) {
  __shared__ PanelLds L;
  const int t = threadIdx.x, G = gridDim.x, g = blockIdx.x;
  const int ln = t & 63, wv = t >> 6;
  const int top = min(b, m - j0);                  // rows of the top block
  const int below0 = j0 + top;                     // first row below it
  const int r0 = below0 + g * rows_per_wg;         // owned rows [r0, r1)
  const int r1 = min(m, r0 + rows_per_wg);
  const int R = max(0, r1 - r0);
  const int XS = qr_stride(b), TS = b + 1;
  double* Ap = A + j0 + (int64_t)j0 * lda;         // panel origin
  for (int e = t; e < top * b; e += kQrBlock) {
    const int i = e % top, k = e / top;
    L.T[i * TS + k] = Ap[i + (int64_t)k * lda];
  }
  for (int e = t; e < R * b; e += kQrBlock) {
    const int r = e % R, k = e / R;
    L.X[r * XS + k] = A[(r0 + r) + (int64_t)(j0 + k) * lda];
  }
  if (g == 0)
    for (int e = t; e < kGridSets * kQrSums; e += kQrBlock) grid_clear(totals + (region ^ 1) * kGridSets * kQrSums + e);
  totals += region * kGridSets * kQrSums;
  if (t == 0) L.bad = 0;
  __syncthreads();
  int set = 0, last = 0;    // the next all-reduce's set; sums of the last one
  double* prev = nullptr;   // its totals
  for (int c = 0; c < b;) {
    if (c >= top) {  // no pivot row left: identities
      if (g == 0 && t < b - c) tau[j0 + c + t] = 0.0;
      break;
    }
    const int nk = b - c;
    const int s = min(min(kQrStep, top - c), kQrSums / nk);
    // M's partial sums over the owned rows: lane -> column (two rows at a
    // time where the columns leave half of the lanes), wavefronts over the rows
    {
      double acc[kQrStep] = {};
      const bool two = nk <= 32;
      const int k = two ? ln & 31 : ln, h = two ? ln >> 5 : 0;
      if (k < nk) {
        for (int r = two ? 2 * wv + h : wv; r < R; r += two ? 2 * kQrWaves : kQrWaves) {
          const double* x = L.X + r * XS + c;
          const double xk = x[k];
#pragma unroll
          for (int i = 0; i < kQrStep; ++i)
            if (i < s) acc[i] = fma(x[i], xk, acc[i]);
        }
      }
      double* part = L.red + wv * kQrSums + k;
      if (h == 0 && k < nk)
#pragma unroll
        for (int i = 0; i < kQrStep; ++i)
          if (i < s) part[i * nk] = acc[i];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (h == 1 && k < nk)
#pragma unroll
        for (int i = 0; i < kQrStep; ++i)
          if (i < s) part[i * nk] += acc[i];
    }
    __syncthreads();
    if (t < s * nk) {
      double v = 0.0;
#pragma unroll
      for (int u = 0; u < kQrWaves; ++u) v += L.red[u * kQrSums + t];
      L.M[t] = v;
    }
    grid_settle();
    __syncthreads();
    double* tot = totals + set * kQrSums;
    if (!grid_sum<kQrBlock>(slots + (size_t)set * kQrSums * G, tot, prev, last, s * nk, L.M, &L.bad)) return;
    prev = tot;
    last = s * nk;
    set = set == kGridSets - 1 ? 0 : set + 1;
    if (t < s) L.big[t] = L.M[t * nk + t];
    // the step's reflectors
    double sc[kQrStep];
    int done = 0;
#pragma unroll
    for (int i = 0; i < kQrStep; ++i) {
      sc[i] = 0.0;
      if (i > done || i >= s) continue;  // the step has ended
      const int j = c + i;
      // the top block's part of row i of M (rows below the pivot), and the
      // last pivot's column scaled now that nobody reads it unscaled
      for (int k = j + wv; k < b; k += kQrWaves) {
        const double v = ln > j && ln < top ? L.T[ln * TS + j] * L.T[ln * TS + k] : 0.0;
        const double p = wave_sum_last(v);
        if (ln == 63) L.P[k] = p;
      }
      if (i > 0 && t >= j && t < top) L.T[t * TS + j - 1] *= sc[i > 0 ? i - 1 : 0];
      __syncthreads();
      const double own = L.M[i * nk + i], big = L.big[i];
      if (i > 0 && !(own > kQrKeep * big) && big != 0.0) continue;  // cancelled: a decision every workgroup takes alike
      done = i + 1;
      const double sigma = own + L.P[j], alpha = L.T[j * TS + j];
      double beta = alpha, tc = 0.0;
      if (sigma > 0.0) {
        const double nrm = sqrt(alpha * alpha + sigma);
        beta = -copysign(nrm, alpha);
        const double den = alpha - beta;
        sc[i] = 1.0 / den;
        tc = 2.0 / (1.0 + sigma / (den * den));
      }
      if (t > i && t < nk)
        L.W[i * kQrMaxB + c + t] = tc * (sc[i] * (L.M[i * nk + t] + L.P[c + t]) + L.T[j * TS + c + t]);
      __syncthreads();
      // the top block, and M of the step's later columns, after this reflector
      for (int e = t; e < (top - j) * (nk - i - 1); e += kQrBlock) {
        const int q = e / (nk - i - 1), r = j + q, k = j + 1 + e - q * (nk - i - 1);
        const double y = q == 0 ? 1.0 : L.T[r * TS + j] * sc[i];
        L.T[r * TS + k] -= y * L.W[i * kQrMaxB + k];
      }
      const int left = s - i - 1;
      for (int e = t; e < left * nk; e += kQrBlock) {
        const int u = i + 1 + e / nk, k = e - (e / nk) * nk;
        if (k < u) continue;
        const double wu = L.W[i * kQrMaxB + c + u], wk = L.W[i * kQrMaxB + c + k];
        const double yu = sc[i] * L.M[i * nk + u], yk = sc[i] * L.M[i * nk + k], yy = sc[i] * (sc[i] * own);
        L.M[u * nk + k] = L.M[u * nk + k] - wu * yk - wk * yu + wu * wk * yy;
        if (k == u) L.big[u] += wu * wu * yy;
      }
      // the pivot entry becomes R's diagonal (row j's other entries are above)
      if (t == 0) {
        L.T[j * TS + j] = beta;
        if (g == 0) tau[j0 + j] = tc;
      }
      __syncthreads();
    }
    // the last reflector's column of the top block (a column that ended the
    // step early has scaled it already)
#pragma unroll
    for (int i = 0; i < kQrStep; ++i)
      if (done == s && i == s - 1 && t > c + i && t < top) L.T[t * TS + c + i] *= sc[i];
    // owned rows: the step's columns, a row per thread
    for (int r = t; r < R; r += kQrBlock) {
      double* xr = L.X + r * XS + c;
      double x[kQrStep];
#pragma unroll
      for (int i = 0; i < kQrStep; ++i) x[i] = i < done ? xr[i] : 0.0;
#pragma unroll
      for (int i = 0; i < kQrStep; ++i) {
        if (i >= done) break;
        x[i] *= sc[i];
#pragma unroll
        for (int u = i + 1; u < kQrStep; ++u)
          if (u < done) x[u] -= x[i] * L.W[i * kQrMaxB + c + u];
        xr[i] = x[i];
      }
    }
    __syncthreads();
    // and the later ones
    {
      const int nl = nk - done;
      const bool two = nl <= 32;
      const int k = two ? ln & 31 : ln, h = two ? ln >> 5 : 0;
      if (k < nl) {
        double wk[kQrStep];
#pragma unroll
        for (int i = 0; i < kQrStep; ++i) wk[i] = i < done ? L.W[i * kQrMaxB + c + done + k] : 0.0;
        for (int r = two ? 2 * wv + h : wv; r < R; r += two ? 2 * kQrWaves : kQrWaves) {
          double* x = L.X + r * XS + c;
          double v = x[done + k];
#pragma unroll
          for (int i = 0; i < kQrStep; ++i)
            if (i < done) v -= x[i] * wk[i];
          x[done + k] = v;
        }
      }
    }
    __syncthreads();
    c += done;
  }
  // write back: owned rows, and the top block from workgroup 0
  for (int e = t; e < R * b; e += kQrBlock) {
    const int r = e % R, k = e / R;
    A[(r0 + r) + (int64_t)(j0 + k) * lda] = L.X[r * XS + k];
  }
  if (g == 0)
    for (int e = t; e < top * b; e += kQrBlock) {
      const int i = e % top, k = e / top;
      Ap[i + (int64_t)k * lda] = L.T[i * TS + k];
    }
}

__global__ __launch_bounds__(256) void k_qr_clear(double* __restrict__ places, int64_t count) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256)
    grid_clear(places + e);
}

// Q (m x ncols, ldq) = the identity's first ncols columns
__global__ __launch_bounds__(256) void k_qr_eye(double* __restrict__ Q, int64_t ldq, int m, int ncols) {
  const int64_t total = (int64_t)m * ncols;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int c = (int)(e / m), r = (int)(e - (int64_t)c * m);
    Q[r + (int64_t)c * ldq] = r == c ? 1.0 : 0.0;
  }
}

}  // namespace

// places: kGridSets sets of slots, then two regions of totals
static size_t qr_places(int wgs) { return (size_t)kGridSets * kQrSums * (wgs + 2); }

size_t qr_sync_bytes(int max_wg) {
  return qr_places(std::min(max_wg, kGridMaxWg)) * sizeof(double);
}

int qr_max_block() { return kQrMaxB; }

int qr_panel_grid(int device, int rows_below, int b, int* grid, int* rows_per_wg) {
  int cus = 0, per = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return -1;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void*>(k_qr_panel), kQrBlock, 0) !=
      hipSuccess)
    return -1;
  const int maxg = std::max(1, std::min(kGridMaxWg, cus * std::max(per, 1)));
  // as few workgroups as the LDS allows: a grid all-reduce costs more with
  // more workgroups, and a workgroup's 16 wavefronts share its rows' work
  const int cap = kQrXCap / std::max(b, 1);
  int G = std::max(1, (rows_below + cap - 1) / cap);
  if (G > maxg) return 1;  // too many rows for the resident grid
  *grid = G;
  *rows_per_wg = std::max((rows_below + G - 1) / G, 0);
  return 0;
}

int launch_geqrf(int device, int m, int n, double* A, int lda, double* tau, int b, void* sync_buf, size_t sync_bytes,
                 const BtPlan& plan, void* bt_scratch, hipStream_t st) {
  // totals first, then slots; every slot is empty again when a panel ends,
  // whatever its grid
  double* totals = reinterpret_cast<double*>(sync_buf);
  double* slots = totals + 2 * kGridSets * kQrSums;
  int G0 = 1, R0 = 0, region = 0;
  if (qr_panel_grid(device, std::max(0, m - std::min(b, n)), std::min(b, n), &G0, &R0) != 0) return BDC_ERR_TOO_LARGE;
  if (qr_sync_bytes(G0) > sync_bytes) return BDC_ERR_TOO_LARGE;
  const int64_t places = (int64_t)qr_places(G0);
  hipLaunchKernelGGL(k_qr_clear, dim3((unsigned)((places + 255) / 256)), dim3(256), 0, st, totals, places);
  for (int j0 = 0; j0 < n; j0 += b) {
    const int bw = std::min(b, n - j0);
    const int top = std::min(bw, m - j0);
    const int rows_below = m - j0 - top;
    int G = 1, R = 0;
    if (qr_panel_grid(device, rows_below, bw, &G, &R) != 0) return BDC_ERR_TOO_LARGE;
    if (qr_sync_bytes(G) > sync_bytes) return BDC_ERR_TOO_LARGE;
    int64_t lda64 = lda;
    void* args[] = {&A, &lda64, &m, &j0, const_cast<int*>(&bw), &R, &tau, &slots, &totals, &region};
    if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_qr_panel), dim3(G), dim3(kQrBlock), args, 0, st) !=
        hipSuccess)
      return BDC_ERR_HIP;
    region ^= 1;
    // trailing columns: A_t <- H_{bw-1} ... H_0 A_t = Q_panel^T A_t
    const int nt = n - j0 - bw;
    if (nt > 0)
      launch_backtr(1, m - j0, nt, bw, 0, A + j0 + (int64_t)j0 * lda, 1, lda, tau + j0,
                    A + j0 + (int64_t)(j0 + bw) * lda, lda, plan, bt_scratch, st);
  }
  return BDC_OK;
}

void launch_orgqr(int m, int ncols, int k, const double* A, int lda, const double* tau, double* Q, int ldq,
                  const BtPlan& plan, void* bt_scratch, hipStream_t st) {
  const int64_t total = (int64_t)m * ncols;
  hipLaunchKernelGGL(k_qr_eye, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 65536)), dim3(256), 0, st, Q,
                     (int64_t)ldq, m, ncols);
  // blocks from the last to the first; block j acts on rows and columns from
  // its first pivot j b on (the columns before it are still those of the
  // identity, which its reflectors leave unchanged)
  const int b = plan.group;
  const int nblk = (k + b - 1) / b;
  for (int q = nblk - 1; q >= 0; --q) {
    const int i0 = q * b, bw = std::min(b, k - i0);
    if (i0 >= m || i0 >= ncols) continue;
    launch_backtr(0, m - i0, ncols - i0, bw, 0, A + i0 + (int64_t)i0 * lda, 1, lda, tau + i0,
                  Q + i0 + (int64_t)i0 * ldq, ldq, plan, bt_scratch, st);
  }
}

}  // namespace bdc
