// Leaf solves of the divide-and-conquer tree (Algorithm 2 step (1): the
// bottom subproblems by QR iteration).
//
// One workgroup per leaf of m <= 32 rows and m+s columns: implicit-shift
// Golub-Kahan sweeps with a Wilkinson shift, zero diagonal chasing, the
// accumulated W (m x m) and Q ((m+s) x (m+s)) stored column-major in LDS so
// that a wavefront's lanes (a row each) touch consecutive words.  The leaf is
// first scaled by a power of two so no square can overflow; the values are
// scaled back on output.  Output columns are written sorted by value
// (ascending); each physical column records the leaf's row range as its
// support.
#include "bdc_internal.h"

namespace bdc {
namespace {

constexpr double kEps = 0x1p-52;

// lane k's value of a per-lane double, as a wave-uniform value
__device__ inline double lane_val(double v, int k) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), k);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), k);
  return __hiloint2double(hi, lo);
}

// (c, s, r) with c f + s g = r >= 0 and -s f + c g = 0.  The leaf is scaled
// so that |f|, |g| <= 2; the reciprocal square root (hardware estimate and
// two Newton steps) is used unless f^2 + g^2 is near underflow.
__device__ inline void givens(double f, double g, double& c, double& s, double& r) {
  if (g == 0.0) {
    c = f >= 0.0 ? 1.0 : -1.0;
    s = 0.0;
    r = fabs(f);
    return;
  }
  const double q = fma(f, f, g * g);
  if (q > 0x1p-960) {
    double y = __builtin_amdgcn_rsq(q);
    const double hq = 0.5 * q;
    y = y * fma(-hq * y, y, 1.5);
    y = y * fma(-hq * y, y, 1.5);
    c = f * y;
    s = g * y;
    r = q * y;
  } else {
    r = hypot(f, g);
    c = f / r;
    s = g / r;
  }
}

// The same without its careful branches: what givens() returns
// where g != 0 and f^2 + g^2 > 2^-960.
__device__ inline void givens_fast(double f, double g, double& c, double& s, double& r) {
  const double q = fma(f, f, g * g);
  double y = __builtin_amdgcn_rsq(q);
  const double hq = 0.5 * q;
  y = y * fma(-hq * y, y, 1.5);
  y = y * fma(-hq * y, y, 1.5);
  c = f * y;
  s = g * y;
  r = q * y;
}

// columns (i, j) of an LDS matrix (column stride ld) <- (c a_i + s a_j,
// -s a_i + c a_j), row = lane
__device__ inline void rot_cols(double* A, int ld, int rows, int i, int j, double c, double s, int lane) {
  if (lane < rows) {
    const double ai = A[lane + i * ld];
    const double aj = A[lane + j * ld];
    A[lane + i * ld] = c * ai + s * aj;
    A[lane + j * ld] = -s * ai + c * aj;
  }
}

// lane i's value from lane i + 1 / i - 1 (0 past the ends)
template <int CTRL>
__device__ inline double wave_shift(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double from_above(double v) { return wave_shift<0x130>(v); }  // wave_shl:1
__device__ inline double from_below(double v) { return wave_shift<0x138>(v); }  // wave_shr:1

__device__ inline double wave_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// Two wavefronts per leaf.  Wavefront 0 runs the Givens chain of a sweep and
// leaves its rotations' arguments in LDS; wavefront 1 does the rest: the
// rotations from their arguments (lane k: step k), the tests before a sweep
// (lane i holds d_i and e_i, the superdiagonal entry right of d_i), the shift
// (lane i: were the block to end at i, so that it does not wait for the tests),
// the rare rotations that are no sweep, and, while the next sweep's chain runs,
// the last sweep's rotations of W and Q (lane r: row r of the column-major LDS
// copies; the column being rotated forward stays in a register).
//
// The chain bounds the time: 35 FP64 operations and two reciprocal square
// roots a step, about 1150 steps for a 32-row leaf, on one wavefront.  So it
// holds nothing else: no test (each step's rotations take givens()' usual
// path; a rotation that would not have shows afterwards by s = 0 or a tiny r,
// and wavefront 1 redoes such a sweep step by step), no cross-lane read, no
// update of W or Q, and as few LDS writes as the rotations can be had from
// (25 cycles each).  Measured (leaves of 16..32 rows): the leaves of n = 100
// 132 us, of n = 1000 212 and of n = 16384 247; 155, 237 and 280 with (c, s) and
// the new entries posted and the shift after the tests; 260, 443 and 555 for
// one wavefront doing everything with a test per rotation; 40000 leaves of a
// batch, which fill the chip either way, 4.2, 4.8 and 6.2 ms.  Several leaves
// per chain wavefront (a lane each) measured slower in both regimes (322-369 us
// and 6.2-8 ms): lanes wait for the longest block.
template <int ML>
struct LeafLds {
  static constexpr int kLd = ML + 1;  // column stride (doubles)
  double W[ML * kLd];
  double Q[(ML + 1) * kLd];
  struct Sweep {            // one posted sweep, by parity
    double2 in[ML + 2];     // (d_i, e_i) before it
    double2 yz[ML + 2];     // step k: the arguments of the rotation of Q's columns (k, k+1)
    double2 nd[ML + 2];     // and (x) the first one of W's, whose second is s d_{k+1}
    double2 rq[ML + 2];     // (c, s) of the two rotations
    double2 rw[ML + 2];
    double2 last;           // (d_hi, e_{hi-1}) after it
  } sw[2];
  double2 yz;               // the first rotation's two entries
  int2 block;               // the sweep's block (lo, hi); hi = 0: no more sweeps
};

// one sweep's chain on the entries of `in`: steps lo .. lo + n - 1
template <int ML>
__device__ inline void leaf_chain(typename LeafLds<ML>::Sweep& S, int lo, int n, double y, double z) {
  const double2 v0 = S.in[lo], v1 = S.in[lo + 1];
  double dk = v0.x, ek = v0.y, dk1 = v1.x, ek1 = v1.y;
  typename LeafLds<ML>::Sweep* p = reinterpret_cast<typename LeafLds<ML>::Sweep*>(&S.in[lo]);  // moves with k
#pragma unroll 2
  for (int k = 0; k < n; ++k) {
    const double2 v2 = p->in[2];
    double c, s, r, c2, s2, r2;
    givens_fast(y, z, c, s, r);
    const double ndk = fma(c, dk, s * ek);
    const double bulge = s * dk1;
    const double nek = fma(c, ek, -(s * dk));
    const double ndk1 = c * dk1;
    givens_fast(ndk, bulge, c2, s2, r2);
    p->yz[0] = make_double2(y, z);
    p->nd[0].x = ndk;
    y = fma(nek, c2, ndk1 * s2);      // e_k
    dk = fma(ndk1, c2, -(nek * s2));  // d_{k+1}
    z = s2 * ek1;                     // the bulge right of e_k
    ek = c2 * ek1;                    // e_{k+1} (ek1 = 0 at the block's end)
    dk1 = v2.x;
    ek1 = v2.y;
    p = reinterpret_cast<typename LeafLds<ML>::Sweep*>(reinterpret_cast<double2*>(p) + 1);
  }
  S.last = make_double2(dk, y);
}

// the rotations of one sweep on row `lane` of W and Q
template <int ML>
__device__ inline void leaf_apply(LeafLds<ML>& S, const typename LeafLds<ML>::Sweep& R, int lo, int hi, int lane) {
  constexpr int kLd = LeafLds<ML>::kLd;
  double* q = S.Q + lane;
  double* w = S.W + lane;
  double qk = q[lo * kLd], wk = w[lo * kLd];
  for (int k = lo; k < hi; ++k) {
    const double2 a = R.rq[k], b = R.rw[k];
    const double qk1 = q[(k + 1) * kLd], wk1 = w[(k + 1) * kLd];
    q[k * kLd] = fma(qk, a.x, a.y * qk1);
    qk = fma(qk1, a.x, -(qk * a.y));
    w[k * kLd] = fma(wk, b.x, b.y * wk1);
    wk = fma(wk1, b.x, -(wk * b.y));
  }
  q[hi * kLd] = qk;
  w[hi * kLd] = wk;
}

// The same for leaves of at most 32 columns: lanes 0..31 have Q's rows, lanes
// 32..63 W's, so that a step is half the instructions (a batch's leaves 4.38 ->
// 4.23 ms; hidden behind the chain otherwise).
template <int ML>
__device__ inline void leaf_apply_halves(LeafLds<ML>& S, const typename LeafLds<ML>::Sweep& R, int lo, int hi,
                                         int lane) {
  constexpr int kLd = LeafLds<ML>::kLd;
  double* x = (lane < 32 ? S.Q : S.W) + (lane & 31);
  const double2* rot = lane < 32 ? R.rq : R.rw;
  double xk = x[lo * kLd];
  for (int k = lo; k < hi; ++k) {
    const double2 a = rot[k];
    const double xk1 = x[(k + 1) * kLd];
    x[k * kLd] = fma(xk, a.x, a.y * xk1);
    xk = fma(xk1, a.x, -(xk * a.y));
  }
  x[hi * kLd] = xk;
}

template <int ML>
__global__ __launch_bounds__(128) void k_leaf(const LeafDesc* __restrict__ leaves, Work w) {
  constexpr int kLd = LeafLds<ML>::kLd;
  __shared__ LeafLds<ML> S;
  double* const W = S.W;
  double* const Q = S.Q;
  const int lane = threadIdx.x & 63;

  if (threadIdx.x < 64) {
    for (int par = 0;; par ^= 1) {
      __syncthreads();
      const double2 yz = S.yz;
      const int lo = __builtin_amdgcn_readfirstlane(S.block.x), hi = __builtin_amdgcn_readfirstlane(S.block.y);
      if (hi == 0) return;
      if (lane == 0) leaf_chain<ML>(S.sw[par], lo, hi - lo, yz.x, yz.y);
      __syncthreads();
    }
  }

  const LeafDesc L = leaves[blockIdx.x];
  const int m = L.m, s = L.s, ms = m + s, r0 = L.r0;
  const int64_t ld = L.ld;
  const int64_t pv = L.vec_off;
  unsigned long long nrot_w = 0, nrot_q = 0;  // rotations applied to W and to Q
  const bool row = lane < ms;  // W's row m, which nothing reads, stands in for the row that W has not when s = 1

  for (int i = lane; i < ML * kLd; i += 64) W[i] = 0.0;
  for (int i = lane; i < (ML + 1) * kLd; i += 64) Q[i] = 0.0;
  if (lane < m) W[lane + lane * kLd] = 1.0;
  if (lane < ms) Q[lane + lane * kLd] = 1.0;

  // load and scale by a power of two
  double dv = 0.0, ev = 0.0;
  if (lane < m) dv = w.ctl->io.d[pv + r0 + lane];
  if (lane < m - 1 + s) ev = w.ctl->io.e[pv + r0 + lane];
  // every entry of d and e belongs to exactly one leaf or one merge's middle
  // row, so leaves and merges between them check all of the input
  const bool bad = __any(!(fabs(dv) <= 1.79769313486231570e308) || !(fabs(ev) <= 1.79769313486231570e308));
  if (bad && lane == 0) atomicOr(&w.ctl->nonfinite, 1);
  const double amax = wave_max(fmax(fabs(dv), fabs(ev)));
  double p = 1.0;
  if (amax > 0.0 && amax <= 1.79e308) {
    int ex;
    frexp(amax, &ex);
    p = ldexp(1.0, ex);
  }
  double dreg = dv / p;  // d_lane
  double ereg = ev / p;  // e_lane (lane m-1: the extra column's entry when s = 1)
  const double tiny = kEps * (amax / p);

  // s = 1: remove the extra column's entry, bottom row first.  The right
  // rotation of columns (j, m) zeroes B[j, m] and moves a fill-in to B[j-1, m].
  if (s == 1) {
    double f = lane_val(ereg, m - 1);
    if (lane == m - 1) ereg = 0.0;
    for (int j = m - 1; j >= 0; --j) {
      double c, sn, r;
      givens(lane_val(dreg, j), f, c, sn, r);
      if (lane == j) dreg = r;
      if (j > 0) {
        const double t = lane_val(ereg, j - 1);
        if (lane == j - 1) ereg = c * t;
        f = -sn * t;
      }
      rot_cols(Q, kLd, ms, j, m, c, sn, lane);
      ++nrot_q;
    }
  }

  const int max_steps = w.max_leaf_sweeps * (m > 0 ? m : 1);
  int steps = 0;
  int hi = m - 1, lo = 0;
  double mu = 0.0;
  bool go = false, pending = false;  // a sweep posted for this parity; the last sweep's rotations not applied yet
  int phi = 0, plo = 0;
  double c = 0.0, sn = 0.0, c2 = 0.0, sn2 = 0.0;  // step lane's rotations of the last sweep
  auto apply = [&](int par) {
    typename LeafLds<ML>::Sweep& R = S.sw[par];
    if (lane <= ML) {
      R.rq[lane] = make_double2(c, sn);
      R.rw[lane] = make_double2(c2, sn2);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (ms <= 32) {
      if ((lane & 31) < ms) leaf_apply_halves<ML>(S, R, plo, phi, lane);
    } else if (row) {
      leaf_apply<ML>(S, R, plo, phi, lane);
    }
  };
  for (int par = 0;; par ^= 1) {
    // the posted sweep's outcome, then the tests before the next one
    if (go) {
      const typename LeafLds<ML>::Sweep& R = S.sw[par ^ 1];
      const int at = lane <= ML ? lane : 0;
      const double2 yz = R.yz[at], last = R.last;
      double r, r2;
      givens_fast(yz.x, yz.y, c, sn, r);
      givens_fast(R.nd[at].x, sn * R.in[at + 1].x, c2, sn2, r2);
      // s = 0 where g = 0 (or g / r underflowed); r < 2^-470 well before f^2 + g^2 <= 2^-960
      const bool odd = lane >= lo && lane < hi && (sn == 0.0 || sn2 == 0.0 || !(r2 > 0x1p-470) || !(r > 0x1p-470));
      const double rn = from_above(r);
      if (__any(odd) || bad) {
        // again from the entries as posted, every rotation by givens()
        double dk = lane_val(dreg, lo), ek = lane_val(ereg, lo);
        double y = fma(dk, dk, -mu), z = dk * ek;
        for (int k = lo; k < hi; ++k) {
          const double dk1 = lane_val(dreg, k + 1), ek1 = k < hi - 1 ? lane_val(ereg, k + 1) : 0.0;
          double kc, ks, kr, kc2, ks2, kr2;
          givens(y, z, kc, ks, kr);
          if (k > lo && lane == k - 1) ereg = kr;
          const double ndk = fma(kc, dk, ks * ek);
          const double nek = fma(kc, ek, -(ks * dk));
          const double ndk1 = kc * dk1;
          givens(ndk, ks * dk1, kc2, ks2, kr2);
          if (lane == k) {
            dreg = kr2;
            c = kc;
            sn = ks;
            c2 = kc2;
            sn2 = ks2;
          }
          y = fma(nek, kc2, ndk1 * ks2);
          dk = fma(ndk1, kc2, -(nek * ks2));
          z = ks2 * ek1;
          ek = kc2 * ek1;
        }
        if (lane == hi - 1) ereg = y;
        if (lane == hi) dreg = dk;
      } else {
        if (lane >= lo && lane <= hi) dreg = lane == hi ? last.x : r2;
        if (lane >= lo && lane < hi) ereg = lane == hi - 1 ? last.y : rn;
      }
      nrot_q += hi - lo;
      nrot_w += hi - lo;
      pending = true;
      plo = lo;
      phi = hi;
      go = false;
    }
    double mul = 0.0;
    while (hi > 0) {
      // negligible superdiagonals -> 0; then the unreduced block [lo, hi]
      const double dnext = from_above(dreg);
      if (lane < hi && fabs(ereg) <= kEps * (fabs(dreg) + fabs(dnext))) ereg = 0.0;
      const unsigned long long nz = __ballot(lane < hi && ereg != 0.0);
      {
        // Wilkinson shift were the block to end at this lane: eigenvalue of the
        // trailing 2x2 of B^T B nearer its end (for a block of two, the entry
        // before it is zero)
        const double dm = from_below(dreg), dn = dreg, fm = from_below(ereg);
        const double g = from_below(fm);
        const double t11 = dm * dm + g * g, t12 = dm * fm, t22 = dn * dn + fm * fm;
        const double delta = 0.5 * (t11 - t22);
        const double root = hypot(delta, t12);
        const double denom = delta + (delta >= 0.0 ? root : -root);
        mul = t12 == 0.0 ? t22 : t22 - t12 * t12 / denom;
        asm volatile("" : "+v"(mul));  // here, beside the tests' waits
      }
      hi = nz ? 64 - __builtin_clzll(nz) : 0;
      if (hi == 0) break;
      if (steps >= max_steps) {
        if (lane == 0) atomicAdd(&w.ctl->leaf_capped, 1);
        hi = 0;
        break;
      }
      ++steps;
      const unsigned long long zero_below = ~nz & ((1ull << (hi - 1)) - 1ull);
      lo = zero_below ? 64 - __builtin_clzll(zero_below) : 0;
      const unsigned long long zd = __ballot(lane >= lo && lane <= hi && fabs(dreg) <= tiny);
      if (!zd) {
        go = true;
        break;
      }
      if (pending) apply(par ^ 1);
      pending = false;
      const int i = __builtin_ctzll(zd);
      if (lane == i) dreg = 0.0;
      if (i < hi) {
        // chase B[i, i+1] along row i with left rotations of rows (j, i)
        double f = lane_val(ereg, i);
        if (lane == i) ereg = 0.0;
        for (int j = i + 1; j <= hi; ++j) {
          double kc, ks, kr;
          givens(lane_val(dreg, j), f, kc, ks, kr);
          if (lane == j) dreg = kr;
          if (j < hi) {
            const double t = lane_val(ereg, j);
            f = -ks * t;
            if (lane == j) ereg = kc * t;
          }
          rot_cols(W, kLd, m, j, i, kc, ks, lane);
          ++nrot_w;
        }
      } else {
        // chase B[hi-1, hi] up column hi with right rotations of columns (j, hi)
        double f = lane_val(ereg, hi - 1);
        if (lane == hi - 1) ereg = 0.0;
        for (int j = hi - 1; j >= lo; --j) {
          double kc, ks, kr;
          givens(lane_val(dreg, j), f, kc, ks, kr);
          if (lane == j) dreg = kr;
          if (j > lo) {
            const double t = lane_val(ereg, j - 1);
            f = -ks * t;
            if (lane == j - 1) ereg = kc * t;
          }
          rot_cols(Q, kLd, ms, j, hi, kc, ks, lane);
          ++nrot_q;
        }
      }
    }
    if (go) {
      mu = lane_val(mul, hi);
      if (lane <= ML) S.sw[par].in[lane] = make_double2(dreg, ereg);
      if (lane == lo) S.yz = make_double2(fma(dreg, dreg, -mu), dreg * ereg);
    }
    if (lane == 0) S.block = make_int2(lo, go ? hi : 0);
    __syncthreads();
    if (pending) apply(par ^ 1);
    pending = false;
    if (!go) break;
    __syncthreads();
  }

  // signs, ranks (ascending, ties by index) and output
  double sv = 0.0;
  int rank = 0;
  if (lane < m) {
    sv = fabs(dreg);
    if (dreg < 0.0)
      for (int r = 0; r < m; ++r) W[r + lane * kLd] = -W[r + lane * kLd];
  }
  for (int j = 0; j < m; ++j) {
    const double sj = fabs(lane_val(dreg, j));
    rank += (lane < m && (sj < sv || (sj == sv && j < lane))) ? 1 : 0;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  double* Uw = w.Uw + L.mat_off;
  double* Vw = w.Vw + L.mat_off;
  for (int c = 0; c < m; ++c) {
    const int rc = __shfl(rank, c, 64);
    const int64_t pc = r0 + rc;
    if (lane < m) Uw[(r0 + lane) + pc * ld] = W[lane + c * kLd];
    if (lane < ms) Vw[(r0 + lane) + pc * ld] = Q[lane + c * kLd];
  }
  if (s == 1 && lane < ms) Vw[(r0 + lane) + (int64_t)(r0 + m) * ld] = Q[lane + m * kLd];
  if (lane < m) {
    w.sig[pv + r0 + rank] = sv * p;
    w.col[pv + r0 + lane] = r0 + lane;
    w.ulo[pv + r0 + lane] = r0;
    w.uhi[pv + r0 + lane] = r0 + m;
    w.vlo[pv + r0 + lane] = r0;
    w.vhi[pv + r0 + lane] = r0 + ms;
  }
  if (s == 1 && lane == 0) {
    w.vlo[pv + r0 + m] = r0;
    w.vhi[pv + r0 + m] = r0 + ms;
  }
  // 6 flops per row per rotation
  if (lane == 0) w.leaf_fl[blockIdx.x] = 6ull * (nrot_w * (unsigned long long)m + nrot_q * (unsigned long long)ms);
}

__global__ __launch_bounds__(256) void k_reset(Ctl* ctl, NodeState* st, SecCount* sec, int nnodes, Io io) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->nonfinite = 0;
    ctl->leaf_capped = 0;
    ctl->io = io;
  }
  for (int i = blockIdx.x * 256 + threadIdx.x; i < nnodes; i += gridDim.x * 256) {
    st[i].zmax_bits = 0ull;
    sec[i].evals = 0ull;
    sec[i].terms = 0ull;
    sec[i].capped = 0ull;
  }
}

}  // namespace

void launch_reset(Ctl* ctl, NodeState* nst, SecCount* sec, int nnodes, const Io& io, hipStream_t st) {
  int blocks = (nnodes + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 64) blocks = 64;
  hipLaunchKernelGGL(k_reset, dim3(blocks), dim3(256), 0, st, ctl, nst, sec, nnodes, io);
}

void launch_leaf(const LeafDesc* leaves, int nleaves, int max_m, const Work& w, hipStream_t st) {
  if (nleaves <= 0) return;
  if (max_m <= 8) hipLaunchKernelGGL(k_leaf<8>, dim3(nleaves), dim3(128), 0, st, leaves, w);
  else if (max_m <= 16) hipLaunchKernelGGL(k_leaf<16>, dim3(nleaves), dim3(128), 0, st, leaves, w);
  else if (max_m <= 24) hipLaunchKernelGGL(k_leaf<24>, dim3(nleaves), dim3(128), 0, st, leaves, w);
  else hipLaunchKernelGGL(k_leaf<kMaxLeaf>, dim3(nleaves), dim3(128), 0, st, leaves, w);
}

}  // namespace bdc
