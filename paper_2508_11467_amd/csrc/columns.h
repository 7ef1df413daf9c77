// The columns of a merge before its update products: the rotations of the
// deflated pairs and the gather of the kept columns, as bodies that the
// stand-alone kernels (k_update.hip) and the secular launch (k_secular.hip)
// share.
#pragma once

#include "bdc_internal.h"

namespace bdc {

// A product of the top rows [0, k) reads the kept columns of update positions
// g < n1 + 1 + n2, one of the bottom rows those of g >= n1: of a left-only
// column (g < n1) only the top rows are gathered, of a right-only one (g >=
// n1 + 1 + n2) only the bottom ones, half of what the merge would move with
// whole columns where few columns are shared.
__device__ inline bool column_has_row(const NodeState& st, int g, int row, int k) {
  return row < k ? g < st.n1 + 1 + st.n2 : g >= st.n1;
}

// Rotations, a thread per row; workgroup y of ny of the merge.  kGather: the
// rotated kept columns' rows go to the gathered columns as well (gather_node
// then leaves them out, and neither body reads what the other writes, so the
// two run in one launch).
template <bool kGather>
__device__ inline void rotate_node(const NodeDesc& nd, const Work& w, int y, int ny) {
  const NodeState st = w.st[nd.id];
  const int nrot = st.nrot;
  if (nrot == 0) return;
  const int m = nd.m, s = nd.s, r0 = nd.r0;
  const int64_t ld = nd.ld, pv = nd.vec_off, vo = nd.vec_off + nd.r0;
  const int64_t rb = 2 * vo;
  double* U = w.Uw + nd.mat_off;
  double* V = w.Vw + nd.mat_off;
  for (int base = y * 256; base < m + s; base += ny * 256) {
    const int row = base + threadIdx.x;
    const int gr = r0 + row;
    const bool inV = row < m + s, inU = row < m;
    if (inV) {
      // zero-fill the touched columns outside their current support
      for (int q = 0; q < nrot; ++q) {
        const bool both = w.rot_pos[rb + 2 * q] != 0;
        for (int h = 0; h < 2; ++h) {
          const int pc = w.rot_col[rb + 2 * q + h];
          if (both && inU && (gr < w.ulo[pv + pc] || gr >= w.uhi[pv + pc])) U[gr + pc * ld] = 0.0;
          if (gr < w.vlo[pv + pc] || gr >= w.vhi[pv + pc]) V[gr + pc * ld] = 0.0;
        }
      }
      for (int q = 0; q < nrot; ++q) {
        const bool both = w.rot_pos[rb + 2 * q] != 0;
        const int pp = w.rot_col[rb + 2 * q], pj = w.rot_col[rb + 2 * q + 1];
        const double c = w.rot_cs[rb + 2 * q], sn = w.rot_cs[rb + 2 * q + 1];
        if (both && inU) {
          const double a = U[gr + pp * ld], b = U[gr + pj * ld];
          U[gr + pp * ld] = c * a + sn * b;
          U[gr + pj * ld] = -sn * a + c * b;
        }
        const double a = V[gr + pp * ld], b = V[gr + pj * ld];
        V[gr + pp * ld] = c * a + sn * b;
        V[gr + pj * ld] = -sn * a + c * b;
      }
    }
    if constexpr (kGather) {
      // the kept columns among them, found 4 x 64 positions at a time (all
      // lanes together; every lane then copies its own row)
      double* GU = w.ctl->io.U + nd.mat_off;
      double* GV = w.ctl->io.VT + nd.mat_off;
      const int lane = threadIdx.x & 63;
      for (int g0 = 0; g0 < st.N; g0 += 256) {
        int rf[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int g = g0 + 64 * u + lane;
          const int i = g < st.N ? w.gsurv[vo + g] : -1;
          rf[u] = i > 0 ? w.srot[vo + i] : (i == 0 && st.nzero_d > 0 ? kRotV : 0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          for (unsigned long long left = __ballot(rf[u] != 0); left; left &= left - 1) {
            const int b = __builtin_ctzll(left), g = g0 + 64 * u + b;
            const int f = __builtin_amdgcn_readlane(rf[u], b);
            const int i = w.gsurv[vo + g];
            const int64_t pc = i == 0 ? r0 + nd.k - 1 : w.scol[vo + i];
            if (!inV || !column_has_row(st, g, row, nd.k)) continue;
            if ((f & kRotU) && inU) GU[gr + (int64_t)(r0 + g) * ld] = U[gr + pc * ld];
            if (f & kRotV) GV[gr + (int64_t)(r0 + g) * ld] = V[gr + pc * ld];
          }
      }
    }
  }
}

// The rows of the node's kept columns that the products read, in update
// order, both sides.  A wavefront takes four consecutive columns and 256 rows
// of them: lane c looks up column c's place, support and flags once (the
// lookups are a chain of three dependent loads), then the lanes run along the
// rows, two columns' loads in flight before their stores.  (A thread per
// element, each with its own lookups and divisions: 2.7 ms for the 2000-problem
// batch's gathers, bound by the lookups; beside the secular solves the gathers
// add 2.1 ms that way and 1.7 this way.)  U rows run to m, V rows to m + s.  kSkipRotated: columns that a rotation of this launch writes
// are left to rotate_node.
constexpr int kGatherCols = 4, kGatherRows = 256;

template <bool kSkipRotated>
__device__ inline void gather_node(const NodeDesc& nd, const Work& w, int y, int ny) {
  const NodeState st = w.st[nd.id];
  const int m = nd.m, s = nd.s, r0 = nd.r0, k = nd.k, R = nd.m + nd.s, N = st.N;
  const int64_t ld = nd.ld, pv = nd.vec_off, vo = nd.vec_off + nd.r0;
  const double* U = w.Uw + nd.mat_off + r0;
  const double* V = w.Vw + nd.mat_off + r0;
  double* GU = w.ctl->io.U + nd.mat_off + r0 + (int64_t)r0 * ld;
  double* GV = w.ctl->io.VT + nd.mat_off + r0 + (int64_t)r0 * ld;
  const int lane = threadIdx.x & 63;
  const int chunks = (R + kGatherRows - 1) / kGatherRows;
  const int units = (N + kGatherCols - 1) / kGatherCols * chunks;
  for (int u = y * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); u < units; u += ny * 4) {
    const int g0 = u / chunks * kGatherCols, row0 = u % chunks * kGatherRows;
    // column g0 + (lane % 4): its place (-1: the unit vector e_{k-1}) and the
    // rows to read and to write (relative to the node), none where left out
    const int g = min(g0 + (lane & (kGatherCols - 1)), N - 1);
    const int i = w.gsurv[vo + g];
    const int ra = g < st.n1 + 1 + st.n2 ? 0 : k;
    const int rb = g != g0 + (lane & (kGatherCols - 1)) ? ra : (g < st.n1 ? k : R);  // past the last column: none
    int pcu, pcv, ul, uh, vl, vh, rau = ra, rbu = min(rb, m), rav = ra, rbv = rb;
    if (i == 0) {
      // d = 0 position: left vector e_{k-1} (the middle row), right vector x1
      pcu = -1;
      pcv = r0 + k - 1;
      ul = uh = 0;
      vl = 0;
      vh = R;
      if (kSkipRotated && st.nzero_d > 0) rbv = rav;
    } else {
      const int pc = w.scol[vo + i], rf = w.srot[vo + i];
      const bool fu = (rf & kRotU) != 0, fv = (rf & kRotV) != 0;
      pcu = pcv = pc;
      ul = fu ? 0 : w.ulo[pv + pc] - r0;
      uh = fu ? m : w.uhi[pv + pc] - r0;
      vl = fv ? 0 : w.vlo[pv + pc] - r0;
      vh = fv ? R : w.vhi[pv + pc] - r0;
      if (kSkipRotated && fu) rbu = rau;
      if (kSkipRotated && fv) rbv = rav;
    }
    auto at = [](int v, int c) { return __builtin_amdgcn_readlane(v, c); };
#pragma unroll
    for (int c0 = 0; c0 < kGatherCols; c0 += 2) {
      double x[2][2][4];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int cu = at(pcu, c0 + c), cv = at(pcv, c0 + c);
        const int a = max(at(rau, c0 + c), at(ul, c0 + c)), b = min(at(rbu, c0 + c), at(uh, c0 + c));
        const int d = max(at(rav, c0 + c), at(vl, c0 + c)), e = min(at(rbv, c0 + c), at(vh, c0 + c));
        const double* pu = U + (int64_t)cu * ld;
        const double* pw = V + (int64_t)cv * ld;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = row0 + 64 * q + lane;
          x[c][0][q] = (cu < 0 && row == k - 1) ? 1.0 : 0.0;
          x[c][1][q] = 0.0;
          if (row >= a && row < b) x[c][0][q] = pu[row];
          if (row >= d && row < e) x[c][1][q] = pw[row];
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int a = at(rau, c0 + c), b = at(rbu, c0 + c), d = at(rav, c0 + c), e = at(rbv, c0 + c);
        double* qu = GU + (int64_t)(g0 + c0 + c) * ld;
        double* qv = GV + (int64_t)(g0 + c0 + c) * ld;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = row0 + 64 * q + lane;
          if (row >= a && row < b) qu[row] = x[c][0][q];
          if (row >= d && row < e) qv[row] = x[c][1][q];
        }
      }
    }
  }
}

// workgroups per merge that the two bodies can use
inline int rotate_units(int max_m) { return (max_m + 1 + 255) / 256; }
inline int64_t gather_units(int max_m) {
  return (int64_t)((max_m + 4 * kGatherCols - 1) / (4 * kGatherCols)) * ((max_m + kGatherRows) / kGatherRows);
}

}  // namespace bdc
