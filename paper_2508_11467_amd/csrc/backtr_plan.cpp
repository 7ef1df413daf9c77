// Scratch and depth slices of the back-transformation (k_backtr.hip).  Host code
// only (no HIP calls), so it also builds and runs in the host checks.
#include <algorithm>

#include "backtr.h"

namespace bdc {
namespace {

constexpr int kBtSlices = 64;           // slices of W, at most (unless kBtSliceRows asks for more),
constexpr size_t kBtSliceDoubles = size_t(32) << 20;  // and what they hold together (likewise)
// the fixed scratch: slices of W of a chunk and what they may hold
constexpr int kBtChunkSlices = 16;
constexpr size_t kBtChunkDoubles = size_t(1) << 19;

}  // namespace

// Depth slice of W = Y^T C for `rows` rows, p columns and groups of K: the
// multiple of 128 (up to 4096 rows) that costs least by a plain count of the
// tiles per CU (two at a time on 256 CUs, 2 cycles per row of a 128-column tile
// and row of depth; Y^T Y's share beside them) and the partial sums' traffic
// (written and read, 2000 bytes a cycle).  A function of rows, p and K only,
// so every panel width and chunk adds in the same order.
int bt_slice(int rows, int p, int K) {
  const int tm = bt_tile_rows(K);
  const int64_t tr = (K + tm - 1) / tm, tiles = tr * ((p + 127) / 128), own = tr * ((K + 127) / 128);
  int best = kBtSliceRows;
  double cost = 1e300;
  for (int n = (rows + kBtSliceRows - 1) / kBtSliceRows; n <= kBtSlices; ++n) {
    const int s = ((rows + n - 1) / n + 127) / 128 * 128;
    if (s > kBtSliceRows) continue;
    const int64_t z = (rows + s - 1) / s;
    if (cost < 1e300 && (size_t)z * K * p > kBtSliceDoubles) break;
    const int64_t wg = tiles * z + (own * rows + s - 1) / s, rest = wg % 512;
    const double units = 2.0 * (wg / 512) + (rest == 0 ? 0.0 : rest <= 256 ? 1.0 : 2.0);
    const double c = units * std::min(s, rows) * 2.0 * tm + (double)z * K * p * 16.0 / 2000.0;
    if (c < cost) {
      cost = c;
      best = s;
    }
  }
  return best;
}

size_t backtr_limit_bytes(int m, int panel, int block) {
  const size_t w = (size_t)block * std::max(panel, block);
  return 8 * ((size_t)m * block + (size_t)block * block + w + 32 * w) + 4 * 256;
}

// Scratch: the packed reflectors of a chunk, the slices of W and of Y^T Y,
// their sums over earlier chunks, T^{-1}, its inverted diagonal blocks and Z.
// With group = block and fixed it is never more than backtr_limit_bytes.  W's
// part holds whatever slices bt_slice gives any group of the call, also a last
// one of fewer reflectors: never more than `most`, and more than `whole` only
// while they take no more than kBtSliceDoubles.
BtPlan backtr_plan(int m, int p, int panel, int group, bool fixed) {
  BtPlan b{};
  b.panel = std::max(1, std::min(panel, p));
  b.group = group;
  b.fixed = fixed;
  const size_t K = (size_t)std::min(group, m), w = (size_t)b.panel, rows = (size_t)m;
  const size_t nb = (K + kTB - 1) / kTB, db = std::min<size_t>(K, kTB);
  const size_t most = std::min<size_t>(kBtSlices, (rows + 127) / 128), whole = (rows + kBtSliceRows - 1) / kBtSliceRows;
  b.slices = fixed ? (int)std::max<size_t>(1, std::min<size_t>(kBtChunkSlices, kBtChunkDoubles / (K * w))) : 0;
  size_t off = 0;
  auto take = [&](size_t doubles) {
    const size_t r = off;
    off += doubles;
    return r;
  };
  b.yp = take((fixed ? std::min<size_t>(rows, kBtChunk) : rows) * K);
  b.p = take(fixed ? std::min<size_t>(b.slices, most) * K * w
                   : std::max(std::min(most * K * p, kBtSliceDoubles), whole * K * p));
  b.pt = take(K * K * (((fixed ? std::min<size_t>(rows, kBtChunkT) : rows) + kTSlice - 1) / kTSlice));
  b.wsum = take(fixed ? K * w : 0);
  b.tsum = take(fixed ? K * K : 0);
  b.ti = take(K * K);
  b.di = take(nb * db * db);
  b.z = take(K * w);
  b.bytes = off * 8;
  return b;
}

}  // namespace bdc
