// Workgroup-level reductions and scans for 256-thread blocks (4 wave64s).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace bdc {

constexpr int kBlock = 256;

// v combined over the wavefront in the order of lane distances 32, 16, 8, 4, 2
// and 1, in all lanes (op commutative).  Half-wavefront and row swaps, then row
// rotations (after the distance of 8 a row repeats every 8 lanes, and so on, so
// a rotation meets the same partner): no LDS round trips, which made up most of
// the small merges' reductions (a shuffle of a double is 57 cycles).
template <class Op>
__device__ __forceinline__ double half_wave_all(double v, Op op) {  // from the distance of 16 on
  auto swap16 = [&](double x) {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
    return op(__hiloint2double(hi[0], lo[0]), __hiloint2double(hi[1], lo[1]));
  };
  auto rotate = [&](double x, auto ctrl) {
    constexpr int c = decltype(ctrl)::value;
    return op(x, __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), c, 0xF, 0xF, false),
                                  __builtin_amdgcn_update_dpp(0, __double2loint(x), c, 0xF, 0xF, false)));
  };
  v = swap16(v);
  v = rotate(v, std::integral_constant<int, 0x128>{});  // row_ror:8
  v = rotate(v, std::integral_constant<int, 0x124>{});
  v = rotate(v, std::integral_constant<int, 0x122>{});
  return rotate(v, std::integral_constant<int, 0x121>{});
}

// x of the lower half of the wavefront and of the upper half, in both halves
struct Halves {
  double lower, upper;
};
__device__ __forceinline__ Halves wave_halves(double x) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
  return Halves{__hiloint2double(hi[0], lo[0]), __hiloint2double(hi[1], lo[1])};
}

template <class Op>
__device__ __forceinline__ double wave_all(double v, Op op) {
  const Halves h = wave_halves(v);
  return half_wave_all(op(h.lower, h.upper), op);
}

// sum of the lanes' squares, a lane's own square unrounded where it meets the
// other half's
__device__ __forceinline__ double wave_sum_squares(double v) {
  const Halves h = wave_halves(v * v);
  return half_wave_all(fma(v, v, (threadIdx.x & 32) ? h.lower : h.upper), [](double a, double b) { return a + b; });
}

__device__ inline double wave_sum(double v) {
  return wave_all(v, [](double a, double b) { return a + b; });
}

// x plus lane-shifted x's by DPP (no LDS round trip): a shift or broadcast
// `Ctrl` into the rows of 16 lanes that `Rows` names; lanes without a source
// add zero.
template <int Ctrl, int Rows>
__device__ __forceinline__ double dpp_add(double x) {
  return x + __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), Ctrl, Rows, 0xF, false),
                              __builtin_amdgcn_update_dpp(0, __double2loint(x), Ctrl, Rows, 0xF, false));
}

// sum over each row of 16 lanes, in all of them
__device__ __forceinline__ double row_sum(double x) {
  x = dpp_add<0x128, 0xF>(x);  // row_ror:8
  x = dpp_add<0x124, 0xF>(x);
  x = dpp_add<0x122, 0xF>(x);
  return dpp_add<0x121, 0xF>(x);
}

// sum over the wavefront, in lane 63
__device__ __forceinline__ double wave_sum_last(double x) {
  x = dpp_add<0x111, 0xF>(x);     // row_shr:1
  x = dpp_add<0x112, 0xF>(x);
  x = dpp_add<0x114, 0xF>(x);
  x = dpp_add<0x118, 0xF>(x);     // lane 15 of a row: the row's sum
  x = dpp_add<0x142, 0xA>(x);     // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xC>(x);  // row_bcast:31 into rows 2 and 3
}

__device__ inline double wave_maxd(double v) {
  return wave_all(v, [](double a, double b) { return fmax(a, b); });
}

__device__ inline double wave_prod(double v) {
  return wave_all(v, [](double a, double b) { return a * b; });
}

// All threads of the 256-thread block get the block maximum.
__device__ inline double block_max(double v, double* sh /* >= 4 */) {
  v = wave_maxd(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  return fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

__device__ inline double block_sum(double v, double* sh /* >= 4 */) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Exclusive prefix sum over the block of K counters per thread.  sh must hold
// 256*K ints.  total[] receives the block totals.
template <int K>
__device__ inline void block_exscan(int (&v)[K], int (&total)[K], int* sh) {
  const int t = threadIdx.x;
  __syncthreads();
  for (int q = 0; q < K; ++q) sh[q * kBlock + t] = v[q];
  __syncthreads();
  // Hillis-Steele inclusive scan per counter
  for (int off = 1; off < kBlock; off <<= 1) {
    int add[K];
    for (int q = 0; q < K; ++q) add[q] = t >= off ? sh[q * kBlock + t - off] : 0;
    __syncthreads();
    for (int q = 0; q < K; ++q) sh[q * kBlock + t] += add[q];
    __syncthreads();
  }
  for (int q = 0; q < K; ++q) {
    total[q] = sh[q * kBlock + kBlock - 1];
    v[q] = sh[q * kBlock + t] - v[q];
  }
  __syncthreads();
}

// The same for a block of BS threads (a multiple of 64): sh holds BS*K ints.
template <int K, int BS>
__device__ inline void block_exscan_n(int (&v)[K], int (&total)[K], int* sh) {
  const int t = threadIdx.x;
  __syncthreads();
  for (int q = 0; q < K; ++q) sh[q * BS + t] = v[q];
  __syncthreads();
  for (int off = 1; off < BS; off <<= 1) {
    int add[K];
    for (int q = 0; q < K; ++q) add[q] = t >= off ? sh[q * BS + t - off] : 0;
    __syncthreads();
    for (int q = 0; q < K; ++q) sh[q * BS + t] += add[q];
    __syncthreads();
  }
  for (int q = 0; q < K; ++q) {
    total[q] = sh[q * BS + BS - 1];
    v[q] = sh[q * BS + t] - v[q];
  }
  __syncthreads();
}

// Exclusive prefix sums of K counters over a block of BS threads (a multiple
// of 64) with wavefront shuffles: a scan inside each wavefront, then the
// wavefront totals.  sh must hold K * BS/64 ints.  Same results as
// block_exscan_n (integer sums), with two barriers.
template <int K, int BS>
__device__ inline void block_exscan_w(int (&v)[K], int (&total)[K], int* sh) {
  constexpr int NW = BS / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int inc[K];
  for (int q = 0; q < K; ++q) {
    int x = v[q];
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    inc[q] = x;
  }
  __syncthreads();
  if (lane == 63)
    for (int q = 0; q < K; ++q) sh[q * NW + wv] = inc[q];
  __syncthreads();
  for (int q = 0; q < K; ++q) {
    int before = 0, all = 0;
    for (int u = 0; u < NW; ++u) {
      const int t = sh[q * NW + u];
      if (u < wv) before += t;
      all += t;
    }
    total[q] = all;
    v[q] = before + inc[q] - v[q];
  }
  __syncthreads();
}

// Block sum for BS threads; the wave sums are added in wave order.
template <int BS>
__device__ inline double block_sum_n(double v, double* sh /* >= BS/64 */) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int q = 0; q < BS / 64; ++q) s += sh[q];
  return s;
}

// Block maximum for BS threads.
template <int BS>
__device__ inline double block_max_n(double v, double* sh /* >= BS/64 */) {
  v = wave_maxd(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double s = sh[0];
  for (int q = 1; q < BS / 64; ++q) s = fmax(s, sh[q]);
  return s;
}

}  // namespace bdc
