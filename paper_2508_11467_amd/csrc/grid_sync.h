// Exchange of values between the workgroups of a cooperative launch (all
// resident) through device memory, without barriers and without fences.
//
// On gfx950 every XCD has an L2 of its own, so a device-scope release writes
// back an L2 and an acquire invalidates one, and a barrier made of them costs
// about 10 us and takes the caches' contents with it.  Here every exchanged
// word carries its own arrival: a place holds kEmpty (a NaN that no
// computation makes) until its one writer puts a value there, and a reader
// loads it until it is something else.  All of it goes through relaxed
// device-scope atomics (loads and stores that pass the L2s by); nothing
// relies on the order in which two stores become visible, except that a place
// cleared by its owner is seen cleared at its next use, which is at least two
// whole sums over the grid (and a wait for the clearing store) later.
//
// A sum over the grid of cnt values takes two of these exchanges: workgroup w
// puts its value q at slots[q * G + w]; the values are dealt to the
// workgroups, a wavefront each, which add the G parts in a fixed order and
// put the total; everybody takes the totals.  Three sets of slots and totals
// are used in turn: a workgroup clears its slots of a sum when it has the
// totals, and the totals it put when the next sum is complete (everybody has
// taken them by then).
//
// Every wait is bounded, and a thread waits out the bound once: after an expired
// wait it takes whatever is there, the next sum of its workgroup waits for
// nothing and returns false, and the kernel ends with its work undone.  (The
// bound is a minute or more.  All workgroups are resident once they run, so only
// a launch that another one keeps from its CUs for that long gets there.)
#pragma once

#include <hip/hip_runtime.h>

#include "block_util.h"

namespace bdc {

constexpr unsigned kSpin = 1u << 26;   // loads of a place before a wait expires
constexpr int kGridMaxWg = 512;        // workgroups of a grid, at most
constexpr int kGridSets = 3;
constexpr unsigned long long kEmpty = 0x7FF9B1D5C0DE5EEDull;

__device__ inline void grid_put(double* p, double v) {
  unsigned long long b = (unsigned long long)__double_as_longlong(v);
  if (b == kEmpty) b = 0x7FF8000000000000ull;  // any other NaN
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void grid_clear(double* p) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline unsigned long long grid_peek(const double* p) {
  return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the value of b, a peek at p, or of p once it is there; ok = false when the
// wait expired (with ok false already there is none)
__device__ inline double grid_take(const double* p, unsigned long long b, bool& ok) {
  for (unsigned it = 0; b == kEmpty; ++it) {
    if (!ok || it == kSpin) {
      ok = false;
      break;
    }
    __builtin_amdgcn_s_sleep(1);
    b = grid_peek(p);
  }
  return __longlong_as_double((long long)b);
}

// Completion of this thread's earlier stores (the clears of places that are
// about to be used again); free where loads issued after them are back.
__device__ inline void grid_settle() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Totals of cnt values over the grid: v[q] (LDS, written before a workgroup
// barrier) in, totals out in the same place.  slots, totals: this sum's set;
// prev: the last sum's totals (prev_cnt of them).  All NT threads of all G
// workgroups call it; bad: one word of LDS, zero before the kernel's first
// sum, not zero where a wait of the workgroup has expired.  Ends with a
// workgroup barrier.
template <int NT>
__device__ inline bool grid_sum(double* slots, double* totals, double* prev, int prev_cnt, int cnt, double* v,
                                unsigned* bad) {
  constexpr int NW = NT / 64;
  const int t = threadIdx.x, ln = t & 63, wv = t >> 6;
  const int G = gridDim.x, g = blockIdx.x;
  bool ok = *bad == 0;
  for (int q = t; q < cnt; q += NT) grid_put(slots + (size_t)q * G + g, v[q]);
  // the values dealt to this workgroup
  for (int q = g + G * wv; q < cnt; q += G * NW) {
    const double* s = slots + (size_t)q * G;
    double sum = 0.0;
    for (int w0 = 0; w0 < G; w0 += 256) {
      unsigned long long b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) b[u] = w0 + 64 * u + ln < G ? grid_peek(s + w0 + 64 * u + ln) : 0ull;
#pragma unroll
      for (int u = 0; u < 4; ++u) sum += grid_take(s + w0 + 64 * u + ln, b[u], ok);
    }
    sum = wave_sum_last(sum);
    if (ln == 63) grid_put(totals + q, sum);
  }
  for (int q = t; q < cnt; q += NT) v[q] = grid_take(totals + q, grid_peek(totals + q), ok);
  if (!ok) *bad = 1;
  __syncthreads();
  for (int q = t; q < cnt; q += NT) grid_clear(slots + (size_t)q * G + g);
  for (int q = g + G * wv; q < prev_cnt; q += G * NW)
    if (ln == 63) grid_clear(prev + q);
  return *bad == 0;
}

}  // namespace bdc
