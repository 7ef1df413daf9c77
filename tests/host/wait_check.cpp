// Host check of the bounded waits of a grid's exchange
// (paper_2508_11467_amd/csrc/grid_sync.h), compiled by
// tests/test_host_waits.py without a GPU: one thread, and device memory in
// which some places stay empty.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <set>

// the device functions that the header uses, as one thread on the host has them
struct Index {
  int x;
};
static Index threadIdx{0}, blockIdx{0}, gridDim{1};
static void __syncthreads() {}
static double __longlong_as_double(long long v) {
  double d;
  std::memcpy(&d, &v, 8);
  return d;
}
static long long __double_as_longlong(double d) {
  long long v;
  std::memcpy(&v, &d, 8);
  return v;
}
static void __builtin_amdgcn_s_sleep(int) {}
static unsigned long long g_loads = 0, g_arrives = 0;  // loads so far; the load that finds a value
static unsigned long long load(const unsigned long long* p);
#define __hip_atomic_load(p, order, scope) load(p)
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
#define __HIP_MEMORY_SCOPE_AGENT 0

#include "grid_sync.h"

static unsigned long long load(const unsigned long long* p) {
  ++g_loads;
  return g_loads == g_arrives ? 0x3FF0000000000000ull : *p;
}

using namespace bdc;

static int fails = 0;
#define CHECK(c)                                                          \
  do {                                                                    \
    if (!(c)) {                                                           \
      std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
      ++fails;                                                            \
    }                                                                     \
  } while (0)

int main() {
  double place[4];
  for (double& p : place) grid_clear(&p);
  bool ok = true;
  // a value that comes late (a device held by another launch for a while)
  g_arrives = 1ull << 25;
  CHECK(grid_take(place, grid_peek(place), ok) == 1.0 && ok);
  // one that does not come ends the wait, and no later place is waited for
  g_loads = g_arrives = 0;
  for (double& p : place) (void)grid_take(&p, grid_peek(&p), ok);
  CHECK(!ok && g_loads <= kSpin + 8ull);
  // nor is anything in a sum that the workgroup enters with a wait expired
  double slots[2 * kGridSets], totals[2 * kGridSets], v[2] = {1.0, 2.0};
  for (double& p : slots) grid_clear(&p);
  for (double& p : totals) grid_clear(&p);
  unsigned bad = 1;
  gridDim.x = 2;  // the other workgroup never comes
  g_loads = 0;
  CHECK(!grid_sum<64>(slots, totals, totals, 0, 2, v, &bad));
  CHECK(g_loads <= 16);
  std::printf("%d failures\n", fails);
  return fails != 0;
}
