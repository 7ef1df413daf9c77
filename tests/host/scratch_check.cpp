// Host check of what the C entry points do with their scratch
// (paper_2508_11467_amd/csrc/api.cpp), built without a GPU by
// tests/test_host_scratch.py: the HIP runtime is a small fake (memory with a
// limit, a last error that stays until it is read, counters), the launchers
// note the plans that they are given.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "backtr.h"
#include "bdc.h"
#include "bdc_internal.h"
#include "gebrd.h"
#include "qr.h"

using namespace bdc;

static int fails = 0;
#define CHECK(c)                                                          \
  do {                                                                    \
    if (!(c)) {                                                           \
      std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
      ++fails;                                                            \
    }                                                                     \
  } while (0)

// ---------------------------------------------------------------- the fake runtime
static size_t g_limit = SIZE_MAX, g_used = 0;  // device memory
static std::map<void*, size_t> g_mem;
static hipError_t g_last = hipSuccess;
static int g_graphs = 0, g_leaves = 0;  // sequences launched, leaf launches
static int g_mallocs = 0, g_frees = 0, g_syncs = 0;
static int g_devices = 1, g_streams = 0;
static bool g_capturing = false;
static hipStream_t g_synced = nullptr, g_recorded = nullptr;  // last one waited for by the host; the stream of the last event
static std::map<std::pair<hipStream_t, hipStream_t>, int> g_waits;  // (stream waited for, waiting one)

static int traffic() { return g_mallocs + g_frees + g_syncs; }

static hipError_t fail(hipError_t e) { return g_last = e; }

extern "C" {
hipError_t hipGetDeviceCount(int* n) { return *n = g_devices, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes) {
  ++g_mallocs;
  if (g_capturing) return *p = nullptr, fail(hipErrorStreamCaptureUnsupported);
  if (bytes > g_limit - g_used) return *p = nullptr, fail(hipErrorOutOfMemory);
  *p = std::malloc(1);
  g_mem[*p] = bytes;
  g_used += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  ++g_frees;
  g_used -= g_mem.at(p);
  g_mem.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t hipStreamSynchronize(hipStream_t st) { return g_synced = st, ++g_syncs, hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t st) { return g_recorded = st, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0.0f, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  ++g_streams;
  return *s = (hipStream_t)2, hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t, unsigned) { return g_waits[{g_recorded, st}]++, hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return *g = (hipGraph_t)3, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return *e = (hipGraphExec_t)4, hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  return *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return ++g_graphs, hipSuccess; }
}

// ---------------------------------------------------------------- the launchers
static BtPlan g_plan{};       // of the last back-transformation
static size_t g_scratch = 0;  // and the bytes of its scratch

static void note(const BtPlan& plan, void* scratch) {
  g_plan = plan;
  g_scratch = g_mem.at(scratch);
  CHECK(plan.bytes <= g_scratch);
}

namespace bdc {
void launch_backtr(int, int, int, int, int, const double*, int64_t, int64_t, const double*, double*, int,
                   const BtPlan& plan, void* scratch, hipStream_t) {
  note(plan, scratch);
}
int launch_geqrf(int, int, int, double*, int, double*, int, void*, size_t, const BtPlan& plan, void* scratch,
                 hipStream_t) {
  note(plan, scratch);
  return BDC_OK;
}
void launch_orgqr(int, int, int, const double*, int, const double*, double*, int, const BtPlan& plan, void* scratch,
                  hipStream_t) {
  note(plan, scratch);
}
void* backtr_fixed_scratch(int) { return nullptr; }
size_t qr_sync_bytes(int) { return 4096; }
int qr_max_block() { return 64; }
int launch_gebrd(int, int m, int n, double*, int, double*, double*, double*, double*, int b, void* work, size_t bytes,
                 int max_wg, hipStream_t) {
  CHECK(bytes == g_mem.at(work) && gebrd_work_bytes(m, n, b, max_wg) <= bytes);
  return BDC_OK;
}
int oz_supported(int) { return 1; }
bool crt_supported(int) { return true; }
int mlp_parts(int) { return 1; }
size_t mlp_pack_bytes() { return 8; }
void launch_reset(Ctl*, NodeState*, SecCount*, int, const Io&, hipStream_t) {}
void launch_leaf(const LeafDesc*, int, int, const Work&, hipStream_t) { ++g_leaves; }
void launch_prep(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_rotate(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_gather(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_secular(const NodeDesc*, int, int, bool, const Work&, hipStream_t) {}
void launch_lowner(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_vectors(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_order(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_update(const NodeDesc*, int, int, const Work&, const Tuning&, hipStream_t) {}
void launch_update_crt(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_update_ozaki(const NodeDesc*, int, int, const Work&, hipStream_t) {}
void launch_harvest(const NodeDesc*, int, int, const Work&, const Harvest&, hipStream_t) {}
void launch_final_single(int64_t, const Work&, hipStream_t) {}
void launch_final(const int64_t*, const int64_t*, const int64_t*, const int64_t*, const int64_t*, const int32_t*,
                  const int32_t*, int64_t, int64_t, const Work&, hipStream_t) {}
void launch_mlp_pack(const float*, unsigned short*, hipStream_t) {}
void launch_mlp_forward(const float*, const float*, int, float*, hipStream_t) {}
void launch_mlp_grad(const float*, const float*, const float*, const int*, int, float*, float*, hipStream_t) {}
void launch_adam(float*, float*, float*, const float*, int, const float*, float*, float*, int, float, float,
                 hipStream_t) {}
}  // namespace bdc

// ---------------------------------------------------------------- the checks
static double d_arg;  // stands for any device array

static bdc_handle_t handle(size_t cap = 0, int device = 0) {
  bdc_options_t o;
  bdc_default_options(&o);
  o.workspace_cap_bytes = cap;
  bdc_handle_t h = nullptr;
  CHECK(bdc_create(&h, device, &o) == BDC_OK);
  return h;
}

static int apply(bdc_handle_t h, int m, int p, int k, int block = 0) {
  return bdc_apply_reflectors(h, 0, m, p, k, 0, &d_arg, 1, m, &d_arg, &d_arg, m, block, nullptr);
}
static int geqrf(bdc_handle_t h, int m, int n) { return bdc_geqrf(h, m, n, &d_arg, m, &d_arg, 0, nullptr); }
static int orgqr(bdc_handle_t h, int m, int n) {
  return bdc_orgqr(h, m, n, n, &d_arg, m, &d_arg, &d_arg, m, 0, nullptr);
}

// Memory that holds the scratch of one block at a time but not that of a
// group: the call is served and reports no error, and neither does the next.
static void out_of_memory() {
  const int m = 3000, p = 700, k = 900;
  bdc_handle_t h = handle();
  g_limit = backtr_limit_bytes(m, p, 64);
  CHECK(backtr_plan(m, p, p, kBtMaxGroup, false).bytes > g_limit);
  CHECK(apply(h, m, p, k) == BDC_OK);
  CHECK(g_plan.group == 64 && g_plan.fixed);
  CHECK(apply(h, m, p, k) == BDC_OK);
  CHECK(orgqr(h, m, p) == BDC_OK);
  // and where there is none at all, the status says so
  g_limit = g_used;
  CHECK(apply(h, 2 * m, p, k) == BDC_ERR_NOMEM);
  g_limit = SIZE_MAX;
  CHECK(apply(h, m, p, k) == BDC_OK);
  CHECK(bdc_destroy(h) == BDC_OK);
}

// Where a cap, or the memory there is, admits only one block at a time, the
// scratch is kept from call to call like any other: the second round of calls
// allocates, frees and waits for nothing.
static void kept() {
  const int m = 3000, p = 700, k = 900;
  for (int capped = 0; capped < 2; ++capped) {
    const size_t most = backtr_limit_bytes(m, p, 64);
    bdc_handle_t h = handle(capped ? most : 0);
    g_limit = capped ? SIZE_MAX : most + qr_sync_bytes(1);
    for (int round = 0; round < 3; ++round) {
      const int before = traffic();
      CHECK(apply(h, m, p, k) == BDC_OK && g_plan.group == 64 && g_plan.fixed);
      CHECK(orgqr(h, m, p) == BDC_OK && g_plan.group == 64);
      CHECK(geqrf(h, m, p) == BDC_OK);
      CHECK(apply(h, m - 100, p, k) == BDC_OK);
      if (round > 0) CHECK(traffic() == before);
    }
    // a scratch that fits is still had
    CHECK(apply(h, 500, 100, 300) == BDC_OK && g_plan.group == kBtMaxGroup);
    g_limit = SIZE_MAX;
    CHECK(bdc_destroy(h) == BDC_OK);
  }
}

// Few reflectors take the scratch and the depth slices of as many, not those of
// a full group.
static void few_reflectors() {
  const int m = 1000000, p = 64;
  for (int k : {1, 4, 20, 64}) {
    bdc_handle_t h = handle();
    CHECK(apply(h, m, p, k) == BDC_OK);
    CHECK(g_scratch <= 1.25 * backtr_limit_bytes(m, p, 64));
    CHECK(bdc_destroy(h) == BDC_OK);
  }
  // the products Y^T [C | Y] have a workgroup for about every CU
  for (int k : {20, 64, 100}) {
    const int rows = 20000, cols = 1000, tm = bt_tile_rows(k), slice = bt_slice(rows, cols, k);
    const int slices = (rows + slice - 1) / slice, tiles = (k + tm - 1) / tm * ((cols + 127) / 128);
    CHECK(slices * tiles >= 200);
  }
  // The last group of a call is no wider than what is left of it; whatever is
  // left, its slices fit what the plan holds.
  for (int m1 : {1, 63, 129, 1000, 4097, 20000, 300000})
    for (int p1 : {1, 130, 1000})
      for (int group : {1, 32, 64, 128}) {
        const BtPlan b = backtr_plan(m1, p1, p1, group, false);
        const size_t held = (b.pt - b.p) / p1;
        for (int bw = 1; bw <= std::min(group, m1); ++bw)
          for (int rows : {m1, (m1 + 1) / 2, std::min(m1, bw)}) {
            const int s = bt_slice(rows, p1, bw);
            CHECK((size_t)((rows + s - 1) / s) * bw <= held);
          }
      }
}

// Under a stream capture nothing may be allocated.  The scratch of an earlier
// call of the same sizes serves any number of reflectors.
static void captured() {
  for (int m : {100, 3000, 60000}) {
    bdc_handle_t h = handle();
    CHECK(apply(h, m, 700, 20) == BDC_OK);
    const int before = traffic();
    g_capturing = true;
    for (int k : {20, 64, 65, 2000}) CHECK(apply(h, m, 700, k) == BDC_OK);
    CHECK(traffic() == before);
    g_capturing = false;
    CHECK(apply(h, m, 700, 2000) == BDC_OK && g_plan.group == kBtMaxGroup && !g_plan.fixed);
    CHECK(bdc_destroy(h) == BDC_OK);
  }
}

// Solves are captured on every device that there is.
static void many_devices() {
  g_devices = 100;
  for (int device : {0, 63, 64, 99}) {
    bdc_handle_t a = handle(0, device), b = handle(0, device);
    double out[3];
    const int before = g_streams;
    for (bdc_handle_t h : {a, b, a}) CHECK(bdc_svd(h, 100, out, out, out, out + 1, out + 2, nullptr) == BDC_OK);
    CHECK(g_streams == before + 1);  // one capture stream for the device's handles
    CHECK(bdc_destroy(a) == BDC_OK && bdc_destroy(b) == BDC_OK);
  }
}

// A cap that held the reduction's scratch when its exchange had no places of
// m and n (2 x 64 groups' and 2 x 2048 workgroups' sums of 66 and a barrier's
// state) still does.
static void reduction_under_a_cap() {
  for (int block : {0, 3, 32})
    for (int m : {40, 5000, 60000, 2000000})
      for (int n : {40, 1000}) {
        const int b = block ? block : 32;
        const size_t cap = 4352 + 8 * ((size_t)2 * b * m + (size_t)2 * b * n + 2 * (2048 + 64) * 66);
        bdc_handle_t h = handle(cap);
        int before = 0;
        for (int round = 0; round < 2; ++round) {
          CHECK(bdc_gebrd(h, m, n > m ? m : n, &d_arg, m, &d_arg, &d_arg, &d_arg, &d_arg, block, nullptr) == BDC_OK);
          if (round) CHECK(traffic() == before);
          before = traffic();
        }
        CHECK(bdc_destroy(h) == BDC_OK);
        h = handle(cap / 2);
        if (m > 5000)
          CHECK(bdc_gebrd(h, m, n, &d_arg, m, &d_arg, &d_arg, &d_arg, &d_arg, block, nullptr) == BDC_ERR_NOMEM);
        CHECK(bdc_destroy(h) == BDC_OK);
      }
}

// A solve on another stream than the last one starts after that one has ended,
// whatever its buffers (both use the handle's workspace); on the same stream,
// and under a capture, nothing is added.
static void streams() {
  hipStream_t a = (hipStream_t)16, b = (hipStream_t)32;
  double x[6];
  bdc_handle_t h = handle();
  CHECK(bdc_svd(h, 100, x, x, x, x + 1, x + 2, a) == BDC_OK);
  CHECK(g_waits.empty());
  const int before = g_syncs;
  CHECK(bdc_svd(h, 100, x, x, x, x + 1, x + 2, a) == BDC_OK);
  CHECK(g_waits.empty() && g_syncs == before);
  CHECK(bdc_svd(h, 100, x, x, x + 3, x + 4, x + 5, b) == BDC_OK);
  CHECK(g_waits.count({a, b}) == 1 || (g_syncs > before && g_synced == a));
  CHECK(bdc_svd(h, 100, x, x, x, x + 1, x + 2, nullptr) == BDC_OK);
  CHECK(g_waits.count({b, nullptr}) == 1 || g_synced == b);
  g_waits.clear();
  g_capturing = true;
  const int traffic_before = traffic();
  CHECK(bdc_svd(h, 100, x, x, x, x + 1, x + 2, a) == BDC_OK);
  CHECK(g_waits.empty() && traffic() == traffic_before);
  g_capturing = false;
  CHECK(bdc_destroy(h) == BDC_OK);
}

// A solve under the caller's own capture is recorded launch by launch: a
// captured sequence launched there would run at once, with the last call's
// buffers.
static void captured_solve() {
  double x[6];
  bdc_handle_t h = handle();
  CHECK(bdc_svd(h, 100, x, x, x, x + 1, x + 2, nullptr) == BDC_OK);
  CHECK(g_graphs == 1);
  g_capturing = true;
  g_leaves = 0;
  const int before = traffic();
  CHECK(bdc_svd(h, 100, x, x, x + 3, x + 4, x + 5, nullptr) == BDC_OK);
  CHECK(g_graphs == 1 && g_leaves == 1 && traffic() == before);
  g_capturing = false;
  CHECK(bdc_svd(h, 100, x, x, x, x + 1, x + 2, nullptr) == BDC_OK);
  CHECK(g_graphs == 2 && g_leaves == 1);
  CHECK(bdc_destroy(h) == BDC_OK);
}

int main(int argc, char** argv) {
  const std::string which = argc > 1 ? argv[1] : "";
  if (which == "out_of_memory") out_of_memory();
  else if (which == "kept") kept();
  else if (which == "few_reflectors") few_reflectors();
  else if (which == "captured") captured();
  else if (which == "many_devices") many_devices();
  else if (which == "reduction_under_a_cap") reduction_under_a_cap();
  else if (which == "streams") streams();
  else if (which == "captured_solve") captured_solve();
  else return 2;
  CHECK(g_mem.empty());
  std::printf("%s: %d failures\n", which.c_str(), fails);
  return fails != 0;
}
