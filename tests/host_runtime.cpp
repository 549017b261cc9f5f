// The library's host code on a HIP runtime that only keeps account: device
// memory is a range of addresses handed out first fit (nothing behind them),
// kernels are noted by name and grid, copies and graph launches counted. For
// what cannot be arranged on a device on demand: memory that runs out at a
// chosen size, a freed address that comes back. Usage: host_runtime SCENARIO;
// exits 0 when every expectation of the scenario holds.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "vofmt.h"

// ------------------------------------------------------------ the runtime
namespace {

constexpr size_t kBase = 1ull << 40;
size_t g_total = 1ull << 38;       // bytes of device memory
std::map<size_t, size_t> g_live;   // address -> bytes
bool g_capturing = false;          // of the caller's stream
hipError_t g_last = hipSuccess;    // the error that hipGetLastError reports

struct Launch {
  std::string kernel;
  dim3 grid;
  bool operator==(const Launch &o) const {
    return kernel == o.kernel && grid.x == o.grid.x && grid.y == o.grid.y && grid.z == o.grid.z;
  }
};
std::map<const void *, std::string> g_kernels;
std::vector<Launch> g_launches;
int g_uploads = 0, g_graph_launches = 0, g_device_copies = 0, g_frees = 0;

size_t used() {
  size_t s = 0;
  for (auto &a : g_live) s += a.second;
  return s;
}
bool live(const void *p) { return g_live.count((size_t)p) != 0; }

hipError_t fail(hipError_t e) { return g_last = e; }

}  // namespace

hipError_t noalloc_setup(int) { return hipSuccess; }

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
  bytes = (bytes + 4095) & ~(size_t)4095;
  size_t at = kBase;
  for (auto &a : g_live) {
    if (a.first - at >= bytes) break;
    at = a.first + a.second;
  }
  if (at + bytes > kBase + g_total) {
    *p = nullptr;
    return fail(hipErrorOutOfMemory);
  }
  g_live[at] = bytes;
  *p = (void *)at;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (p && !g_live.erase((size_t)p)) return fail(hipErrorInvalidValue);
  g_frees += p != nullptr;
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total) {
  *free_bytes = g_total - used();
  *total = g_total;
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { return (*p = malloc(bytes)) ? hipSuccess : fail(hipErrorOutOfMemory); }
hipError_t hipHostFree(void *p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyHostToDevice) ++g_uploads;
  if (kind == hipMemcpyDeviceToDevice) ++g_device_copies;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDeviceCount(int *n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)1;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = (hipGraph_t)1;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *e = (hipGraphExec_t)1;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
  ++g_graph_launches;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = (hipEvent_t)1;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **, size_t, hipStream_t) {
  g_launches.push_back({g_kernels[f], grid});
  return hipSuccess;
}
static dim3 g_grid, g_block;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  g_grid = grid;
  g_block = block;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream) {
  *grid = g_grid;
  *block = g_block;
  *shared = 0;
  *stream = nullptr;
  return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
  g_kernels[host] = name;
}
}

// ------------------------------------------------------------ the scenarios
namespace {

int g_bad = 0;
#define EXPECT(cond)                                        \
  do {                                                      \
    if (!(cond)) {                                          \
      printf("line %d: not so: %s\n", __LINE__, #cond);     \
      ++g_bad;                                              \
    }                                                       \
  } while (0)

constexpr size_t kRoom = 4 << 20;     // less than any call of 64^3 cells or more needs
double *const kField = (double *)16;  // a caller's pointer (never followed)

vofmt_box cube(int n, int ntr) { return vofmt_box{n, n, n, ntr, kField, kField, kField, kField}; }

struct Ctx {
  vofmt_ctx *c = nullptr;
  Ctx() { EXPECT(vofmt_create(&c, 0) == VOFMT_OK); }
  ~Ctx() {
    vofmt_destroy(c);
    EXPECT(g_live.empty());
  }
  int batch(vofmt_box b, int nsteps, const vofmt_tuning *t = nullptr) {
    return vofmt_advect_batched(c, 1, &b, 0, nsteps, t, nullptr);
  }
  int advect(int n, int ntr, int nsteps) {
    return vofmt_advect(c, n, n, n, ntr, kField, kField, kField, kField, 0, nsteps, nullptr);
  }
};

// A graph is launched again only while the tables that it reads are in place: not
// after another call has given its slab back, even if the same address returns.
void graph_after_failed_growth() {
  Ctx x;
  EXPECT(x.batch(cube(64, 2), 2) == VOFMT_OK);
  EXPECT(x.batch(cube(64, 2), 2) == VOFMT_OK);
  EXPECT(g_uploads == 1 && g_graph_launches == 2);  // the second call took the first one's graph
  EXPECT(x.batch(cube(1024, 3), 2) == VOFMT_OK && g_uploads == 2);
  EXPECT(x.batch(cube(64, 2), 2) == VOFMT_OK && g_uploads == 3);
  g_total = used();
  EXPECT(x.batch(cube(1400, 1), 2) == VOFMT_E_NOMEM);  // the slab is gone
  EXPECT(x.batch(cube(64, 2), 2) == VOFMT_OK);
  EXPECT(g_uploads == 4);
  EXPECT(x.batch(cube(64, 2), 2) == VOFMT_OK);
  EXPECT(g_uploads == 4 && g_graph_launches == 6);
}

// A call that found no memory says so itself; the next call is none the worse.
void call_after_no_memory() {
  Ctx x;
  const size_t total = g_total;
  g_total = 1 << 20;
  EXPECT(x.advect(128, 1, 2) == VOFMT_E_NOMEM);
  g_total = total;
  EXPECT(x.advect(16, 1, 2) == VOFMT_OK);
}

// A captured call keeps its third field copy: a later call that would need a
// larger one goes without it (its result is copied back), nothing is freed.
void captured_third_copy() {
  Ctx x;
  EXPECT(x.advect(96, 1, 2) == VOFMT_OK);  // every other buffer is large enough from here on
  EXPECT(x.batch(cube(64, 1), 2) == VOFMT_OK);
  const size_t before = used();
  EXPECT(x.advect(48, 1, 1) == VOFMT_OK && g_device_copies == 0);
  const size_t third = used() - before;
  EXPECT(third >= 8u * 48 * 48 * 48 && g_frees == 0);
  g_capturing = true;
  EXPECT(x.advect(48, 1, 1) == VOFMT_OK && g_device_copies == 0);
  g_capturing = false;
  EXPECT(x.advect(96, 1, 1) == VOFMT_OK);
  EXPECT(g_device_copies == 1 && g_frees == 0 && used() == before + third);
  EXPECT(x.batch(cube(64, 1), 1) == VOFMT_OK);
  EXPECT(g_launches.back().kernel.find("k_copy_b") != std::string::npos);
  EXPECT(g_frees == 0 && used() == before + third);
  EXPECT(x.advect(40, 1, 1) == VOFMT_OK && g_device_copies == 1);  // fits: no copy back
}

// The third field copy is given back to a call that finds no memory otherwise,
// unless a captured graph works in it; a cached graph that did is made anew.
void third_copy_given_back() {
  {
    Ctx x;
    EXPECT(x.batch(cube(160, 1), 1) == VOFMT_OK && g_uploads == 1);
    EXPECT(x.batch(cube(160, 1), 1) == VOFMT_OK && g_uploads == 1);
    g_total = kRoom + used();
    EXPECT(x.advect(64, 1, 2) == VOFMT_OK);  // needs more than there is
    EXPECT(g_frees == 1);
    EXPECT(x.batch(cube(160, 1), 1) == VOFMT_OK && g_uploads == 2);
    EXPECT(g_launches.back().kernel.find("k_copy_b") != std::string::npos);
  }
  g_total = 1ull << 38;
  g_frees = 0;
  Ctx x;
  EXPECT(x.advect(96, 1, 1) == VOFMT_OK);
  g_capturing = true;
  EXPECT(x.advect(96, 1, 1) == VOFMT_OK);
  g_capturing = false;
  g_total = kRoom + used();
  EXPECT(x.batch(cube(64, 1), 2) == VOFMT_E_NOMEM && g_frees == 0);
}

// The third field copy leaves a quarter of the device's memory to others.
void third_copy_leaves_room() {
  Ctx x;
  EXPECT(x.advect(128, 1, 2) == VOFMT_OK);
  const size_t field = 8u * 128 * 128 * 128, before = used();
  g_total = 4 * (before + field) / 3 - 4096;
  EXPECT(x.advect(128, 1, 1) == VOFMT_OK && g_device_copies == 1 && used() == before);
  g_total = 4 * (before + field) / 3 + 4096;
  EXPECT(x.advect(128, 1, 1) == VOFMT_OK && g_device_copies == 1 && used() == before + field);
  g_total = before + field;  // at hand: taken, however full the device is by then
  EXPECT(x.advect(128, 1, 3) == VOFMT_OK && g_device_copies == 1);
}

// The autotuner's candidates hold the launches of an untuned call, so that a caller
// who tunes is at least as fast as one who does not; chunk 16 or 64 as well.
void tuning_holds_untuned() {
  Ctx x;
  for (int n : {32, 60, 128, 200, 256}) {
    g_launches.clear();
    EXPECT(x.batch(cube(n, 5), 2) == VOFMT_OK);
    const std::vector<Launch> untuned = g_launches;
    g_launches.clear();
    const vofmt_tuning t{32, 16};
    EXPECT(x.batch(cube(n, 5), 2, &t) == VOFMT_OK);
    EXPECT(g_launches.empty() || g_launches == untuned);  // (empty: the same graph)
    g_launches.clear();
    const vofmt_tuning fixed{32, 4};
    EXPECT(x.batch(cube(n, 5), 2, &fixed) == VOFMT_OK);
    for (const Launch &l : g_launches) EXPECT(l.grid.x == 4 * 256);
  }
}

// Every candidate is timed on the caller's fields, not on those that the candidates
// before it have advanced.
void tuning_on_equal_fields() {
  Ctx x;
  const vofmt_box b[3] = {cube(40, 2), cube(64, 1), cube(33, 3)};
  vofmt_tuning best;
  EXPECT(vofmt_autotune_batched(x.c, 3, b, 2, &best, nullptr, nullptr) == VOFMT_OK);
  EXPECT(g_device_copies == 3 * 12);
}

const std::map<std::string, std::function<void()>> kScenarios = {
    {"graph_after_failed_growth", graph_after_failed_growth},
    {"call_after_no_memory", call_after_no_memory},
    {"captured_third_copy", captured_third_copy},
    {"third_copy_given_back", third_copy_given_back},
    {"third_copy_leaves_room", third_copy_leaves_room},
    {"tuning_holds_untuned", tuning_holds_untuned},
    {"tuning_on_equal_fields", tuning_on_equal_fields},
};

}  // namespace

int main(int argc, char **argv) {
  const auto s = kScenarios.find(argc > 1 ? argv[1] : "");
  if (s == kScenarios.end()) {
    for (auto &k : kScenarios) printf("%s\n", k.first.c_str());
    return 2;
  }
  s->second();
  return g_bad ? 1 : 0;
}
