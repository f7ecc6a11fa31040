// engine_host.cpp -- the engine and the step graphs (api.hip) over a stand-in for
// the HIP runtime.  It keeps what is in flight: a graph launched on a stream
// runs until that stream, or an event recorded behind it, is waited for, and
// until then the graph and the memory allocated for it may not go.  Handles are
// checked too.  A kernel launch can be refused, in a capture or outside.  Exit
// status: the number of failed checks.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "df.h"

namespace {

int g_failed = 0;
void fail(const char *what) {
  std::printf("FAILED %s\n", what);
  ++g_failed;
}

struct Handles {
  std::set<void *> live;
  void *make() {
    void *p = std::malloc(8);
    live.insert(p);
    return p;
  }
  void need(void *p, const char *what) {
    if (!live.count(p)) fail(what);
  }
  void drop(void *p, const char *what) {
    need(p, what);
    if (live.erase(p)) std::free(p);
  }
};
Handles streams, events, graphs, execs;
std::map<void *, int> in_flight;             // graph exec -> launches that nothing has waited for
std::map<void *, std::vector<void *>> behind;  // event -> the execs launched before it
std::vector<void *> queue;                   // launches, oldest first (the test has one launching stream)
std::set<void *> device;                     // hipMalloc'd
hipStream_t g_stream;
bool capturing = false;
int recorded = 0;        // launches of the current capture
int refuse = -1;         // the launch of a capture that is refused
hipError_t last = hipSuccess;

void finish(const std::vector<void *> &done) {
  for (void *e : done) in_flight.erase(e);
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) { *d = 0; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { device.insert(*p = std::malloc(n)); return hipSuccess; }
hipError_t hipFree(void *p) {
  if (!in_flight.empty()) fail("device memory freed under a graph in flight");
  device.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)events.make(); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { events.drop(e, "event destroyed twice"); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  events.need(e, "record of no event");
  behind[e] = queue;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { events.need(e, "query of no event"); return hipErrorNotReady; }
hipError_t hipEventSynchronize(hipEvent_t e) {
  events.need(e, "wait for no event");
  finish(behind[e]);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)streams.make(); return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t *s) { return hipStreamCreateWithFlags(s, 0); }
hipError_t hipStreamDestroy(hipStream_t s) { streams.drop(s, "stream destroyed twice"); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (s == g_stream) finish(queue);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  capturing = true;
  recorded = 0;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  capturing = false;
  *g = (hipGraph_t)graphs.make();
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { graphs.drop(g, "graph destroyed twice"); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *e = (hipGraphExec_t)execs.make();
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  if (in_flight.count(e)) fail("graph destroyed in flight");
  execs.drop(e, "instantiated graph destroyed twice");
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  execs.need(e, "launch of no graph");
  g_stream = s;
  in_flight[e] = 1;
  queue.push_back(e);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipPeekAtLastError(void) { return last; }
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = nullptr; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
  *g = *b = dim3(1);
  *m = 0;
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) {
  if (capturing && recorded++ == refuse) {
    refuse = -1;
    return last = hipErrorOutOfMemory;
  }
  return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
}

namespace {

df_mesh_desc mesh(int levels) {
  df_mesh_desc d{};
  d.nx = d.ny = d.nz = 16;
  d.nlevels = levels;
  d.dx0 = 0.1;
  d.gamma = 1.4;
  d.cfl = 0.4;
  d.precision = DF_FP64;
  d.seed = 1;
  return d;
}
const double perturber[5] = {1e-3, 0.1, 1e-3, 0.5, 0.1};

// jobs admitted while others run, then the engine goes with the last replay in
// flight and a replaced graph still to be reaped
void teardown(hipStream_t main) {
  const df_mesh_desc d = mesh(1), nested = mesh(2);
  size_t one = 0, two = 0;
  if (df_engine_job_bytes(&d, &one) || df_engine_job_bytes(&nested, &two)) return fail("job bytes");
  const size_t bytes = 2 * one + two;
  void *arena = std::aligned_alloc(256, bytes);
  df_engine *E = nullptr;
  int32_t slot = -1;
  if (df_engine_create(arena, bytes, main, 2, &E)) return fail("create");
  if (df_engine_admit(E, &d, perturber, 8, &slot) || df_engine_step(E, 1)) return fail("first job");
  if (df_engine_admit(E, &nested, perturber, 8, &slot) || df_engine_step(E, 1)) return fail("second job");
  if (df_engine_admit(E, &d, perturber, 8, &slot) || df_engine_step(E, 1)) return fail("third job");
  if (in_flight.empty()) fail("nothing in flight before the teardown");
  if (df_engine_destroy(E)) fail("destroy");
  std::free(arena);
  queue.clear();
  behind.clear();
  if (!streams.live.empty() || !events.live.empty() || !graphs.live.empty() || !execs.live.empty() || !device.empty())
    fail("handles or device memory left");
}

// a launch that the runtime refuses inside the engine's capture: the step says
// so, and the next one captures again
void refused_in_engine() {
  const df_mesh_desc d = mesh(2);
  size_t bytes = 0;
  if (df_engine_job_bytes(&d, &bytes)) return fail("job bytes");
  void *arena = std::aligned_alloc(256, bytes);
  df_engine *E = nullptr;
  int32_t slot = -1;
  int64_t n[3];
  if (df_engine_create(arena, bytes, nullptr, 2, &E) || df_engine_admit(E, &d, perturber, 8, &slot)) return fail("create");
  refuse = 7;
  if (df_engine_step(E, 1) != DF_EDEVICE) fail("a refused launch of a capture is not reported");
  if (df_engine_stats(E, n) || n[0] != 0 || n[1] != 0) fail("the incomplete graph was kept");
  if (df_engine_step(E, 1) || df_engine_stats(E, n) || n[0] != 1 || n[1] != 1) fail("the step after it");
  if (df_engine_destroy(E)) fail("destroy");
  std::free(arena);
}

// the same in a nested run's step graph
void refused_in_run() {
  const df_mesh_desc d = mesh(2);
  df_run *R = nullptr;
  size_t bytes = 0;
  if (df_init_mesh(&d, &R) || df_required_bytes(R, &bytes)) return fail("mesh");
  void *arena = std::aligned_alloc(256, bytes);
  if (df_bind(R, arena, bytes, nullptr)) return fail("bind");
  if (df_set_perturber(R, perturber[0], perturber[1], perturber[2], perturber[3], perturber[4])) return fail("perturber");
  refuse = 7;
  if (df_step(R, 2) != DF_EDEVICE) fail("a refused launch of a capture is not reported");
  if (!queue.empty()) fail("the incomplete graph was launched");
  if (df_step(R, 2) || queue.size() != 1) fail("the step after it");
  if (df_destroy(R)) fail("destroy");
  std::free(arena);
}

}  // namespace

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "null stream") teardown(nullptr);
  else if (what == "own stream") teardown(reinterpret_cast<hipStream_t>(0x1000));
  else if (what == "launch refused in the engine") refused_in_engine();
  else if (what == "launch refused in a step graph") refused_in_run();
  else fail("unknown check");
  return g_failed;
}
