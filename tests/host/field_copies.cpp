// field_copies.cpp -- the field copies of fieldio.hip over a stand-in for the
// HIP runtime with two devices: its entry points below check what a real one
// refuses (an event recorded on another device's stream), carry out the
// library's two kernels on the host, and can be told to fail.  Prints one line
// per check; the exit status is the number of failed ones.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "fieldio.h"

namespace {

struct FakeStream { int dev; };
struct FakeEvent { int dev; };
int g_dev = 0;                       // the calling thread's current device
hipError_t g_last = hipSuccess;      // the sticky error of hipGetLastError
bool g_no_pinned = false;            // hipHostMalloc fails
int g_pinned = 0, g_pinned_total = 0, g_events = 0;
// (kernels are registered before this file's own globals are constructed)
std::map<const void *, std::string> &names() {
  static std::map<const void *, std::string> m;
  return m;
}
dim3 g_grid, g_block;
hipStream_t g_stream;

hipError_t note(hipError_t e) {
  if (e != hipSuccess) g_last = e;
  return e;
}
int dev_of(hipStream_t s) { return s ? reinterpret_cast<FakeStream *>(s)->dev : g_dev; }

template <typename T>
void run_kernel(bool out, void **a) {
  const dfk::Geo &G = *static_cast<dfk::Geo *>(a[0]);
  T *f = *static_cast<T **>(a[1]);
  const unsigned e0 = *static_cast<unsigned *>(a[2]), e1 = *static_cast<unsigned *>(a[3]);
  const double back = *static_cast<double *>(a[4]);
  const unsigned a0 = *static_cast<unsigned *>(a[5]), n = *static_cast<unsigned *>(a[6]);
  double *h = *static_cast<double **>(a[7]);
  for (unsigned t = 0; t < n; ++t) {
    const size_t e = a0 + t, i = e % e0, j = e / e0 % e1, k = e / e0 / e1;
    T &v = f[(size_t)G.off + i + j * (size_t)G.sy + k * (size_t)G.sz];
    if (out) h[t] = back + (double)v;
    else v = (T)(h[t] - back);
  }
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = g_dev; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_dev = d; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d) { *d = dev_of(s); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  if (g_no_pinned) return note(hipErrorOutOfMemory);
  *p = std::malloc(n);
  ++g_pinned;
  ++g_pinned_total;
  return hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); --g_pinned; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new FakeEvent{g_dev});
  ++g_events;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<FakeEvent *>(e); --g_events; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  return note(reinterpret_cast<FakeEvent *>(e)->dev == dev_of(s) ? hipSuccess : hipErrorInvalidHandle);
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t s) {
  g_grid = g;
  g_block = b;
  g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
  *g = g_grid;
  *b = g_block;
  *m = 0;
  *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t) {
  const std::string &k = names()[f];
  const bool out = k.find("k_field_out") != std::string::npos;
  if (k.find("IfE") != std::string::npos) run_kernel<float>(out, args);
  else run_kernel<double>(out, args);
  return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {
  names()[host] = name;
}
}

namespace {

int failed = 0;
void check(bool ok, const char *what) {
  std::printf("%s %s\n", ok ? "ok    " : "FAILED", what);
  failed += ok ? 0 : 1;
}

// a level's padded array and its geometry, and the copies of one field
struct Level {
  dfk::Geo G{};
  int e[3];
  std::vector<char> dev;
  bool fp32;
  Level(int n0, int n1, int n2, bool f32) : e{n0, n1, n2}, fp32(f32) {
    G.sy = (n0 + 1 + 15) / 16 * 16;
    G.sz = G.sy * (n1 + 1);
    G.off = 16;
    dev.assign((size_t)(G.off + (long)G.sz * (n2 + 1)) * (f32 ? 4 : 8), 0x55);
  }
  size_t count() const { return (size_t)e[0] * e[1] * e[2]; }
  hipError_t put(hipStream_t st, const std::vector<double> &v) {
    return dfio::field_io(st, G, fp32, dev.data(), e, 1.0, nullptr, v.data());
  }
  hipError_t get(hipStream_t st, std::vector<double> &v) {
    v.assign(count(), 0.0);
    return dfio::field_io(st, G, fp32, dev.data(), e, 1.0, v.data(), nullptr);
  }
};

// values that both storage types hold exactly, less the background 1
std::vector<double> values(size_t n) {
  std::vector<double> v(n);
  for (size_t i = 0; i < n; ++i) v[i] = 1.0 + (double)(i % 1021) / 1024.0;
  return v;
}

// put and get through st; the entries outside the field stay as they were
bool roundtrip(hipStream_t st, int n0, int n1, int n2, bool fp32) {
  Level L(n0, n1, n2, fp32);
  const std::vector<char> before = L.dev;
  const std::vector<double> want = values(L.count());
  std::vector<double> got;
  if (L.put(st, want) != hipSuccess || L.get(st, got) != hipSuccess || got != want) return false;
  const size_t es = fp32 ? 4 : 8;
  for (int k = 0; k < n2; ++k)
    for (int j = 0; j < n1; ++j)
      std::memset(L.dev.data() + ((size_t)L.G.off + (size_t)j * L.G.sy + (size_t)k * L.G.sz) * es, 0x55, n0 * es);
  return L.dev == before;
}

}  // namespace

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  FakeStream s0{0}, s1{1};
  hipStream_t st0 = reinterpret_cast<hipStream_t>(&s0), st1 = reinterpret_cast<hipStream_t>(&s1);
  if (what == "device") {
    dfio::User run;
    check(roundtrip(st0, 20, 10, 6, false), "the current device's stream");
    check(roundtrip(st1, 20, 10, 6, true), "another device's stream");
    check(g_dev == 0, "the current device is put back");
    g_dev = 1;
    check(roundtrip(st0, 20, 10, 6, false) && roundtrip(st1, 20, 10, 6, false), "the same from the other device");
    check(roundtrip(nullptr, 20, 10, 6, false), "the null stream");
    check(g_pinned == 4, "one idle pair of buffers per device");
  } else if (what == "no pinned memory") {
    dfio::User run;
    g_no_pinned = true;
    check(roundtrip(st0, 2, 2, 2, false) && roundtrip(st0, 2, 2, 2, true), "fields of eight values");
    check(roundtrip(st0, 130, 97, 61, false) && roundtrip(st0, 130, 97, 61, true), "fields of more than a slab");
    check(hipGetLastError() == hipSuccess, "no error left for the next launch");
    g_no_pinned = false;
    check(roundtrip(st0, 130, 97, 61, false) && g_pinned == 2, "staging buffers again once they can be had");
  } else {
    check(false, "unknown check");
  }
  check(g_pinned == 0 && g_events == 0, "buffers and events given back with the last user");
  return failed;
}
