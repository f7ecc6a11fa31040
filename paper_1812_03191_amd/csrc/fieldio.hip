// fieldio.hip -- a level's field to and from host memory.
//
// Bound by the host side: a field of 128^3 FP64 is 16.8 MB, which the link
// moves in 0.3 ms and which the caller's pages, fresh from the allocator, take
// 1.5 ms to receive.  So the device packs: a kernel reads the padded rows of
// departures and writes the values themselves, in FP64 and without padding,
// straight into pinned host memory (no device buffer, no second pass over the
// values on the host), slab by slab into two buffers, and each slab is copied
// to the caller's memory while the next is written.  The five fields of 128^3
// FP64: 31.5 ms when one padded array at a time was copied to pageable memory
// and converted value by value, 9 ms so.  (Three copying threads took 6 ms, but
// beside a program's own thread pool they overran the process's CPU share: a
// snapshot of 4 x 128^3 in FP32 went from 34 to 44 ms, with eight to 101.)
#include "fieldio.h"

#include <algorithm>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>

namespace dfio {

namespace {

constexpr size_t SLAB = (size_t)4 << 20;  // bytes of one staging buffer
constexpr size_t KEEP = 4;                // staging pairs kept while runs are alive

// field entry a (x fastest over e0 x e1 entries per row and plane) at its
// element of the padded level array
__device__ __forceinline__ unsigned entry(const dfk::Geo &G, unsigned a, unsigned e0, unsigned e1) {
  const unsigned i = a % e0, r = a / e0;
  return (unsigned)G.off + i + (r % e1) * (unsigned)G.sy + (r / e1) * (unsigned)G.sz;
}

template <typename T>
__global__ void __launch_bounds__(256) k_field_out(dfk::Geo G, const T *f, unsigned e0, unsigned e1, double back,
                                                   unsigned a0, unsigned n, double *out) {
  const unsigned t = blockIdx.x * 256 + threadIdx.x;
  if (t < n) out[t] = back + (double)f[entry(G, a0 + t, e0, e1)];
}

template <typename T>
__global__ void __launch_bounds__(256) k_field_in(dfk::Geo G, T *f, unsigned e0, unsigned e1, double back,
                                                  unsigned a0, unsigned n, const double *in) {
  const unsigned t = blockIdx.x * 256 + threadIdx.x;
  if (t < n) f[entry(G, a0 + t, e0, e1)] = (T)(in[t] - back);
}

// two pinned buffers and the events that end the kernels on them
struct Stage {
  int dev = 0;
  double *buf[2] = {nullptr, nullptr};
  hipEvent_t ev[2] = {nullptr, nullptr};
};

void stage_free(Stage *s) {
  for (int q = 0; q < 2; ++q) {
    if (s->ev[q]) (void)hipEventDestroy(s->ev[q]);
    if (s->buf[q]) (void)hipHostFree(s->buf[q]);
  }
  delete s;
}

std::mutex g_mu;
Stage *g_free[KEEP];  // idle pairs
size_t g_nfree = 0;
int g_users = 0;

// a pair for a stream: its events belong to the stream's device, whichever
// device is the calling thread's current one
hipError_t stage_take(hipStream_t st, Stage **out) {
  int dev = 0, was = 0;
  hipError_t e = hipStreamGetDevice(st, &dev);
  if (e == hipSuccess) e = hipGetDevice(&was);
  if (e != hipSuccess) return e;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    for (size_t k = 0; k < g_nfree; ++k)
      if (g_free[k]->dev == dev) {
        *out = g_free[k];
        g_free[k] = g_free[--g_nfree];
        return hipSuccess;
      }
  }
  Stage *s = new (std::nothrow) Stage();
  if (!s) return hipErrorOutOfMemory;
  s->dev = dev;
  if (was != dev) e = hipSetDevice(dev);
  for (int q = 0; q < 2 && e == hipSuccess; ++q) {
    e = hipHostMalloc((void **)&s->buf[q], SLAB, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s->ev[q], hipEventDisableTiming);
  }
  if (was != dev) {
    const hipError_t back = hipSetDevice(was);
    if (e == hipSuccess) e = back;
  }
  if (e != hipSuccess) {
    stage_free(s);
    return e;
  }
  *out = s;
  return hipSuccess;
}

void stage_give(Stage *s) {
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_users > 0 && g_nfree < KEEP) {
      g_free[g_nfree++] = s;
      return;
    }
  }
  stage_free(s);
}

}  // namespace

User::User() {
  std::lock_guard<std::mutex> lk(g_mu);
  ++g_users;
}
User::~User() {
  Stage *drop[KEEP];
  size_t n = 0;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (--g_users == 0)
      while (g_nfree) drop[n++] = g_free[--g_nfree];
  }
  while (n) stage_free(drop[--n]);
}

namespace {

// The copy without staging buffers, where none can be had: the field's padded
// rows as they are to pageable memory, and the values between there and the
// caller's; in the other direction the rows' other entries go back unchanged.
template <typename T>
hipError_t field_io_pageable(hipStream_t st, const dfk::Geo &G, T *dev, const int e[3], double back, double *out,
                             const double *in) {
  const size_t n = (size_t)e[0] + (size_t)(e[1] - 1) * G.sy + (size_t)(e[2] - 1) * G.sz;
  const std::unique_ptr<T[]> raw(new (std::nothrow) T[n]);
  if (!raw) return hipErrorOutOfMemory;
  dev += G.off;
  hipError_t rc = hipMemcpyAsync(raw.get(), dev, n * sizeof(T), hipMemcpyDeviceToHost, st);
  if (rc == hipSuccess) rc = hipStreamSynchronize(st);
  if (rc != hipSuccess) return rc;
  size_t a = 0;
  for (int k = 0; k < e[2]; ++k)
    for (int j = 0; j < e[1]; ++j) {
      T *row = raw.get() + (size_t)j * G.sy + (size_t)k * G.sz;
      for (int i = 0; i < e[0]; ++i, ++a) {
        if (out) out[a] = back + (double)row[i];
        else row[i] = (T)(in[a] - back);
      }
    }
  if (out) return hipSuccess;
  rc = hipMemcpyAsync(dev, raw.get(), n * sizeof(T), hipMemcpyHostToDevice, st);
  const hipError_t end = hipStreamSynchronize(st);
  return rc != hipSuccess ? rc : end;
}

}  // namespace

hipError_t field_io(hipStream_t st, const dfk::Geo &G, bool fp32, void *dev, const int e[3], double back, double *out,
                    const double *in) {
  const size_t count = (size_t)e[0] * e[1] * e[2];  // below 2^31: a level's entries are
  const size_t slab = SLAB / sizeof(double), nslab = (count + slab - 1) / slab;
  Stage *s = nullptr;
  hipError_t rc = stage_take(st, &s);
  if (rc != hipSuccess) {
    (void)hipGetLastError();  // (the next launch is not to report it)
    if (fp32) return field_io_pageable<float>(st, G, (float *)dev, e, back, out, in);
    return field_io_pageable<double>(st, G, (double *)dev, e, back, out, in);
  }
  auto launch = [&](size_t k) -> hipError_t {
    const unsigned a0 = (unsigned)(k * slab), n = (unsigned)std::min(slab, count - k * slab);
    const dim3 gr((n + 255) / 256), bl(256);
    double *b = s->buf[k & 1];
    const unsigned e0 = (unsigned)e[0], e1 = (unsigned)e[1];
    if (out && fp32) k_field_out<float><<<gr, bl, 0, st>>>(G, (const float *)dev, e0, e1, back, a0, n, b);
    else if (out) k_field_out<double><<<gr, bl, 0, st>>>(G, (const double *)dev, e0, e1, back, a0, n, b);
    else if (fp32) k_field_in<float><<<gr, bl, 0, st>>>(G, (float *)dev, e0, e1, back, a0, n, b);
    else k_field_in<double><<<gr, bl, 0, st>>>(G, (double *)dev, e0, e1, back, a0, n, b);
    const hipError_t err = hipGetLastError();
    return err != hipSuccess ? err : hipEventRecord(s->ev[k & 1], st);
  };
  auto host = [&](size_t k) {  // slab k between its buffer and the caller's memory
    const size_t a = k * slab, m = std::min(slab, count - a) * sizeof(double);
    if (out) std::memcpy(out + a, s->buf[k & 1], m);
    else std::memcpy(s->buf[k & 1], in + a, m);
  };
  if (out) {
    size_t queued = 0;  // slabs whose kernel and event are on the stream
    for (size_t k = 0; k < nslab && rc == hipSuccess; ++k) {
      for (; queued < nslab && queued < k + 2 && rc == hipSuccess; ++queued) rc = launch(queued);
      if (rc == hipSuccess) rc = hipEventSynchronize(s->ev[k & 1]);
      if (rc == hipSuccess) host(k);
    }
  } else {
    for (size_t k = 0; k < nslab && rc == hipSuccess; ++k) {
      if (k >= 2) rc = hipEventSynchronize(s->ev[k & 1]);
      if (rc != hipSuccess) break;
      host(k);
      rc = launch(k);
    }
  }
  // nothing on the stream uses the buffers once they are given back
  const hipError_t end = hipStreamSynchronize(st);
  stage_give(s);
  return rc != hipSuccess ? rc : end;
}

}  // namespace dfio
