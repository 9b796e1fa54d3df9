// A stand-in for the HIP runtime, for checks of the library's host code on a
// machine without a GPU.  An executable that includes this file and links
// libsv.so has its definitions of the runtime's functions take precedence:
// kernels are recorded by name and not run, copies to the device are recorded
// with their bytes, and a chosen launch can be made to fail.  Device pointers
// are plain numbers that nobody reads, so any state size will do.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>
#include <string>
#include <vector>

namespace rt {

struct Event {
  std::string kernel;  // empty: a copy to the device
  size_t bytes = 0;    // of a copy
  size_t allocated = 0;  // host bytes allocated since start() when it was issued
};

inline std::vector<Event> &events() {
  static std::vector<Event> e;
  return e;
}
inline std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> k;
  return k;
}
inline long fail_at = -1;  // launches until one fails
inline size_t recorded = 0;  // events recorded since start()
inline size_t allocated = 0, live = 0, peak = 0;  // host bytes since start()
inline bool counting = false;

inline void start() {
  events().clear();
  recorded = 0;
  allocated = live = peak = 0;
  counting = true;
}
inline void stop() { counting = false; }

// The kernels launched since start(), template arguments and namespaces apart.
inline std::vector<std::string> launched() {
  std::vector<std::string> out;
  for (const Event &e : events())
    if (!e.kernel.empty()) out.push_back(e.kernel);
  return out;
}

// "k_name" from a mangled name: what follows it is upper case
inline std::string short_name(const char *mangled) {
  const std::string s(mangled);
  const size_t at = s.find("k_");
  if (at == std::string::npos) return s;
  size_t end = at;
  while (end < s.size() && (s[end] == '_' || (s[end] >= 'a' && s[end] <= 'z') || (s[end] >= '0' && s[end] <= '9'))) ++end;
  return s.substr(at, end - at);
}

}  // namespace rt

// every allocation of the process, the library's included
void *operator new(size_t n) {
  size_t *p = static_cast<size_t *>(std::malloc(n + 16));
  if (!p) throw std::bad_alloc();
  p[0] = n;
  p[1] = rt::counting;
  if (rt::counting) {
    rt::allocated += n;
    rt::live += n;
    if (rt::live > rt::peak) rt::peak = rt::live;
  }
  return p + 2;
}
void operator delete(void *q) noexcept {
  if (!q) return;
  size_t *p = static_cast<size_t *>(q) - 2;
  if (p[1] && rt::counting && rt::live >= p[0]) rt::live -= p[0];
  std::free(p);
}
void operator delete(void *q, size_t) noexcept { operator delete(q); }
void *operator new[](size_t n) { return operator new(n); }
void operator delete[](void *q) noexcept { operator delete(q); }
void operator delete[](void *q, size_t) noexcept { operator delete(q); }

extern "C" {

void **__hipRegisterFatBinary(const void *) {
  static void *h;
  return &h;
}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {
  rt::kernels()[host] = rt::short_name(name);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
static dim3 rt_grid, rt_block;
static size_t rt_shared;
static hipStream_t rt_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  rt_grid = g;
  rt_block = b;
  rt_shared = s;
  rt_stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
  *g = rt_grid;
  *b = rt_block;
  *s = rt_shared;
  *st = rt_stream;
  return hipSuccess;
}
static hipError_t rt_last = hipSuccess;
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t) {
  if (rt::fail_at >= 0 && rt::fail_at-- == 0) return rt_last = hipErrorLaunchFailure;
  rt::events().push_back({rt::kernels()[f], 0, rt::allocated});
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = rt_last;
  rt_last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipMemcpyAsync(void *, const void *, size_t n, hipMemcpyKind k, hipStream_t) {
  if (k == hipMemcpyHostToDevice) rt::events().push_back({"", n, rt::allocated});
  return hipSuccess;
}
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  *p = std::malloc(n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = reinterpret_cast<hipEvent_t>(1);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) {
  ++rt::recorded;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
  *p = nullptr;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = reinterpret_cast<hipGraph_t>(1);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(1);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"
