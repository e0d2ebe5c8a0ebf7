// A stand-in for the HIP runtime that needs no GPU: it defines the runtime calls that
// libsparc_hip.so makes, so that the library's host code (which device a call works on, which
// kernels a call launches and with what grid, what it allocates) can be run and looked at on
// the CPU.  Kernels are recorded and not executed; device memory is host memory that starts
// at zero and is never touched by a kernel.  Linked into an executable, these definitions come before the
// ones of the real runtime.
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <map>
#include <string>
#include <vector>

namespace fake {

constexpr int kDevices = 2;
constexpr unsigned kMaxGridYZ = 65535;
constexpr size_t kDefaultLds = 65536;

struct Launch {
  std::string kernel;   // demangled as far as the source name: cg_step_kernel
  dim3 grid, block;
  size_t lds;
  int device;           // the stream's
  hipStream_t stream;
};
struct Stream { int device; };
struct Event { int device; };

inline int current = 0;
inline double readback = 0.0;   // what small device-to-host copies return (in every double)
inline std::vector<Launch> launches;
inline std::vector<int> streams_made, events_made;   // the device of each
inline int n_malloc = 0, n_memcpy = 0, n_sync = 0, n_event_sync = 0;
inline float (*elapsed)() = nullptr;   // what the next pair of events is apart (1 ms without one)
inline hipError_t last = hipSuccess;
// registered by the library's constructors, which run before this program's own
inline std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> k;
  return k;
}
inline std::map<std::pair<const void*, int>, size_t> lds_limit;

// the source name inside a mangled one: _ZN5sparc14cg_step_kernel... -> cg_step_kernel
inline std::string source_name(const char* m) {
  const char* p = strstr(m, "5sparc");
  if (!p) return m;
  p += 6;
  const int n = atoi(p);
  while (*p >= '0' && *p <= '9') ++p;
  return std::string(p, n);
}

inline int count(const char* kernel) {
  int n = 0;
  for (const Launch& l : launches) n += l.kernel == kernel;
  return n;
}

inline void clear() {
  launches.clear();
  streams_made.clear();
  events_made.clear();
  n_malloc = n_memcpy = n_sync = n_event_sync = 0;
}

inline int device_of(hipStream_t s) { return s ? ((Stream*)s)->device : current; }

inline hipError_t copy(void* dst, const void* src, size_t n, hipMemcpyKind kind) {
  ++n_memcpy;
  if (kind == hipMemcpyDeviceToHost) {
    char* d = (char*)dst;
    for (size_t i = 0; i + 8 <= n; i += 8) memcpy(d + i, &readback, 8);
    return hipSuccess;
  }
  if (kind == hipMemcpyHostToDevice) memcpy(dst, src, n);
  return hipSuccess;   // device to device: contents are of no interest
}

}  // namespace fake

#define FAKE_EXPORT extern "C" __attribute__((visibility("default")))

FAKE_EXPORT void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
FAKE_EXPORT void __hipUnregisterFatBinary(void**) {}
FAKE_EXPORT void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*,
                                       void*, int*) {
  fake::kernels()[f] = fake::source_name(name);
}
FAKE_EXPORT void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

namespace fake {
struct Config { dim3 grid, block; size_t lds; hipStream_t stream; };
inline Config config;
}
FAKE_EXPORT hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  fake::config = {g, b, lds, s};
  return hipSuccess;
}
FAKE_EXPORT hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = fake::config.grid;
  *b = fake::config.block;
  *lds = fake::config.lds;
  *s = fake::config.stream;
  return hipSuccess;
}

FAKE_EXPORT hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, hipStream_t s) {
  const int dev = fake::device_of(s);
  fake::launches.push_back({fake::kernels()[f], g, b, lds, dev, s});
  size_t limit = fake::kDefaultLds;
  const auto it = fake::lds_limit.find({f, dev});
  if (it != fake::lds_limit.end()) limit = it->second;
  const bool ok = g.x && g.y && g.z && b.x && b.x * b.y * b.z <= 1024 && g.x <= 0x7fffffffu && g.y <= fake::kMaxGridYZ &&
                  g.z <= fake::kMaxGridYZ && lds <= limit;
  if (!ok) fake::last = hipErrorInvalidConfiguration;
  return ok ? hipSuccess : hipErrorInvalidConfiguration;
}

FAKE_EXPORT hipError_t hipGetDeviceCount(int* n) { *n = fake::kDevices; return hipSuccess; }
FAKE_EXPORT hipError_t hipGetDevice(int* d) { *d = fake::current; return hipSuccess; }
FAKE_EXPORT hipError_t hipSetDevice(int d) { fake::current = d; return hipSuccess; }
#undef hipGetDeviceProperties
FAKE_EXPORT hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t* p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  return hipSuccess;
}
FAKE_EXPORT const char* hipGetErrorString(hipError_t) { return "fake"; }
FAKE_EXPORT hipError_t hipGetLastError() {
  const hipError_t e = fake::last;
  fake::last = hipSuccess;
  return e;
}
FAKE_EXPORT hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char scratch[64];
  *p = scratch;
  return hipSuccess;
}
FAKE_EXPORT hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int v) {
  fake::lds_limit[{f, fake::current}] = (size_t)v;
  return hipSuccess;
}
FAKE_EXPORT hipError_t hipMalloc(void** p, size_t n) {
  ++fake::n_malloc;
  *p = calloc(1, n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
FAKE_EXPORT hipError_t hipFree(void* p) { free(p); return hipSuccess; }
FAKE_EXPORT hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { return fake::copy(d, s, n, k); }
FAKE_EXPORT hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  return fake::copy(d, s, n, k);
}
FAKE_EXPORT hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) {
  return hipSuccess;
}
FAKE_EXPORT hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
FAKE_EXPORT hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }

FAKE_EXPORT hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  fake::streams_made.push_back(fake::current);
  *s = (hipStream_t) new fake::Stream{fake::current};
  return hipSuccess;
}
FAKE_EXPORT hipError_t hipStreamDestroy(hipStream_t s) { delete (fake::Stream*)s; return hipSuccess; }
FAKE_EXPORT hipError_t hipStreamSynchronize(hipStream_t) { ++fake::n_sync; return hipSuccess; }
FAKE_EXPORT hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
FAKE_EXPORT hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
FAKE_EXPORT hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
FAKE_EXPORT hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
FAKE_EXPORT hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
FAKE_EXPORT hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
FAKE_EXPORT hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

FAKE_EXPORT hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  fake::events_made.push_back(fake::current);
  *e = (hipEvent_t) new fake::Event{fake::current};
  return hipSuccess;
}
FAKE_EXPORT hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
FAKE_EXPORT hipError_t hipEventDestroy(hipEvent_t e) { delete (fake::Event*)e; return hipSuccess; }
FAKE_EXPORT hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  return ((fake::Event*)e)->device == fake::device_of(s) ? hipSuccess : hipErrorInvalidHandle;
}
FAKE_EXPORT hipError_t hipEventSynchronize(hipEvent_t) { ++fake::n_event_sync; return hipSuccess; }
FAKE_EXPORT hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = fake::elapsed ? fake::elapsed() : 1.0f;
  return hipSuccess;
}
