// A HIP runtime without a GPU, for tests of librh's host side: device memory is
// the host's, kernels are checked and not run, streams and graphs do nothing.
// Loaded before librh (global symbols), it stands in for the real runtime.
// It counts device memory and refuses what a test tells it to, and refuses a
// launch whose dynamic LDS is above the bound its kernel was last given.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>

namespace {

std::recursive_mutex mu;
std::map<void *, size_t> live;
size_t live_bytes = 0, peak_bytes = 0;
bool busy = false;
int64_t n_allocs = 0, n_launches = 0, n_streams = 0, max_bytes = -1, max_one = -1;
std::map<const void *, size_t> bound;
std::map<void *, int64_t> waits;
std::map<std::string, int> refuse;  // calls to let through before one is refused (memory: an allocation, for lack of it)
hipError_t last = hipSuccess;
constexpr size_t kDefaultLds = 64 * 1024, kLds = 160 * 1024;
char symbol[(size_t)128 << 20];

hipError_t done(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
bool refused(const char *name) {
  auto it = refuse.find(name);
  if (it == refuse.end()) return false;
  if (it->second-- > 0) return false;
  refuse.erase(it);
  return true;
}
hipError_t alloc(void **p, size_t n) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if ((max_bytes >= 0 && live_bytes + n > (size_t)max_bytes) || (max_one >= 0 && n > (size_t)max_one) || refused("memory"))
    return done(hipErrorOutOfMemory);
  if (refused("hipMalloc")) return done(hipErrorInvalidValue);
  *p = std::calloc(1, n ? n : 1);
  live[*p] = n;
  live_bytes += n;
  if (live_bytes > peak_bytes) peak_bytes = live_bytes;
  ++n_allocs;
  return hipSuccess;
}
hipError_t release(void *p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  auto it = live.find(p);
  if (it == live.end()) return p ? done(hipErrorInvalidValue) : hipSuccess;
  live_bytes -= it->second;
  live.erase(it);
  std::free(p);
  return hipSuccess;
}

}  // namespace

extern "C" {

// ---- what a test sets and reads
void fake_limit(int64_t all, int64_t one) { max_bytes = all, max_one = one; }
void fake_refuse(const char *name, int after) { refuse[name] = after; }
int64_t fake_live() { return (int64_t)live_bytes; }
int64_t fake_peak() { return (int64_t)peak_bytes; }
void fake_peak_reset() { peak_bytes = live_bytes; }
int64_t fake_allocs() { return n_allocs; }
int64_t fake_launches() { return n_launches; }
int64_t fake_streams() { return n_streams; }
void fake_busy(int all) { busy = all != 0; }  // whether work on a stream is under way
int64_t fake_waits(void *stream) { return waits[stream]; }

// ---- the runtime
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeWallClockRate ? 100000 : (int)kLds;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->name, "none");
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  std::lock_guard<std::recursive_mutex> l(mu);
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "refused"; }
hipError_t hipMalloc(void **p, size_t n) { return alloc(p, n); }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return *p = std::calloc(1, n ? n : 1), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (refused("hipMemcpy")) return done(hipErrorInvalidValue);
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) {
  if (refused("hipMemcpyAsync")) throw std::bad_alloc();  // (as a vector of the library's own would)
  return hipMemcpy(d, s, n, k);
}
hipError_t hipMemcpy2D(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind) {
  for (size_t i = 0; i < h; ++i) std::memcpy((char *)d + i * dp, (const char *)s + i * sp, w);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = symbol, hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) { return std::memset(a, 0, sizeof *a), hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (refused("hipFuncSetAttribute") || (size_t)v > kLds) return done(hipErrorInvalidValue);
  return bound[f] = (size_t)v, hipSuccess;
}
struct Call {
  dim3 g, b;
  size_t lds;
  hipStream_t s;
};
static thread_local Call call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  return call = Call{g, b, lds, s}, hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
  return *g = call.g, *b = call.b, *lds = call.lds, *s = call.s, hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t) {
  std::lock_guard<std::recursive_mutex> l(mu);
  auto it = bound.find(f);
  const size_t most = it == bound.end() ? kDefaultLds : it->second > kDefaultLds ? it->second : kDefaultLds;
  if (g.x == 0 || g.y == 0 || b.x == 0 || b.x * b.y * b.z > 1024 || lds > most) return done(hipErrorInvalidValue);
  ++n_launches;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (refused("hipStreamCreateWithFlags")) return done(hipErrorInvalidValue);
  return ++n_streams, *s = (hipStream_t)std::malloc(1), hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return std::free((void *)s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  return ++waits[(void *)s], hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return *g = (hipGraph_t)std::malloc(1), hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  return *e = (hipGraphExec_t)std::malloc(1), hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { return std::free((void *)g), hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { return std::free((void *)e), hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)std::malloc(1), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free((void *)e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return busy ? done(hipErrorNotReady) : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { return *s = hipStreamCaptureStatusNone, hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }

}  // extern "C"
