// A HIP runtime that runs nothing: memory is host memory, copies are made at
// once, and every launch, event and stream call is written to a log.  Loaded
// ahead of libccut.so (tests/_hosthip.py) it shows what the library enqueues,
// in what order and on which streams, without a GPU.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::string g_log;
std::map<const void *, std::string> g_kernels;
long g_ids = 0;
const char *g_fail = "";  // allocations by this name fail
std::string g_copied;     // what the last hipMemcpy copied (a plan's programs)
struct {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
} g_config;

void *new_id() { return (void *)(++g_ids); }
template <class... A>
void put(const char *format, A... a) {
  char line[512];
  std::snprintf(line, sizeof(line), format, a...);
  g_log += line;
  g_log += '\n';
}
hipError_t allocate(const char *name, void **p, size_t n) {
  if (!std::strcmp(name, g_fail)) return hipErrorOutOfMemory;
  put("%s %zu", name, n);
  *p = std::calloc(n ? n : 1, 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
std::string fail_name;
}  // namespace

extern "C" {
const char *host_hip_log() { return g_log.c_str(); }
void host_hip_clear() { g_log.clear(); }
const char *host_hip_copied(size_t *n) { return *n = g_copied.size(), g_copied.data(); }
void host_hip_fail(const char *name) {
  fail_name = name;
  g_fail = fail_name.c_str();
}

void **__hipRegisterFatBinary(const void *) { return (void **)new_id(); }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
  g_kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
  g_config = {grid, block, shmem, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *stream) {
  *grid = g_config.grid;
  *block = g_config.block;
  *shmem = g_config.shmem;
  *stream = g_config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t, hipStream_t stream) {
  put("launch %p %s %u %u", (void *)stream, g_kernels[f].c_str(), grid.x, block.x);
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return allocate("hipMalloc", p, n); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return allocate("hipHostMalloc", p, n); }
hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  g_copied.assign((const char *)s, n);
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t stream) {
  put("copy %p %zu", (void *)stream, n);
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t stream) {
  put("memset %p %zu", (void *)stream, n);
  return std::memset(d, v, n), hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)new_id(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return put("sync %p", (void *)s), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  return put("wait %p %p", (void *)s, (void *)e), hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { return put("begin %p", (void *)s), hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
  put("end %p", (void *)s);
  return *g = (hipGraph_t)new_id(), hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
  return *st = hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t)new_id();
  return put("instantiate %p", (void *)*x), hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) { return put("replay %p", (void *)x), hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return put("drop %p", (void *)x), hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)new_id(), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return put("record %p %p", (void *)s, (void *)e), hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return put("waited %p", (void *)e), hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { return std::memset(p, 0, sizeof(*p)), hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static char buffer[1 << 12];
  return *p = buffer, hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
}
