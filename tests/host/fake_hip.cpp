// A stand-in for the HIP runtime, on the CPU: device memory is host memory,
// copies are copies, and a kernel launch is recorded and does nothing.  Linked
// with the library's host code (tests/test_host_code.py), it lets every call
// of the C ABI run without a GPU, with two devices, with a chosen call made to
// fail, and with what the library asked of the runtime open to the test.
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <string>
#include <vector>

struct ihipStream_t {
  int device;
  bool capturing;
};
struct ihipEvent_t {
  int unused;
};
struct ihipGraph {
  int unused;
};
struct hipGraphExec {
  int device;
};

namespace {
struct Launch {
  std::string name;
  dim3 grid, block;
  void *out;  // third argument of k_sum, where the drag goes
};
struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
};
thread_local int device = 0;
std::recursive_mutex mu;  // of the records
std::map<std::string, int> calls, fail_at;
// (kernels register before this file's own initialisers run)
std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> k;
  return k;
}
std::vector<Launch> launches;
thread_local std::vector<Config> configs;
thread_local hipError_t last = hipSuccess;
int wrong_device = 0;  // work given to a stream of another device
const double *watch = nullptr;
size_t watch_n = 0;
double watch_value = 0.0;
long watch_bad = 0;
int copying = 1;
alignas(256) char symbol[1 << 16];

// counts a call of the runtime; the chosen one fails
hipError_t call(const char *name) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  const int n = ++calls[name];
  auto f = fail_at.find(name);
  if (f != fail_at.end() && f->second == n) {
    fail_at.erase(f);
    return last = hipErrorOutOfMemory;
  }
  return hipSuccess;
}
void copy(void *dst, const void *src, size_t n, hipMemcpyKind kind) {
  if (kind == hipMemcpyDeviceToHost && dst == (const void *)watch)
    for (size_t k = 0; k < watch_n; k++) watch_bad += watch[k] != watch_value;
  if (copying) memcpy(dst, src, n);
}
}  // namespace

extern "C" {
// ---- what a test sets and reads ----
void fake_reset(void) {
  calls.clear();
  fail_at.clear();
  launches.clear();
  wrong_device = 0;
  watch = nullptr;
  watch_bad = 0;
  last = hipSuccess;
  device = 0;
  copying = 1;
}
void fake_fail(const char *name, int nth) { fail_at[name] = calls[name] + nth; }
// without copies and fills, device memory is not touched and large grids are cheap
void fake_copying(int on) { copying = on; }
int fake_calls(const char *name) { return calls[name]; }
int fake_wrong_device(void) { return wrong_device; }
int fake_launches(void) { return (int)launches.size(); }
const char *fake_launch(int k, unsigned grid[3], void **out) {
  const Launch &l = launches[k];
  grid[0] = l.grid.x, grid[1] = l.grid.y, grid[2] = l.grid.z;
  *out = l.out;
  return l.name.c_str();
}
// the values of a host array must be `value` until a copy replaces them
void fake_watch(const double *p, size_t n, double value) {
  watch = p, watch_n = n, watch_value = value, watch_bad = 0;
}
long fake_watch_bad(void) { return watch_bad; }

// ---- the runtime ----
hipError_t hipGetDevice(int *d) { return *d = device, hipSuccess; }
hipError_t hipSetDevice(int d) { return device = d, hipSuccess; }
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipMalloc(void **p, size_t n) {
  if (call("hipMalloc") != hipSuccess) return last;
  *p = aligned_alloc(256, (n + 255) / 256 * 256);
  return copying ? (memset(*p, 0, n), hipSuccess) : hipSuccess;
}
hipError_t hipFree(void *p) { return free(p), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  if (call("hipHostMalloc") != hipSuccess) return last;
  return *p = calloc(1, n), hipSuccess;
}
hipError_t hipHostFree(void *p) { return free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
  return call("hipMemcpy") != hipSuccess ? last : (copy(d, s, n, k), hipSuccess);
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) {
  return call("hipMemcpyAsync") != hipSuccess ? last : (copy(d, s, n, k), hipSuccess);
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h,
                            hipMemcpyKind, hipStream_t) {
  if (call("hipMemcpy2DAsync") != hipSuccess) return last;
  for (size_t j = 0; copying && j < h; j++) memcpy((char *)d + j * dp, (const char *)s + j * sp, w);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
  if (call("hipMemsetAsync") != hipSuccess) return last;
  return copying ? (memset(d, v, n), hipSuccess) : hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
  return a->type = hipMemoryTypeUnregistered, hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = symbol, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  if (call("hipStreamCreate") != hipSuccess) return last;
  return *s = new ihipStream_t{device, false}, hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t *s) { return hipStreamCreateWithFlags(s, 0); }
hipError_t hipStreamDestroy(hipStream_t s) {
  call("hipStreamDestroy");
  return delete s, hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return call("hipStreamSynchronize"); }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
  *st = s->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  if (call("hipStreamBeginCapture") != hipSuccess) return last;
  return s->capturing = true, hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
  s->capturing = false;
  return *g = new ihipGraph(), hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  if (call("hipGraphInstantiate") != hipSuccess) return last;
  return *e = new hipGraphExec{device}, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return delete g, hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  call("hipGraphExecDestroy");
  return delete e, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  wrong_device += e->device != s->device;
  return call("hipGraphLaunch");
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = new ihipEvent_t(), hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = new ihipEvent_t(), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return delete e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return call("hipEventRecord"); }
hipError_t hipEventSynchronize(hipEvent_t) { return call("hipEventSynchronize"); }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { return *t = 0.0f, hipSuccess; }

// ---- launches ----
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  Launch l{kernels()[f], grid, block, nullptr};
  if (l.name.find("k_sum") != std::string::npos) l.out = *(void **)args[2];
  launches.push_back(l);
  return call("hipLaunchKernel");
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  return configs.push_back({grid, block, shared, s}), hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid, *block = c.block, *shared = c.shared, *s = c.stream;
  return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *,
                           void *, void *, int *) {
  kernels()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
}
