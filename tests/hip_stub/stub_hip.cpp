// A stand-in for the HIP runtime, for tests of the library's host code without
// a GPU: memory is host memory, copies happen at once, kernels are not run.
// Calls that order or launch work are logged; the tests set what a launch
// returns, whether streams are busy, and an error left by an earlier call.
// As in the HIP runtime, hipGetLastError returns and clears the last error of
// any call of the thread, and a call that succeeds leaves it alone.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

constexpr size_t kMigrateArgs = 48;
std::string g_log;
hipError_t g_pending = hipSuccess;    // what hipGetLastError would return
hipError_t g_launch = hipSuccess;     // status of the next launches
hipError_t g_record = hipSuccess;     // status of the next event records
hipError_t g_wait = hipSuccess;       // status of the next stream waits
bool g_busy = false;                  // streams and events have not finished
bool g_capturing = false;
int g_events = 0;
hipError_t g_copy = hipSuccess;       // status of the next asynchronous copies
std::vector<unsigned long long> g_copies;   // source, destination and bytes of each since stub_clear
unsigned char g_migrate[64];          // the arguments of the last migration kernel

// Kernel names by handle; built on first use, as the library's objects register theirs while it is loaded.
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> m;
  return m;
}

hipError_t done(hipError_t e) {
  if (e != hipSuccess && e != hipErrorNotReady) g_pending = e;
  return e;
}

template <class T>
void note(const char* what, T* on) {
  g_log += what;
  g_log += ' ';
  g_log += std::to_string((unsigned long long)(uintptr_t)on);
  g_log += '\n';
}

hipError_t launched(const void* f, void** args, hipStream_t s) {
  auto it = kernels().find(f);
  const std::string what = "launch " + (it == kernels().end() ? std::string("?") : it->second);
  note(what.c_str(), s);
  if (what.find("k_migrate") != std::string::npos) std::memcpy(g_migrate, args[0], kMigrateArgs);
  return done(g_launch);
}

hipError_t alloc(void** p, size_t n, const char* what) {
  if (n > (size_t)1 << 40) return done(hipErrorOutOfMemory);
  note(what, (void*)n);
  *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096 + 4096);
  if (!*p) return done(hipErrorOutOfMemory);
  std::memset(*p, 0, n);
  return hipSuccess;
}

}  // namespace

extern "C" {

// What the tests call.
const char* stub_log() { return g_log.c_str(); }
void stub_clear() {
  g_log.clear();
  g_copies.clear();
}
void stub_copy(int e) { g_copy = (hipError_t)e; }
int stub_copies(const unsigned long long** at) {
  *at = g_copies.data();
  return (int)(g_copies.size() / 3);
}
void stub_pending(int e) { g_pending = (hipError_t)e; }
int stub_peek() { return (int)g_pending; }
void stub_launch(int e) { g_launch = (hipError_t)e; }
void stub_record(int e) { g_record = (hipError_t)e; }
void stub_wait(int e) { g_wait = (hipError_t)e; }
void stub_busy(int b) { g_busy = b != 0; }
const void* stub_migrate_args() { return g_migrate; }
void stub_capturing(int c) { g_capturing = c != 0; }

// Registration of the compiled kernels and device variables.
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) {
  *g = dim3(1);
  *b = dim3(1);
  *l = 0;
  *s = nullptr;
  return hipSuccess;
}

hipError_t hipGetLastError() {
  const hipError_t e = g_pending;
  g_pending = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "stub error"; }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { return done(d == 0 ? hipSuccess : hipErrorInvalidDevice); }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { note("device_sync", (void*)nullptr); return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) { return alloc(p, n, "malloc"); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return alloc(p, n, "host_malloc"); }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  *base = p;
  *size = (size_t)1 << 40;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof(*a));
  a->type = hipMemoryTypeDevice;
  a->devicePointer = const_cast<void*>(p);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = aligned_alloc(4096, 1 << 20);
  *p = scratch;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  note("copy", st);
  g_copies.insert(g_copies.end(), {(unsigned long long)(uintptr_t)s, (unsigned long long)(uintptr_t)d, n});
  if (done(g_copy) == hipSuccess) std::memcpy(d, s, n);
  return g_copy;
}

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)(uintptr_t)(0x1000 + 16 * ++g_events);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return g_busy ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { note("record", s); return done(g_record); }
hipError_t hipEventSynchronize(hipEvent_t e) { note("event_sync", e); return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return g_busy ? hipErrorNotReady : hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { note("stream_sync", s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) { note("stream_wait", s); return done(g_wait); }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
  *c = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** a, size_t, hipStream_t s) { return launched(f, a, s); }
hipError_t hipExtLaunchKernel(const void* f, dim3, dim3, void** a, size_t, hipStream_t s, hipEvent_t, hipEvent_t,
                              int) {
  return launched(f, a, s);
}

}  // extern "C"
