// A HIP runtime of two devices that executes nothing, for host-side tests of libhgnn.so: memory is host memory, a launch only
// makes its stream busy and is written down, a wait makes it idle again.  Loaded before the library (RTLD_GLOBAL), its
// definitions are the ones the library finds.  It also stands in front of hgnn::dev_free and counts the blocks that are given
// back while work is in flight.
#define __HIP_PLATFORM_AMD__ 1
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <set>
#include <string>
#include <vector>

namespace {
constexpr int kDevices = 2;
thread_local int cur = 0;
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
std::map<const void*, std::string> names;
std::map<void*, int> live;             // allocation -> device
std::set<hipStream_t> busy[kDevices];  // streams with work in flight
std::vector<std::string> launched;
std::string launched_text;
size_t live_bytes = 0;
std::map<void*, size_t> sizes;
int mallocs = 0, frees = 0, freed_busy = 0, fail_at = -1, fail_waits = 0;
bool capturing = false, spoiled = false;
std::string library;
dim3 push_grid, push_block;
size_t push_shmem;
int last_grid = 0, last_block = 0;
hipStream_t push_stream;

// the test makes streams of device d as 0x1000 * (d + 1) + anything
int device_of(hipStream_t s) {
  const uintptr_t v = reinterpret_cast<uintptr_t>(s);
  return v == 0 ? cur : int(v / 0x1000) - 1;
}
void work(hipStream_t s) { busy[device_of(s)].insert(s); }
// a call that a capture in progress does not allow, in the relaxed mode or at all
bool refused(bool always = false) {
  if (!capturing || (mode == hipStreamCaptureModeRelaxed && !always)) return false;
  spoiled = true;
  return true;
}
}  // namespace

extern "C" {
// ---- what the test asks
int fake_last_grid() { return last_grid; }
int fake_last_block() { return last_block; }
void fake_reset(const char* lib) {
  library = lib;
  launched.clear();
  for (auto& b : busy) b.clear();
  mallocs = frees = freed_busy = fail_waits = 0;
  fail_at = -1;
  capturing = spoiled = false;
  cur = 0;
}
int fake_busy(int d) { return int(busy[d].size()); }
int fake_mallocs() { return mallocs; }
int fake_frees() { return frees; }
int fake_freed_busy() { return freed_busy; }
int fake_live() { return int(live.size()); }
size_t fake_live_bytes() { return live_bytes; }
int fake_spoiled() { return spoiled; }
void fake_capture(int on) { capturing = on != 0; }
void fake_fail_malloc(int n) { fail_at = n < 0 ? -1 : mallocs + n; }
void fake_fail_waits(int on) { fail_waits = on; }
const char* fake_launched() {  // kernels since the last reset, one a line
  launched_text.clear();
  for (const auto& n : launched) launched_text += n + "\n";
  return launched_text.c_str();
}

// ---- the runtime
hipError_t hipGetDevice(int* d) { *d = cur; return hipSuccess; }
hipError_t hipSetDevice(int d) {
  if (d < 0 || d >= kDevices) return hipErrorInvalidDevice;
  cur = d;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  const hipStreamCaptureMode old = mode;
  mode = *m;
  *m = old;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  if (refused(true)) return hipErrorStreamCaptureUnsupported;
  if (fail_waits) return hipErrorUnknown;
  busy[cur].clear();
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (fail_waits) return hipErrorUnknown;
  busy[device_of(s)].erase(s);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  if (mallocs++ == fail_at) return hipErrorInvalidValue;
  *p = calloc(n, 1);
  if (*p) live[*p] = cur, sizes[*p] = n, live_bytes += n;
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  ++frees;
  const auto it = live.find(p);
  if (it == live.end()) return hipErrorInvalidValue;
  if (fail_waits) return hipErrorUnknown;
  busy[it->second].clear();
  live.erase(it);
  live_bytes -= sizes[p];
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(n, 1);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  memcpy(d, s, n);
  work(st);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  memset(d, v, n);
  work(st);
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t s) {
  work(s);
  last_grid = int(grid.x), last_block = int(block.x);
  launched.push_back(names.count(f) ? names[f] : "?");
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "an error of the test's runtime"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : (a == hipDeviceAttributeL2CacheSize ? 4 << 20 : 64);
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950");
  p->warpSize = 64;
  p->multiProcessorCount = 256;
  p->maxThreadsPerBlock = 1024;
  p->maxThreadsPerMultiProcessor = 2048;
  return hipSuccess;
}
int hipGetStreamDeviceId(hipStream_t s) { return device_of(s); }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char* mem = static_cast<char*>(calloc(32 << 20, 1));
  *p = mem;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) {
  push_grid = g, push_block = b, push_shmem = sh, push_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* s) {
  *g = push_grid, *b = push_block, *sh = push_shmem, *s = push_stream;
  return hipSuccess;
}
}  // extern "C"

namespace hgnn {
__attribute__((visibility("default"))) void dev_free(const void* p) {
  static void (*real)(const void*) = nullptr;
  if (!real) real = reinterpret_cast<void (*)(const void*)>(dlsym(dlopen(library.c_str(), RTLD_NOLOAD | RTLD_LAZY), "_ZN4hgnn8dev_freeEPKv"));
  const auto it = live.find(const_cast<void*>(p));
  if (it != live.end() && !busy[it->second].empty()) ++freed_busy;
  real(p);
}
}  // namespace hgnn
