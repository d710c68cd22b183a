// A HIP runtime of plain host memory for tests of the library's host paths on a machine without a GPU:
// "device" memory is host memory, copies are made at once and kernels are only written down (the table copy
// k_stage runs, so that later launches' descriptor tables can be read).  Loaded with global visibility
// before libblb.so, whose HIP calls then bind to it.  The stub_* functions set limits and failures.
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <condition_variable>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

namespace {
long new_countdown = 0;  // > 0: that many-th operator new from now, outside this file, throws
thread_local int inside = 0;
struct Inside {
  Inside() { ++inside; }
  ~Inside() { --inside; }
};
std::recursive_mutex mu;
size_t total_bytes = size_t(288) << 30;
int meet = 0, met = 0;  // device waits that return together
std::map<void*, size_t> live;  // device allocations
size_t live_bytes = 0, peak_bytes = 0, cap_bytes = 0;
int fail_copies = 0, fail_device_syncs = 0;
std::condition_variable_any together;
thread_local hipError_t last = hipSuccess;
size_t largest_host = 0;
unsigned largest_host_flags = 0;
std::map<const void*, std::string> kernels;
struct Launch {
  std::string name;
  unsigned grid;
  unsigned char arg0[64];  // the first argument's bytes
};
std::vector<Launch> launches;
std::vector<std::string> events;  // launches, copies and waits in order
struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
};
thread_local std::vector<Config> configs;
intptr_t handles = 0x1000;

hipError_t done(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
void* map_bytes(size_t n) {
  void* p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  return p == MAP_FAILED ? nullptr : p;
}
hipError_t take(void** p, size_t n) {
  Inside quiet;
  std::lock_guard<std::recursive_mutex> lk(mu);
  if (cap_bytes && live_bytes + n > cap_bytes) return done(hipErrorOutOfMemory);
  if (!(*p = map_bytes(n))) return done(hipErrorOutOfMemory);
  live[*p] = n;
  live_bytes += n;
  if (live_bytes > peak_bytes) peak_bytes = live_bytes;
  return hipSuccess;
}
hipError_t give(void* p) {
  if (!p) return hipSuccess;
  std::lock_guard<std::recursive_mutex> lk(mu);
  const auto it = live.find(p);
  if (it == live.end()) return done(hipErrorInvalidValue);
  live_bytes -= it->second;
  munmap(p, it->second);
  live.erase(it);
  return hipSuccess;
}
hipError_t copy(void* d, const void* s, size_t n) {
  if (fail_copies > 0) {
    --fail_copies;
    return done(hipErrorUnknown);
  }
  memcpy(d, s, n);
  return hipSuccess;
}
template <class T>
hipError_t handle(T* h) {
  *h = (T)(handles += 16);
  return hipSuccess;
}
}  // namespace

void* operator new(size_t n) {
  if (!inside && new_countdown > 0 && --new_countdown == 0) throw std::bad_alloc();
  void* p = malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {
size_t stub_live() { return live_bytes; }
size_t stub_peak(int reset) {
  const size_t p = peak_bytes;
  if (reset) peak_bytes = live_bytes;
  return p;
}
void stub_cap(size_t bytes) { cap_bytes = bytes; }
void stub_total(size_t bytes) { total_bytes = bytes; }
void stub_meet(int n) { meet = n, met = 0; }
void stub_fail_copies(int n) { fail_copies = n; }
void stub_fail_device_syncs(int n) { fail_device_syncs = n; }
void stub_fail_new(long n) { new_countdown = n; }
unsigned stub_host_flags() { return largest_host_flags; }  // of the largest pinned allocation
int stub_last_error() { return (int)last; }
void stub_clear() {
  launches.clear();
  events.clear();
}
int stub_launches() { return (int)launches.size(); }
const char* stub_launch_name(int i) { return launches[i].name.c_str(); }
unsigned stub_launch_grid(int i) { return launches[i].grid; }
const void* stub_launch_arg0(int i) { return launches[i].arg0; }
int stub_events() { return (int)events.size(); }
const char* stub_event(int i) { return events[i].c_str(); }

void** __hipRegisterFatBinary(const void*) {
  static void* module = nullptr;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  Inside quiet;
  configs.push_back(Config{g, b, s, st});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  const Config c = configs.back();
  configs.pop_back();
  *g = c.grid;
  *b = c.block;
  *s = c.shared;
  *st = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
  Inside quiet;
  std::lock_guard<std::recursive_mutex> lk(mu);
  Launch l{kernels[f], grid.x, {}};
  if (l.name.find("k_stage") != std::string::npos) {
    memcpy(*(void**)args[0], *(void**)args[1], (size_t) * (unsigned*)args[2] * 16);
  } else {
    memcpy(l.arg0, args[0], sizeof(l.arg0));
  }
  events.push_back("launch " + l.name);
  launches.push_back(l);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return take(p, n); }
hipError_t hipFree(void* p) { return give(p); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return take(p, n); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return give(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) {
  if (n > largest_host) largest_host = n, largest_host_flags = flags;
  return (*p = malloc(n)) ? hipSuccess : done(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return copy(d, s, n); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  Inside quiet;
  std::lock_guard<std::recursive_mutex> lk(mu);
  events.push_back("copy");
  return copy(d, s, n);
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemcpyToSymbol(const void*, const void*, size_t, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = map_bytes(size_t(64) << 20);
  *p = scratch;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  p->totalGlobalMem = total_bytes;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  Inside quiet;
  std::unique_lock<std::recursive_mutex> lk(mu);
  events.push_back("wait device");
  if (meet) {
    const int target = (met / meet + 1) * meet;
    ++met;
    together.notify_all();
    together.wait(lk, [&] { return met >= target; });
  }
  if (fail_device_syncs > 0) {
    --fail_device_syncs;
    return done(hipErrorStreamCaptureUnsupported);
  }
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  Inside quiet;
  std::lock_guard<std::recursive_mutex> lk(mu);
  events.push_back("wait stream");
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return handle(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return handle(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return handle(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t* p, int) { return handle(p); }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return handle(g); }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { return handle(e); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}
