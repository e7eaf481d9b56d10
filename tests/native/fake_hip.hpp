// fake_hip.hpp -- the HIP runtime calls that libvsh makes, over host memory
// and without kernels (but the one that copies results out), for tests of the
// host code on machines without a GPU.
// An executable that includes this once and links libvsh.so answers the
// library's calls itself.  Copies and launches wait in a queue until something
// synchronises with them; a chosen call can be made to fail.
#pragma once

#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace fake {

// which of this thread's next allocations outside these calls fails (0: none)
inline thread_local int fail_new = 0;
struct Aside {
  const int was = fail_new;
  Aside() { fail_new = 0; }
  ~Aside() { fail_new = was; }
};

struct Launch {
  std::string kernel;
  uint32_t blocks, threads;
};

struct State {
  std::recursive_mutex mu;
  std::vector<std::function<void()>> queue;  // copies and launches in flight
  std::map<void*, size_t> dev, pinned;       // allocations
  size_t dev_bytes = 0, dev_limit = (size_t)64 << 30;
  int pinned_allocs = 0;
  int cus = 256;
  std::vector<Launch> launches;
  hipError_t last = hipSuccess;
  bool running = false;  // events are not reached while set
  std::map<std::string, int> fail;  // call -> which of its next calls fails (1: the next)
};
inline State& st() {
  static State* s = new State();
  return *s;
}
using Lock = std::lock_guard<std::recursive_mutex>;

inline hipError_t done(hipError_t e) {
  if (e != hipSuccess) st().last = e;
  return e;
}
inline bool told_to_fail(const char* call) {
  auto it = st().fail.find(call);
  if (it == st().fail.end() || --it->second > 0) return false;
  st().fail.erase(it);
  return true;
}
inline void drain() {
  for (auto& f : st().queue) f();
  st().queue.clear();
}
inline void* pages(size_t n, int kind) {
  void* p = mmap(nullptr, n, PROT_READ | PROT_WRITE, kind | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  return p == MAP_FAILED ? nullptr : p;
}
// a launch's configuration on its way to the kernel's host stub
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
};
inline Config& config() {
  static thread_local Config c;
  return c;
}
// the kernels by their host stubs
inline std::map<const void*, std::string>& kernels() {
  static auto* k = new std::map<const void*, std::string>();
  return *k;
}
inline hipError_t release(std::map<void*, size_t>& m, void* p, size_t* bytes) {
  if (!p) return hipSuccess;
  drain();
  auto it = m.find(p);
  if (it == m.end()) return done(hipErrorInvalidValue);
  munmap(p, it->second);
  if (bytes) *bytes -= it->second;
  m.erase(it);
  return hipSuccess;
}

}  // namespace fake

#define FAKE(call)                \
  fake::Aside fake_aside;         \
  fake::Lock fake_lock(fake::st().mu); \
  if (fake::told_to_fail(call)) return fake::done(hipErrorUnknown)

extern "C" {

hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  p->multiProcessorCount = fake::st().cus;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMemGetInfo(size_t* free, size_t* total) {
  *free = *total = (size_t)64 << 30;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* at = fake::pages((size_t)64 << 20, MAP_PRIVATE);
  *p = at;
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  fake::Lock l(fake::st().mu);
  const hipError_t e = fake::st().last;
  fake::st().last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }

hipError_t hipMalloc(void** p, size_t n) {
  FAKE("hipMalloc");
  *p = fake::st().dev_bytes + n > fake::st().dev_limit ? nullptr : fake::pages(n, MAP_PRIVATE);
  if (!*p) return fake::done(hipErrorOutOfMemory);
  fake::st().dev[*p] = n;
  fake::st().dev_bytes += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  FAKE("hipFree");
  return fake::release(fake::st().dev, p, &fake::st().dev_bytes);
}
// as the driver maps it: shared, and not given to forked children
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) {
  FAKE("hipHostMalloc");
  *p = fake::pages(n, MAP_SHARED);
  if (!*p) return fake::done(hipErrorOutOfMemory);
  madvise(*p, n, MADV_DONTFORK);
  fake::st().pinned[*p] = n;
  ++fake::st().pinned_allocs;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  FAKE("hipHostFree");
  return fake::release(fake::st().pinned, p, nullptr);
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) {
  FAKE("hipHostGetDevicePointer");
  *d = h;
  return hipSuccess;
}

hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) {
  FAKE("hipMemcpy");
  fake::drain();
  std::memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  FAKE("hipMemcpyAsync");
  fake::st().queue.push_back([=] { std::memcpy(to, from, n); });
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* to, int v, size_t n, hipStream_t) {
  FAKE("hipMemsetAsync");
  fake::st().queue.push_back([=] { std::memset(to, v, n); });
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  FAKE("hipLaunchKernel");
  fake::st().launches.push_back({fake::kernels()[f], grid.x, block.x});
  if (fake::kernels()[f].find("k_copy_out") != std::string::npos) {
    const uint64_t* from = *static_cast<const uint64_t**>(args[0]);
    uint64_t* to = *static_cast<uint64_t**>(args[1]);
    const uint32_t n = *static_cast<uint32_t*>(args[2]);
    fake::st().queue.push_back([=] { std::memcpy(to, from, n * 8ull); });
  } else {
    fake::st().queue.push_back([] {});
  }
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  fake::config() = {grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  const fake::Config& c = fake::config();
  *grid = c.grid;
  *block = c.block;
  *lds = c.lds;
  *s = c.stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* module = nullptr;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned int, void*, void*, dim3*, dim3*,
                           int*) {
  fake::kernels()[stub] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned int) {
  *s = reinterpret_cast<hipStream_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  FAKE("hipStreamSynchronize");
  fake::drain();
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) {
  FAKE("hipEventRecord");
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) {
  FAKE("hipEventSynchronize");
  fake::drain();
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) {
  FAKE("hipEventQuery");
  if (fake::st().running) return hipErrorNotReady;
  fake::drain();
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}

}  // extern "C"
