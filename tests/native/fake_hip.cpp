// A HIP runtime for tests on the host: device memory is host memory under a
// capacity, kernel launches are counted and do nothing, and everything the
// library takes from the runtime is counted until it is given back.  A program
// that links this file and libdcg.so runs the library's set-up and scheduling
// (not its arithmetic) without a GPU.
#include "fake_hip.hpp"

#include <cstdlib>
#include <cstring>
#include <mutex>
#include <unordered_map>

namespace fake {

State& state() {
  static State s;
  return s;
}

namespace {
std::mutex mu;
// in functions: the library registers its kernels before this file's own
// constructors run
std::unordered_map<void*, size_t>& device_mem() {
  static std::unordered_map<void*, size_t> m;
  return m;
}
std::unordered_map<const void*, std::string>& kernel_name() {
  static std::unordered_map<const void*, std::string> m;
  return m;
}
std::map<std::string, int64_t>& launches() {
  static std::map<std::string, int64_t> m;
  return m;
}
thread_local hipError_t last = hipSuccess;

hipError_t ret(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}

void count_launch(const void* f) {
  std::lock_guard<std::mutex> lk(mu);
  ++launches()[kernel_name()[f]];
}
}  // namespace

int64_t live_bytes() {
  std::lock_guard<std::mutex> lk(mu);
  int64_t b = 0;
  for (const auto& kv : device_mem()) b += int64_t(kv.second);
  return b;
}

int64_t live_blocks(size_t size) {
  std::lock_guard<std::mutex> lk(mu);
  int64_t c = 0;
  for (const auto& kv : device_mem()) c += size == 0 || kv.second == size;
  return c;
}

int64_t launched(const std::string& name) {
  std::lock_guard<std::mutex> lk(mu);
  int64_t c = 0;
  for (const auto& kv : launches())
    if (kv.first.find(name) != std::string::npos) c += kv.second;
  return c;
}

}  // namespace fake

using namespace fake;

namespace {
// An object of the runtime other than device memory.
template <typename T>
hipError_t make(T* out) {
  ++state().objects;
  *out = reinterpret_cast<T>(std::malloc(1));
  return hipSuccess;
}
template <typename T>
hipError_t unmake(T o) {
  if (!o) return ret(hipErrorInvalidValue);
  --state().objects;
  std::free(reinterpret_cast<void*>(o));
  return hipSuccess;
}
}  // namespace

extern "C" {

hipError_t hipMalloc(void** p, size_t size) {
  State& s = state();
  const int64_t call = s.malloc_calls++;
  const int64_t used = live_bytes();
  *p = nullptr;
  if ((s.fail_call >= 0 && call == s.fail_call) || used + int64_t(size) > s.capacity)
    return ret(hipErrorOutOfMemory);
  *p = std::calloc(size ? size : 1, 1);
  if (!*p) return ret(hipErrorOutOfMemory);
  std::lock_guard<std::mutex> lk(mu);
  device_mem()[*p] = size;
  if (used + int64_t(size) > s.peak) s.peak = used + int64_t(size);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  std::lock_guard<std::mutex> lk(mu);
  if (!device_mem().erase(p)) {
    ++state().bad_frees;
    return ret(hipErrorInvalidValue);
  }
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t size, unsigned) {
  ++state().objects;
  *p = std::calloc(size ? size : 1, 1);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  if (p) --state().objects;
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *t = size_t(state().capacity);
  *f = size_t(state().capacity - live_bytes());
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  std::memcpy(d, s, n);
  if (k == hipMemcpyDeviceToHost && state().on_read) state().on_read(d, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  if (v) std::memset(d, v, n);   // memory starts cleared and no kernel writes it
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipGetDevice(int* d) {
  *d = state().device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  state().device = d;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = nullptr;
  return ret(hipErrorInvalidValue);
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return make(s); }
hipError_t hipStreamDestroy(hipStream_t s) { return unmake(s); }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return make(g); }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { return make(e); }
hipError_t hipGraphDestroy(hipGraph_t g) { return unmake(g); }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { return unmake(e); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return make(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return make(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return unmake(e); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  count_launch(f);
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t, hipEvent_t, hipEvent_t,
                              int) {
  count_launch(f);
  return hipSuccess;
}

// what the compiler's launch and registration code calls
struct LaunchConfig {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
};
static thread_local LaunchConfig config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
  config = {g, b, m, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = config.grid;
  *b = config.block;
  *m = config.shmem;
  *s = config.stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*,
                           dim3*, int*) {
  std::lock_guard<std::mutex> lk(mu);
  kernel_name()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"
