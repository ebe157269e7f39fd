// A HIP runtime on host memory for tests of the library's host paths without a
// device: allocations within a limit, copies, kernels that do nothing but for
// the few whose results the host acts on, grids checked against the limits of
// the device, and an operator new that fails on request.  Loaded globally
// before the library, whose references then bind here.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>

namespace {
std::mutex mu;
std::map<const void*, std::string>& names() { static auto* m = new std::map<const void*, std::string>; return *m; }
std::map<void*, size_t>& blocks() { static auto* m = new std::map<void*, size_t>; return *m; }
std::map<std::string, unsigned>& grids() { static auto* m = new std::map<std::string, unsigned>; return *m; }
size_t used = 0, peak = 0, limit = SIZE_MAX;
std::atomic<long> new_left{-1};   // operator new calls until one fails (-1: never)
thread_local bool inside = false;
struct Inside { bool was = inside; Inside() { inside = true; } ~Inside() { inside = was; } };
struct Call { dim3 grid, block; size_t shm; hipStream_t s; };
thread_local Call call;
char handle;
hipError_t run(const void* f, dim3 grid, dim3 block, void** a) {
  Inside in;
  if (grid.x == 0 || grid.y == 0 || grid.z == 0 || grid.y > 65535 || grid.z > 65535 ||
      block.x * block.y * block.z > 1024)
    return hipErrorInvalidConfiguration;
  std::lock_guard<std::mutex> hold(mu);
  const std::string& n = names()[f];
  grids()[n] = grid.x;
  auto is = [&](const char* k) { return n.find(k) != std::string::npos; };
  if (is("k_gj_invert_perm"))   // every record a permutation
    memset(*(int**)a[6], 0, 4 * (size_t)grid.x);
  else if (is("k_block_nonzero"))
    memset(*(uint8_t**)a[3], 1, (size_t)*(int64_t*)a[2]);
  else if (is("k_comp_flags"))   // the velocity components of no cell couple
    memset(*(uint8_t**)a[2], 3, (size_t)*(int*)a[3]);
  else if (is("k_interleave"))
    for (int64_t q = 0; q < *(int64_t*)a[3]; ++q) {
      (*(double**)a[2])[2 * q] = (*(double**)a[0])[q];
      (*(double**)a[2])[2 * q + 1] = (*(double**)a[1])[q];
    }
  return hipSuccess;
}
void* fresh(size_t n) {
  Inside in;
  std::lock_guard<std::mutex> hold(mu);
  if (n > limit - used) return nullptr;
  void* p = calloc(n ? n : 1, 1);
  if (!p) return nullptr;
  blocks()[p] = n;
  used += n;
  if (used > peak) peak = used;
  return p;
}
hipError_t drop(void* p) {
  Inside in;
  std::lock_guard<std::mutex> hold(mu);
  auto it = blocks().find(p);
  if (it == blocks().end()) return p ? hipErrorInvalidValue : hipSuccess;
  used -= it->second;
  blocks().erase(it);
  free(p);
  return hipSuccess;
}
}  // namespace

void* operator new(size_t n) {
  if (!inside && new_left.load() >= 0 && new_left.fetch_sub(1) == 0) throw std::bad_alloc();
  if (void* p = malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void* operator new[](size_t n) { return operator new(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
void operator delete[](void* p) noexcept { free(p); }
void operator delete[](void* p, size_t) noexcept { free(p); }

extern "C" {
void fake_limit(size_t n) { limit = n; }
size_t fake_used() { return used; }
size_t fake_peak(int reset) { if (reset) peak = used; return peak; }
void fake_fail_new(long n) { new_left = n; }
long fake_new_left() { return new_left; }
// the last grid of the kernels whose name holds the text (0: not launched)
unsigned fake_grid(const char* name) {
  unsigned g = 0;
  for (const auto& k : grids())
    if (k.first.find(name) != std::string::npos) g = k.second;
  return g;
}

void** __hipRegisterFatBinary(const void*) { static void* m; return &m; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, hipStream_t s) { call = {g, b, shm, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shm, hipStream_t* s) {
  *g = call.grid; *b = call.block; *shm = call.shm; *s = call.s;
  return hipSuccess;
}
thread_local hipError_t last = hipSuccess;
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t, hipStream_t) {
  const hipError_t e = run(f, g, b, a);
  if (e != hipSuccess) last = e;
  return e;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) {
  return hipLaunchKernel(f, g, b, a, 0, nullptr);
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = fresh(n);
  return *p ? hipSuccess : (last = hipErrorOutOfMemory);
}
hipError_t hipFree(void* p) { return drop(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n ? n : 1, 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { if (n) memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { if (n) memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { if (n) memset(d, v, n); return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) { memset(a, 0, sizeof(*a)); a->numRegs = 128; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static void* ws = calloc(size_t(64) << 20, 1); *p = ws; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)&handle; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)&handle; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0.0f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)&handle; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}
