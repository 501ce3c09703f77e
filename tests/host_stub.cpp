// A HIP runtime of host memory and launchers that compute nothing, for CPU tests of the host runtime (pb_host.cpp):
// "device" memory is the process's own, copies are copies, launches are counted.  What a test wants to happen (a refused
// thread, a smaller GPU) and what it wants to know is in `stub`, read and written through stub_get / stub_set.
#include <dlfcn.h>
#include <pthread.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <string>

#include "pb_device.h"
#include "pb_mlp.h"

namespace {
struct Stub {
  std::atomic<long> cus{256}, threads_refused{0}, pinned_refused{0}, masked{0};
  std::atomic<long> mlp_launches{0}, mlp_ticks_max{0}, fused_launches{0}, plain_launches{0}, waits{0}, device_syncs{0};
} stub;
std::atomic<long>* field(const char* name) {
  const std::string n = name;
  return n == "cus" ? &stub.cus : n == "threads_refused" ? &stub.threads_refused : n == "pinned_refused" ? &stub.pinned_refused : n == "masked" ? &stub.masked : n == "mlp_launches" ? &stub.mlp_launches
       : n == "mlp_ticks_max" ? &stub.mlp_ticks_max : n == "fused_launches" ? &stub.fused_launches
       : n == "plain_launches" ? &stub.plain_launches : n == "waits" ? &stub.waits : n == "device_syncs" ? &stub.device_syncs : nullptr;
}
}  // namespace

extern "C" {
long stub_get(const char* name) { return field(name)->load(); }
void stub_set(const char* name, long v) { field(name)->store(v); }

int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* arg) {
  if (stub.threads_refused > 0) { --stub.threads_refused; return EAGAIN; }
  static auto real = (int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*))dlsym(RTLD_NEXT, "pthread_create");
  return real(t, a, f, arg);
}

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = (int)stub.cus; return hipSuccess; }
hipError_t hipExtStreamGetCUMask(hipStream_t, uint32_t n, uint32_t* m) {
  if (!stub.masked) return hipErrorInvalidValue;
  for (uint32_t i = 0; i < n; ++i) m[i] = 32 * i < (uint32_t)stub.masked ? ~0u : 0u;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { ++stub.device_syncs; return hipSuccess; }
hipError_t hipDeviceGetPCIBusId(char* id, int n, int) {
  const char* name = getenv("STUB_GPU");
  if (!name) return hipErrorInvalidValue;
  strncpy(id, name, n);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return stub.pinned_refused ? hipErrorOutOfMemory : hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++stub.waits; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)&stub; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
}

namespace pb {
void launch_mlp(const MlpArgs& a, int, int, int, bool, hipStream_t) {
  ++stub.mlp_launches;
  if (a.n_ticks > stub.mlp_ticks_max) stub.mlp_ticks_max = a.n_ticks;
}
void launch_mlp_flush(const MlpRec*, int, int, int, hipStream_t) {}
void launch_phase(const StepDesc*, int, const Globals*, int, const float*, int, bool, hipStream_t, int32_t* sync, uint32_t) {
  ++(sync ? stub.fused_launches : stub.plain_launches);
}
void launch_copy_out(float* dst, const float* src, int64_t n, const int32_t* err, int32_t* err_out, hipStream_t) {
  memcpy(dst, src, sizeof(float) * n);
  if (err) *err_out = *err;
}
void launch_natural(float* dst, const float* src, const NatTable& t, hipStream_t) {
  for (int i = 0; i < t.n; ++i) {   // (the order of F_W_PERM, its dimensions from the outermost in)
    const int C = t.l[i].C, K = t.l[i].K;
    const float* p = src + t.l[i].off;
    for (int cb = 0; cb < C / 16; ++cb)
      for (int kb = 0; kb < K / 32; ++kb)
        for (int tap = 0; tap < 9; ++tap)
          for (int kh = 0; kh < 2; ++kh)
            for (int kq = 0; kq < 4; ++kq)
              for (int c = 0; c < 16; ++c)
                for (int e = 0; e < 4; ++e) dst[t.l[i].off + ((size_t)(32 * kb + 16 * kh + 4 * e + kq) * C + 16 * cb + c) * 9 + tap] = *p++;
  }
}
void launch_fill_zero(void* p, size_t bytes, hipStream_t) { memset(p, 0, bytes); }
void launch_set_globals(Globals* g, Globals v, hipStream_t) { *g = v; }
void launch_update_flat(float*, float*, const float*, float*, int64_t, float, float, float, float, float, hipStream_t) {}
hipError_t static_arena(void** p, int* dev) {
  static void* a = aligned_alloc(256, STATIC_ARENA_BYTES);
  *p = a; *dev = 0;
  return hipSuccess;
}
}  // namespace pb
