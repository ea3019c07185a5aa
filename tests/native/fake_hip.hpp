// A HIP runtime of host memory for programs that link libpotts.so: allocations
// and copies are the host's, streams and events are empty, kernels do nothing.
// The library's host code then runs without a GPU.  An allocation can be made to
// fail, and device-to-device copies and the bytes held are recorded.
#pragma once

#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <vector>

namespace fake {

struct Copy {
  const void *dst, *src;
  size_t bytes;
};

inline std::mutex mu;
inline std::map<void *, size_t> held;  // device memory
inline size_t now = 0, peak = 0;
inline long allocations = 0, fail_at = -1;  // hipMalloc number fail_at fails
inline bool fail_all = false;
inline long launches = 0, cooperative = 0, host_allocations = 0;
inline std::vector<Copy> device_copies, host_copies;

inline int alloc(void **p, size_t n) {
  std::lock_guard<std::mutex> lock(mu);
  *p = nullptr;
  if (allocations++ == fail_at || fail_all) return 2;  // hipErrorOutOfMemory
  *p = calloc(1, n ? n : 1);
  held[*p] = n;
  now += n;
  peak = now > peak ? now : peak;
  return 0;
}

inline int release(void *p) {
  std::lock_guard<std::mutex> lock(mu);
  auto it = held.find(p);
  if (it == held.end()) return 0;
  now -= it->second;
  held.erase(it);
  free(p);
  return 0;
}

inline int copy(void *dst, const void *src, size_t n, int kind) {
  std::lock_guard<std::mutex> lock(mu);
  if (kind == 3) device_copies.push_back({dst, src, n});
  if (kind == 2) host_copies.push_back({dst, src, n});
  memmove(dst, src, n);
  return 0;
}

inline char handle[64];

}  // namespace fake

extern "C" {
int hipMalloc(void **p, size_t n) { return fake::alloc(p, n); }
int hipMallocAsync(void **p, size_t n, void *) { return fake::alloc(p, n); }
int hipFree(void *p) { return fake::release(p); }
int hipFreeAsync(void *p, void *) { return fake::release(p); }
int hipHostMalloc(void **p, size_t n, unsigned) { return ++fake::host_allocations, (*p = calloc(1, n)) ? 0 : 2; }
int hipHostFree(void *p) { return free(p), 0; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { return fake::copy(d, s, n, kind); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *) { return fake::copy(d, s, n, kind); }
int hipMemsetAsync(void *d, int v, size_t n, void *) { return memset(d, v, n), 0; }
int hipGetDevice(int *d) { return *d = 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
int hipStreamGetDevice(void *, int *d) { return *d = 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "fake"; }
int hipGetSymbolAddress(void **p, const void *) { return *p = calloc(1, 1 << 20), 0; }
int hipStreamCreate(void **s) { return *s = fake::handle, 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return *s = fake::handle, 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamIsCapturing(void *, int *s) { return *s = 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { return *g = fake::handle, 0; }
int hipGraphInstantiate(void **e, void *, void *, char *, size_t) { return *e = fake::handle, 0; }
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipEventCreate(void **e) { return *e = fake::handle, 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return *e = fake::handle, 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { return *ms = 1.0f, 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { return *n = 1, 0; }
struct Dim {
  uint32_t x, y, z;
};
int hipLaunchKernel(const void *, Dim, Dim, void **, size_t, void *) { return ++fake::launches, 0; }
int hipLaunchCooperativeKernel(const void *, Dim, Dim, void **, unsigned, void *) { return ++fake::cooperative, 0; }
int __hipPushCallConfiguration(Dim, Dim, size_t, void *) { return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *lds, void **s) {
  *g = *b = Dim{1, 1, 1};
  *lds = 0;
  *s = nullptr;
  return 0;
}
void **__hipRegisterFatBinary(const void *) { return reinterpret_cast<void **>(fake::handle); }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}
