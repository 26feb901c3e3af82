// The HIP calls of libpsr.so's host code, without a device: a test loads this
// library first, so that the solver library's calls land here. Kernels are
// counted, not run; host memory, events and waits are counted, and each call
// can be told to fail.
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <new>

extern "C" {

struct State {
  int host_live, event_live;  // allocated and not freed
  int launches, pending;      // kernels enqueued, and since the last wait for the stream
  int device_syncs;
  int host_frees_unsynced;    // host blocks freed with work pending
  int fail_event_sync, fail_new, capturing;
  int64_t mesh_verts, mesh_tris;  // what the mesh totals read as
} host_hip;

enum { kOk = 0, kNoMemory = 2, kInvalid = 1, kCapture = 900 };

int hipGetDeviceCount(int* n) { return *n = 1, kOk; }
int hipGetDevice(int* d) { return *d = 0, kOk; }
int hipSetDevice(int) { return kOk; }
int hipGetLastError() { return kOk; }
int hipMalloc(void** p, size_t n) { return (*p = malloc(n)) ? kOk : kNoMemory; }
int hipFree(void* p) { return free(p), kOk; }
int hipMemcpy(void* d, const void* s, size_t n, int) { return memcpy(d, s, n), kOk; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { return memcpy(d, s, n), kOk; }
int hipGetSymbolAddress(void**, const void*) { return kInvalid; }

int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(1, n < 64 ? 64 : n);
  memcpy(*p, &host_hip.mesh_verts, 2 * sizeof(int64_t));  // the header starts with the totals
  return ++host_hip.host_live, kOk;
}
int hipHostFree(void* p) {
  host_hip.host_frees_unsynced += host_hip.pending != 0;
  return free(p), --host_hip.host_live, kOk;
}
int hipEventCreate(void** e) { return *e = malloc(1), ++host_hip.event_live, kOk; }
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) { return free(e), --host_hip.event_live, kOk; }
int hipEventRecord(void*, void*) { return kOk; }
int hipEventElapsedTime(float* t, void*, void*) { return *t = 0, kOk; }
int hipEventSynchronize(void*) { return host_hip.fail_event_sync || host_hip.capturing ? kCapture : kOk; }
int hipStreamSynchronize(void*) { return host_hip.capturing ? kCapture : (host_hip.pending = 0, kOk); }
int hipDeviceSynchronize() { return host_hip.pending = 0, ++host_hip.device_syncs, kOk; }
int hipStreamIsCapturing(void*, int* s) { return *s = host_hip.capturing, kOk; }

int hipLaunchKernel(const void*, ...) { return ++host_hip.launches, ++host_hip.pending, kOk; }
int __hipPushCallConfiguration(...) { return kOk; }
int __hipPopCallConfiguration(void* grid, void* block, size_t* shared, void** stream) {
  memset(grid, 0, 12);
  memset(block, 0, 12);
  return *shared = 0, *stream = nullptr, kOk;
}

}  // extern "C"

void* operator new(size_t n) {
  void* p = host_hip.fail_new ? nullptr : malloc(n);
  return p ? p : throw std::bad_alloc();
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return host_hip.fail_new ? nullptr : malloc(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
