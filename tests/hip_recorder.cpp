// Host stand-in for the HIP calls of state transfers, loaded before the library
// so that its calls resolve here: device memory is host memory, kernels do
// nothing, allocations and copies are recorded with the current device.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <vector>

namespace {
struct Event {
  int kind, device;  // kind 0: allocation, 1: copy
  uint64_t to, from, bytes;
};
std::vector<Event> events;
int current = 0;
int refuse = 0;  // allocations fail
uint64_t ws_lo = 0, ws_hi = 0;
int ws_device = 0;
}  // namespace

extern "C" {
void rec_workspace(uint64_t lo, uint64_t bytes, int device) {
  ws_lo = lo;
  ws_hi = lo + bytes;
  ws_device = device;
}
void rec_refuse(int on) { refuse = on; }
void rec_clear() { events.clear(); }
int rec_current() { return current; }
uint64_t rec_count() { return events.size(); }
void rec_event(uint64_t i, uint64_t* out) {
  const Event& e = events[i];
  out[0] = (uint64_t)e.kind;
  out[1] = (uint64_t)e.device;
  out[2] = e.to;
  out[3] = e.from;
  out[4] = e.bytes;
}

hipError_t hipGetDevice(int* d) {
  *d = current;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  current = d;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  if ((uint64_t)p < ws_lo || (uint64_t)p >= ws_hi) return hipErrorInvalidValue;
  memset(a, 0, sizeof *a);
  a->device = ws_device;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  if (refuse) return hipErrorOutOfMemory;
  *p = calloc(1, n);
  events.push_back({0, current, (uint64_t)*p, 0, n});
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  events.push_back({1, current, (uint64_t)to, (uint64_t)from, n});
  memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 4;
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = *b = dim3();
  *m = 0;
  *s = nullptr;
  return hipSuccess;
}
}
