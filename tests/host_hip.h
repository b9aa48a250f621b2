// A stand-in for the HIP runtime below the library's host code (csrc/fira.hip, included by the programs before this file): device
// memory is host memory, copies happen at once, kernels do nothing, everything that would be enqueued is counted, the stream
// is "captured" while `capturing` is set, every launch is handed to `on_launch`, the flags that events and host memory are made
// with are kept, and uploads, launches or the records of one event fail while they are told to.
#pragma once
#include <cstdlib>
#include <map>

namespace {
bool capturing = false;
void (*on_launch)(const void* kernel, dim3 grid, void** args) = nullptr;
long enqueued = 0;      // kernels, copies, fills and event records
int failures = 0;
#define CHECK(cond)                                                                       \
  do {                                                                                    \
    if (!(cond)) { ++failures; std::printf("FAIL line %d: %s\n", __LINE__, #cond); }      \
  } while (0)
alignas(256) char static_area[256];
std::map<const void*, unsigned> made_with;      // flags of an event or of host memory
bool uploads_fail = false, launches_fail = false;
const void* failing_event = nullptr;
}  // namespace

extern "C" {
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return capturing ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) {
  *e = (hipEvent_t)std::malloc(1);
  made_with[*e] = flags;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  if (e && e == failing_event) return hipErrorUnknown;
  ++enqueued;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetLastError(void) { return launches_fail ? hipErrorLaunchFailure : hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = static_area; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) {
  *p = std::malloc(n);
  made_with[*p] = flags;
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
  if (launches_fail) return hipErrorLaunchFailure;
  ++enqueued;
  if (on_launch) on_launch(f, grid, args);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
// (copies into the static scratch's stand-in are counted only: it is not the real size)
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (uploads_fail) return hipErrorUnknown;
  ++enqueued;
  if (d != static_area) std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t) {
  ++enqueued;
  for (size_t i = 0; i < h; ++i) std::memcpy((char*)d + i * dp, (const char*)s + i * sp, w);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { ++enqueued; std::memset(d, v, n); return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { static void* h = nullptr; return &h; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
}
