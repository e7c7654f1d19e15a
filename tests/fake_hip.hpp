// A stand-in for the HIP runtime, in host memory, for tests of the library's
// host code on a machine without a GPU: two devices, streams and events that
// belong to one, memory of the kinds the runtime tells apart.  Work is done at
// once.  Define FAKE_HIP_MAIN in the one file of a test program.
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>

namespace fake {

constexpr int kDevices = 2;
struct Stream { int dev; };
struct Event { int dev; };

inline thread_local int current = 0;                 // the thread's current device
inline std::mutex mu;
inline std::map<const void *, hipMemoryType> kinds;  // destinations that are not plain host memory
inline std::map<void *, int> pinned;                 // live pinned allocations
inline std::atomic<int> live_events{0}, copies{0}, foreign_per_thread{0}, failing_malloc{0};
inline std::thread::id owner = std::this_thread::get_id();
inline int copies_until_failure = -1;                // synchronous copies (< 0: none fails)
inline bool ended = false;                           // set at exit: no call may follow

inline void alive() {
  if (ended) {
    std::fprintf(stderr, "HIP call after the runtime's end\n");
    std::abort();
  }
}
inline hipStream_t stream(int dev) { return reinterpret_cast<hipStream_t>(new Stream{dev}); }
inline int device_of(hipStream_t s) {
  if (s == nullptr || s == hipStreamPerThread) return current;
  return reinterpret_cast<Stream *>(s)->dev;
}

}  // namespace fake

#ifdef FAKE_HIP_MAIN
extern "C" {
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetDevice(int *d) { fake::alive(); *d = fake::current; return hipSuccess; }
hipError_t hipSetDevice(int d) {
  fake::alive();
  if (d < 0 || d >= fake::kDevices) return hipErrorInvalidDevice;
  fake::current = d;
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d) { fake::alive(); *d = fake::device_of(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { fake::alive(); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  fake::alive();
  if (fake::failing_malloc) return hipErrorOutOfMemory;
  *p = std::malloc(n);
  std::lock_guard<std::mutex> l(fake::mu);
  fake::pinned[*p] = 1;
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  fake::alive();
  std::lock_guard<std::mutex> l(fake::mu);
  fake::pinned.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  fake::alive();
  *e = reinterpret_cast<hipEvent_t>(new fake::Event{fake::current});
  ++fake::live_events;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  fake::alive();
  delete reinterpret_cast<fake::Event *>(e);
  --fake::live_events;
  return hipSuccess;
}
// An event can be recorded on streams of its own device only.
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  fake::alive();
  return reinterpret_cast<fake::Event *>(e)->dev == fake::device_of(s) ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipEventSynchronize(hipEvent_t) { fake::alive(); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  fake::alive();
  std::memset(a, 0, sizeof(*a));
  std::lock_guard<std::mutex> l(fake::mu);
  const auto it = fake::kinds.find(p);
  a->type = it == fake::kinds.end() ? hipMemoryTypeUnregistered : it->second;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  fake::alive();
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  fake::alive();
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
  fake::alive();
  if (fake::copies_until_failure == 0) return hipErrorUnknown;
  if (fake::copies_until_failure > 0) --fake::copies_until_failure;
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t s) {
  fake::alive();
  ++fake::copies;
  // the per-thread stream of another thread is not ordered after the owner's work
  if (s == hipStreamPerThread && std::this_thread::get_id() != fake::owner) ++fake::foreign_per_thread;
  std::memcpy(dst, src, n);
  return hipSuccess;
}
}
#endif
