// A HIP runtime on host memory, for host-side tests of the library: defined in
// the test's executable, these functions are found before libamdhip64's.
// Kernels do nothing.  Copies and fills run when something waits for them (an
// event or a stream), in order, so that data taken too early is seen to be old.
// Two devices; streams 0x1000 + 256 k + d and what is created under device d belong to
// device d.
#pragma once
#include <hip/hip_runtime_api.h>

#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <utility>
#include <vector>

namespace fake {

struct Event {
  int device;
  long long at = 0;        // operations of its stream before it
  hipStream_t stream = nullptr;
};
struct Stream {
  std::deque<std::function<void()>> todo;
  long long issued = 0, done = 0;
};

inline std::mutex mu;
inline thread_local int current = 0;           // the current device
inline thread_local hipError_t last = hipSuccess;   // what hipGetLastError gives
inline int refuse_malloc = 0;                  // refuse this many pinned allocations
inline int fail_copy = 0;                      // this many copies to the host from now, one fails
inline int refuse_launch = 0;                  // refuse this many launches
inline bool unknown_stream = false;            // hipStreamGetDevice refuses
inline int wait_us = 0;                        // what waiting for an event takes
inline std::map<hipStream_t, Stream> streams;
inline std::set<Event*> events;
inline std::map<char*, size_t> pinned;         // live pinned allocations
inline std::set<const void*> user_pinned;      // test buffers to be taken as pinned
inline long long mallocs = 0, frees = 0;
inline std::vector<std::pair<char*, size_t>> d2h;   // targets of copies to the host

inline hipStream_t stream_of(int device, int k = 0) { return (hipStream_t)(uintptr_t)(0x1000 + 256 * k + device); }
inline int device_of(hipStream_t s) { return (uintptr_t)s > 2 ? (int)((uintptr_t)s & 0xff) : current; }
inline hipError_t err(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
inline void run(Stream& q, long long to) {
  while (q.done < to) {
    q.todo.front()();
    q.todo.pop_front();
    ++q.done;
  }
}
inline void issue(hipStream_t s, std::function<void()> f) {
  std::lock_guard<std::mutex> l(mu);
  Stream& q = streams[s];
  q.todo.push_back(std::move(f));
  ++q.issued;
}
inline bool in_pinned(const void* p) {
  for (auto& a : pinned)
    if ((const char*)p >= a.first && (const char*)p < a.first + a.second) return true;
  return false;
}

}  // namespace fake

#define FAKE extern "C" __attribute__((visibility("default"), used))

FAKE hipError_t hipGetDevice(int* d) { *d = fake::current; return hipSuccess; }
FAKE hipError_t hipSetDevice(int d) {
  if (d < 0 || d > 1) return fake::err(hipErrorInvalidDevice);
  fake::current = d;
  return hipSuccess;
}
FAKE hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) {
  if ((uintptr_t)s < 2) std::abort();   // as the real one does on hipStreamLegacy
  if (fake::unknown_stream) return fake::err(hipErrorInvalidHandle);
  *d = fake::device_of(s);
  return hipSuccess;
}
FAKE hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
FAKE hipError_t hipGetLastError() {
  const hipError_t e = fake::last;
  fake::last = hipSuccess;
  return e;
}
FAKE hipError_t hipGetSymbolAddress(void** p, const void*) {
  static std::vector<char> mem(64u << 20);
  *p = mem.data();
  return hipSuccess;
}
FAKE hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  std::lock_guard<std::mutex> l(fake::mu);
  if (fake::refuse_malloc > 0) {
    --fake::refuse_malloc;
    return fake::err(hipErrorOutOfMemory);
  }
  *p = std::malloc(n);
  fake::pinned[(char*)*p] = n;
  ++fake::mallocs;
  return hipSuccess;
}
// (the real one waits until every stream of the device is idle)
FAKE hipError_t hipHostFree(void* p) {
  std::lock_guard<std::mutex> l(fake::mu);
  if (p == nullptr) return hipSuccess;
  if (fake::pinned.erase((char*)p) == 0) return fake::err(hipErrorInvalidValue);
  std::free(p);
  ++fake::frees;
  return hipSuccess;
}
FAKE hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::lock_guard<std::mutex> l(fake::mu);
  std::memset(a, 0, sizeof(*a));
  a->type = fake::user_pinned.count(p) || fake::in_pinned(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
  return hipSuccess;
}
FAKE hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  std::lock_guard<std::mutex> l(fake::mu);
  auto* v = new fake::Event{fake::current};
  fake::events.insert(v);
  *e = (hipEvent_t)v;
  return hipSuccess;
}
FAKE hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
FAKE hipError_t hipEventDestroy(hipEvent_t e) {
  std::lock_guard<std::mutex> l(fake::mu);
  auto* v = (fake::Event*)e;
  if (fake::events.erase(v) == 0) return fake::err(hipErrorInvalidHandle);
  delete v;
  return hipSuccess;
}
FAKE hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  std::lock_guard<std::mutex> l(fake::mu);
  auto* v = (fake::Event*)e;
  if (v->device != fake::device_of(s)) return fake::err(hipErrorInvalidHandle);
  v->stream = s;
  v->at = fake::streams[s].issued;
  return hipSuccess;
}
FAKE hipError_t hipEventSynchronize(hipEvent_t e) {
  if (fake::wait_us) std::this_thread::sleep_for(std::chrono::microseconds(fake::wait_us));
  std::lock_guard<std::mutex> l(fake::mu);
  auto* v = (fake::Event*)e;
  fake::run(fake::streams[v->stream], v->at);
  return hipSuccess;
}
FAKE hipError_t hipStreamSynchronize(hipStream_t s) {
  std::lock_guard<std::mutex> l(fake::mu);
  fake::Stream& q = fake::streams[s];
  fake::run(q, q.issued);
  return hipSuccess;
}
FAKE hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind k, hipStream_t s) {
  if (k == hipMemcpyHostToDevice) {   // pageable source: taken before the call returns
    std::vector<char> held((const char*)src, (const char*)src + n);
    fake::issue(s, [=] { std::memcpy(dst, held.data(), n); });
  } else {
    if (k == hipMemcpyDeviceToHost) {
      std::lock_guard<std::mutex> l(fake::mu);
      fake::d2h.push_back({(char*)dst, n});
      if (fake::fail_copy > 0 && --fake::fail_copy == 0) return fake::err(hipErrorUnknown);
    }
    fake::issue(s, [=] { std::memcpy(dst, src, n); });
  }
  return hipSuccess;
}
FAKE hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t s) {
  fake::issue(s, [=] { std::memset(p, v, n); });
  return hipSuccess;
}
FAKE hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  if (fake::refuse_launch == 0) return hipSuccess;
  --fake::refuse_launch;
  return fake::err(hipErrorLaunchFailure);
}
FAKE hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) {
  return hipSuccess;
}
