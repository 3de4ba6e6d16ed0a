// A host-only stand-in for the parts of the HIP runtime that the library's host code calls, to run
// that code on the CPU.  "Device" memory is host memory.  A stream is a queue whose work runs only
// when something waits for it (an event wait runs the other stream up to the event, nothing
// further), the latest order that the enqueued waits allow: a missing wait shows as wrong data.
// fail_at makes one enqueue (launch, copy, event record or wait) return an error.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <vector>

namespace fake {

struct Stream;
struct Ticket {  // one record of an event
  Stream* on;
  bool done = false;
};
struct Op {
  std::function<void()> run;
  std::shared_ptr<Ticket> wait, record;
};
struct Stream {
  int device = 0;
  std::deque<Op> ops;
};
struct Alloc {
  size_t bytes;
  bool device;  // else pinned host memory
  int on;
  bool alive;
};

inline int current = 0;
inline Stream null_stream;
inline std::vector<std::unique_ptr<Stream>> streams;
inline std::map<char*, Alloc> allocs;
inline long enqueues = 0, fail_at = 0;  // fail_at: which enqueue fails, counted from 1; 0: none
inline bool fail_late = false;          // a launch that fails is enqueued all the same (an older error reported late)
inline int dead_accesses = 0;           // work that ran on memory already freed

inline Stream* of(hipStream_t s) { return s ? reinterpret_cast<Stream*>(s) : &null_stream; }

inline void run_front(Stream* s);
inline void run_until(const std::shared_ptr<Ticket>& t) {
  while (!t->done) run_front(t->on);
}
inline void run_front(Stream* s) {
  if (s->ops.empty()) std::abort();  // an event that never comes
  Op op = std::move(s->ops.front());
  s->ops.pop_front();
  if (op.wait) run_until(op.wait);
  if (op.run) op.run();
  if (op.record) op.record->done = true;
}
inline void drain(Stream* s) {
  while (!s->ops.empty()) run_front(s);
}
inline void drain_all(int device) {
  if (null_stream.device == device) drain(&null_stream);
  for (auto& s : streams)
    if (s->device == device) drain(s.get());
}

inline bool failing() { return ++enqueues == fail_at; }

inline hipError_t launch(hipStream_t s, std::function<void()> f) {
  const bool fails = failing();
  if (!fails || fail_late) of(s)->ops.push_back(Op{std::move(f), nullptr, nullptr});
  return fails ? hipErrorUnknown : hipSuccess;
}

inline Alloc* find(const void* p) {
  char* c = static_cast<char*>(const_cast<void*>(p));
  auto it = allocs.upper_bound(c);
  if (it == allocs.begin()) return nullptr;
  --it;
  return c < it->first + it->second.bytes ? &it->second : nullptr;
}
// Work that runs calls it for each buffer it touches.
inline void touch(const void* p) {
  const Alloc* a = find(p);
  if (!a || !a->alive) ++dead_accesses;
}

inline hipError_t add(void** p, size_t bytes, bool device) {
  *p = std::aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
  if (!*p) return hipErrorOutOfMemory;
  allocs[static_cast<char*>(*p)] = Alloc{bytes, device, current, true};
  return hipSuccess;
}
// Freed memory is kept and filled, so that late accesses are counted rather than corrupt the heap.
inline hipError_t release(void* p) {
  if (!p) return hipSuccess;
  Alloc& a = allocs.at(static_cast<char*>(p));
  a.alive = false;
  std::memset(p, 0xDD, a.bytes);
  return hipSuccess;
}
inline void release_for_good() {
  for (auto& [p, a] : allocs) std::free(p);
  allocs.clear();
}

}  // namespace fake

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = fake::current, hipSuccess; }
hipError_t hipSetDevice(int d) { return fake::current = d, hipSuccess; }
hipError_t hipDeviceSynchronize() { return fake::drain_all(fake::current), hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipMalloc(void** p, size_t n) { return fake::add(p, n, true); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return fake::add(p, n, false); }
hipError_t hipFree(void* p) { return fake::drain_all(fake::current), fake::release(p); }  // as documented
hipError_t hipHostFree(void* p) { return fake::release(p); }
hipError_t hipMemset(void* p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  return fake::launch(st, [=] {
    fake::touch(d);
    fake::touch(s);
    std::memcpy(d, s, n);
  });
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  const fake::Alloc* x = fake::find(p);
  if (!x || !x->alive) return hipErrorInvalidValue;
  std::memset(a, 0, sizeof(*a));
  a->type = x->device ? hipMemoryTypeDevice : hipMemoryTypeHost;
  a->device = x->on;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  fake::streams.push_back(std::make_unique<fake::Stream>());
  fake::streams.back()->device = fake::current;
  *s = reinterpret_cast<hipStream_t>(fake::streams.back().get());
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return fake::drain(fake::of(s)), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return fake::drain(fake::of(s)), hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
  return *c = hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new std::shared_ptr<fake::Ticket>());
  return hipSuccess;
}
static std::shared_ptr<fake::Ticket>& ticket(hipEvent_t e) { return *reinterpret_cast<std::shared_ptr<fake::Ticket>*>(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete &ticket(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (fake::failing()) return hipErrorUnknown;
  ticket(e) = std::make_shared<fake::Ticket>(fake::Ticket{fake::of(s)});
  fake::of(s)->ops.push_back(fake::Op{nullptr, nullptr, ticket(e)});
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (fake::failing()) return hipErrorUnknown;
  if (ticket(e)) fake::of(s)->ops.push_back(fake::Op{nullptr, ticket(e), nullptr});
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (ticket(e)) fake::run_until(ticket(e));
  return hipSuccess;
}
}  // extern "C"
