// The few runtime calls of the upload ring on the host alone, for a test without a GPU.  "Device" memory is host memory.
// Streams are queues whose work is done as late as the calls allow: when an event in it or the stream itself is waited for.
// hipStreamPerThread names another queue in every thread, as it does in the runtime.
#pragma once

#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <utility>

typedef int hipError_t;
constexpr hipError_t hipSuccess = 0, hipErrorUnknown = 999;
struct StubStream;
typedef StubStream* hipStream_t;
#define hipStreamPerThread ((hipStream_t)2)
enum { hipMemcpyHostToDevice = 1 };
constexpr unsigned hipEventDisableTiming = 2;

struct StubCopy {
    void* dst;
    const void* src;
    size_t bytes;
};
struct StubQueue {
    std::deque<StubCopy> work;
    size_t taken = 0, done = 0;  // copies ever enqueued, ever carried out
};
struct StubEvent {
    StubQueue* queue = nullptr;
    size_t upto = 0;
};
typedef StubEvent* hipEvent_t;

inline std::mutex stub_lock;
inline std::map<std::pair<hipStream_t, int>, StubQueue> stub_queues;
inline int stub_threads = 0;
inline thread_local int stub_thread = 0;  // numbers are not used again, unlike thread ids
inline int stub_fail_copy = -1;  // the copy, counted from here, that is refused

inline StubQueue& stub_queue(hipStream_t st)
{
    if (stub_thread == 0) stub_thread = ++stub_threads;
    return stub_queues[{st, st == hipStreamPerThread ? stub_thread : 0}];
}
inline void stub_run(StubQueue& q, size_t upto)
{
    for (; q.done < upto; ++q.done) {
        memcpy(q.work.front().dst, q.work.front().src, q.work.front().bytes);
        q.work.pop_front();
    }
}

inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n) { return (*p = malloc(n)) != nullptr ? hipSuccess : hipErrorUnknown; }
inline hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new StubEvent(); return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, int, hipStream_t st)
{
    std::lock_guard<std::mutex> g(stub_lock);
    if (stub_fail_copy >= 0 && stub_fail_copy-- == 0) return hipErrorUnknown;
    StubQueue& q = stub_queue(st);
    q.work.push_back({dst, src, n});
    ++q.taken;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t st)
{
    std::lock_guard<std::mutex> g(stub_lock);
    e->queue = &stub_queue(st);
    e->upto = e->queue->taken;
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e)
{
    std::lock_guard<std::mutex> g(stub_lock);
    if (e->queue != nullptr) stub_run(*e->queue, e->upto);
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t st)
{
    std::lock_guard<std::mutex> g(stub_lock);
    StubQueue& q = stub_queue(st);
    stub_run(q, q.taken);
    return hipSuccess;
}
