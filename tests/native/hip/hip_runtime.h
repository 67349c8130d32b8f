// Just enough of the runtime's interface to run host_copy.h on the CPU: one stream whose copies happen later, on a thread of its
// own, and switches that make a call fail.
#pragma once

#include <atomic>
#include <condition_variable>
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <mutex>
#include <thread>

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1, hipMemoryTypeDevice = 2 };
enum hipMemcpyKind { hipMemcpyDeviceToHost = 2 };
constexpr unsigned hipHostMallocDefault = 0, hipEventDisableTiming = 2;
struct hipPointerAttribute_t { hipMemoryType type; };
struct StubEvent { std::atomic<int> pending{0}; };
using hipEvent_t = StubEvent*;
using hipStream_t = struct StubStream*;

struct StubStream {
    std::mutex m;
    std::condition_variable cv;
    std::deque<std::function<void()>> todo;
    bool busy = false, stop = false;
    std::thread worker{[this] {
        std::unique_lock<std::mutex> l(m);
        for (;;) {
            cv.wait(l, [this] { return stop || !todo.empty(); });
            if (todo.empty()) return;
            auto f = std::move(todo.front());
            todo.pop_front();
            busy = true;
            l.unlock();
            f();
            l.lock();
            busy = false;
            cv.notify_all();
        }
    }};
    void push(std::function<void()> f) {
        std::lock_guard<std::mutex> l(m);
        todo.push_back(std::move(f));
        cv.notify_all();
    }
    void drain() {
        std::unique_lock<std::mutex> l(m);
        cv.wait(l, [this] { return todo.empty() && !busy; });
    }
    bool idle() {
        std::lock_guard<std::mutex> l(m);
        return todo.empty() && !busy;
    }
    ~StubStream() {
        { std::lock_guard<std::mutex> l(m); stop = true; cv.notify_all(); }
        worker.join();
    }
};

struct Stub {
    int fail_host_malloc = 0, fail_event_create = -1, fail_set_device = 0;       // event: number of the one that fails
    int fail_copy = -1, fail_sync = -1;                                         // number of the call that fails
    hipMemoryType dst_type = hipMemoryTypeUnregistered;
    int attributes_fail = 0;
    std::atomic<int> copies{0}, syncs{0}, plain{0}, events{0}, host_blocks{0};
};
inline Stub stub;

inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipSetDevice(int) { return stub.fail_set_device ? hipErrorUnknown : hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (stub.fail_host_malloc) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    ++stub.host_blocks;
    return hipSuccess;
}
inline hipError_t hipHostFree(void* p) { std::free(p); --stub.host_blocks; return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    if (stub.events == stub.fail_event_create) return hipErrorOutOfMemory;
    ++stub.events;
    *e = new StubEvent;
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) { --stub.events; delete e; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    e->pending.store(1);
    s->push([e] { e->pending.store(0); });
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
    if (stub.syncs++ == stub.fail_sync) return hipErrorUnknown;
    while (e->pending.load()) std::this_thread::yield();
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) { s->drain(); return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    if (stub.copies++ == stub.fail_copy) return hipErrorUnknown;
    st->push([=] { std::memcpy(d, s, n); });
    return hipSuccess;
}
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    ++stub.plain;
    std::memcpy(d, s, n);
    return hipSuccess;
}
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
    if (stub.attributes_fail) return hipErrorInvalidValue;
    a->type = stub.dst_type;
    return hipSuccess;
}
