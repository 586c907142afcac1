// The HIP calls that host_read.cpp makes, on the CPU: a stream is a thread that does its copies in order,
// pinned memory comes from the heap. Counters and hooks for the checks.
#pragma once

#include <atomic>
#include <condition_variable>
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <mutex>
#include <set>
#include <thread>

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorNotReady = 600, hipErrorUnknown = 999 };
enum hipStreamCaptureMode {
    hipStreamCaptureModeGlobal = 0,
    hipStreamCaptureModeThreadLocal = 1,
    hipStreamCaptureModeRelaxed = 2
};
enum hipMemoryType { hipMemoryTypeUnregistered, hipMemoryTypeHost, hipMemoryTypeDevice, hipMemoryTypeManaged };
enum hipMemcpyKind { hipMemcpyDeviceToHost = 2 };
constexpr unsigned hipHostMallocDefault = 0, hipEventDisableTiming = 2;
struct hipPointerAttribute_t {
    hipMemoryType type;
};

namespace fake {

inline thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
inline std::atomic<int> allocations{0}, live{0}, unrelaxed{0}, runtime_copies{0};
inline std::atomic<bool> fail_alloc{false};
inline std::set<const void *> known;                            // destinations that the runtime knows
inline std::function<hipError_t()> on_sync = [] { return hipSuccess; };  // what waiting for an event does
inline std::atomic<bool> stream_fails{false};                              // and for a stream

struct Event {
    std::mutex m;
    std::condition_variable cv;
    bool done = true;
};
struct Stream {
    std::mutex m;
    std::condition_variable cv;
    std::deque<std::function<void()>> q;
    bool stop = false;
    int running = 0;
    std::thread t;
    Stream() : t([this] { loop(); }) {}
    ~Stream()
    {
        {
            std::lock_guard<std::mutex> l(m);
            stop = true;
        }
        cv.notify_all();
        t.join();
    }
    void push(std::function<void()> f)
    {
        std::lock_guard<std::mutex> l(m);
        q.push_back(std::move(f));
        cv.notify_all();
    }
    void drain()
    {
        std::unique_lock<std::mutex> l(m);
        cv.wait(l, [&] { return q.empty() && !running; });
    }
    void loop()
    {
        std::unique_lock<std::mutex> l(m);
        for (;;) {
            cv.wait(l, [&] { return stop || !q.empty(); });
            if (q.empty())
                return;
            auto f = std::move(q.front());
            q.pop_front();
            running = 1;
            l.unlock();
            f();
            l.lock();
            running = 0;
            cv.notify_all();
        }
    }
};

}  // namespace fake

typedef fake::Event *hipEvent_t;
typedef fake::Stream *hipStream_t;

inline void fake_need_relaxed()
{
    if (fake::mode != hipStreamCaptureModeRelaxed)
        ++fake::unrelaxed;
}
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m)
{
    std::swap(*m, fake::mode);
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    fake_need_relaxed();
    if (fake::fail_alloc)
        return hipErrorUnknown;
    ++fake::allocations;
    ++fake::live;
    *p = malloc(n);
    return hipSuccess;
}
inline hipError_t hipHostFree(void *p)
{
    fake_need_relaxed();
    --fake::live;
    free(p);
    return hipSuccess;
}
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    a->type = fake::known.count(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = new fake::Event;
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e)
{
    delete e;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    {
        std::lock_guard<std::mutex> l(e->m);
        e->done = false;
    }
    s->push([e] {
        std::lock_guard<std::mutex> l(e->m);
        e->done = true;
        e->cv.notify_all();
    });
    return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e)
{
    std::lock_guard<std::mutex> l(e->m);
    return e->done ? hipSuccess : hipErrorNotReady;
}
inline hipError_t hipEventSynchronize(hipEvent_t e)
{
    {
        std::unique_lock<std::mutex> l(e->m);
        e->cv.wait(l, [&] { return e->done; });
    }
    return fake::on_sync();
}
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    ++fake::runtime_copies;
    st->push([=] { memcpy(d, s, n); });
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s)
{
    s->drain();
    return fake::stream_fails ? hipErrorUnknown : hipSuccess;
}
