#include "host_read.h"

#include <sys/mman.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

namespace fdtd {
namespace {

#ifndef MADV_POPULATE_WRITE
#define MADV_POPULATE_WRITE 23
#endif

// Map the whole pages of a buffer that is about to be written (a kernel that cannot leaves it to the copy).
void map_pages(char *p, size_t n)
{
    const uintptr_t page = 4096, a = ((uintptr_t)p + page - 1) / page * page, b = ((uintptr_t)p + n) / page * page;
    if (a < b)
        (void)madvise((void *)a, b - a, MADV_POPULATE_WRITE);
}

bool known_to_runtime(const void *p)
{
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return at.type == hipMemoryTypeHost || at.type == hipMemoryTypeManaged || at.type == hipMemoryTypeDevice;
}

// Pinned memory is made and freed in the relaxed mode: another thread's capture is not concerned.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

}  // namespace

void HostReader::release()
{
    RelaxedCapture relaxed;
    for (int q = 0; q < events_; ++q) (void)hipEventDestroy(ev_[q]);
    events_ = 0;
    if (pinned_)
        (void)hipHostFree(pinned_);
    pinned_ = nullptr;
    slots_ = 0;
}

hipError_t HostReader::begin(int device, hipStream_t s, int n, size_t largest)
{
    device_ = device;
    stream_ = s;
    closed_ = false;
    lo_ = hi_ = nullptr;
    pending_ = 0;
    issued_ = taken_ = done_ = 0;
    err_ = hipSuccess;
    size_t slot = std::min(kSlot, (largest + 4095) / 4096 * 4096);
    int slots = (int)std::min<size_t>(kSlots, ((size_t)n * ((largest + kSlot - 1) / kSlot) + 1) / 2);
    // Making the slots takes about a millisecond, so they wait until an object has read kWorth (two fields of
    // 3 MiB fetched once: 0.4 ms, 1.5 with the slots made). One array alone is worth a slot (0.9 MiB in fresh
    // pages: 0.5 ms by the runtime, 0.2).
    read_ += (size_t)n * largest;
    if (slots < 1 || (n > 1 && read_ < kWorth) || (pinned_ && slot <= slot_ && slots <= slots_))
        return hipSuccess;
    if (pinned_) {  // a larger read than the last: once more only
        slot = kSlot;
        slots = kSlots;
    }
    release();
    RelaxedCapture relaxed;
    const hipError_t got = hipHostMalloc((void **)&pinned_, slot * slots, hipHostMallocDefault);
    if (got != hipSuccess) {
        (void)hipGetLastError();
        pinned_ = nullptr;  // every array is copied by the runtime
        return hipSuccess;
    }
    for (; events_ < slots; ++events_) {
        const hipError_t e = hipEventCreateWithFlags(&ev_[events_], hipEventDisableTiming);
        if (e != hipSuccess) {
            release();
            return e;
        }
    }
    slot_ = slot;
    slots_ = slots;
    return hipSuccess;
}

// Take the next filled slot and copy it out (lk held on entry and on return).
void HostReader::take(std::unique_lock<std::mutex> &lk)
{
    const int q = (int)(taken_++ % slots_);
    const Part p = part_[q];
    pending_ -= p.bytes;
    lk.unlock();
    const hipError_t e = hipEventSynchronize(ev_[q]);
    if (e == hipSuccess)
        memcpy(p.dst, pinned_ + (size_t)q * slot_, p.bytes);
    lk.lock();
    if (e != hipSuccess && err_ == hipSuccess)
        err_ = e;
    part_[q].busy = false;
    ++done_;
    cv_.notify_all();
}

void HostReader::work()
{
    (void)hipSetDevice(device_);
    std::unique_lock<std::mutex> lk(mu_);
    for (;;) {
        cv_.wait(lk, [&] { return taken_ < issued_ || closed_; });
        if (taken_ >= issued_)
            return;
        take(lk);
    }
}

// The caller's first slot, with pages mapped while the stream has not come to it; then as many threads as
// the bytes in the slots are worth. None waits for the stream's earlier work that way.
void HostReader::spawn(std::unique_lock<std::mutex> &lk)
{
    if (taken_ == 0) {
        for (long long c = 0; c < issued_ && hipEventQuery(ev_[0]) == hipErrorNotReady; ++c)
            map_pages(part_[c].dst, part_[c].bytes);
        (void)hipGetLastError();  // "not ready" is none
        take(lk);
    }
    const int cores = std::max(1, (int)std::thread::hardware_concurrency() / 2);
    const int want = (int)std::min<size_t>(std::min(kThreads, cores) - 1, pending_ / kPerThread);
    try {
        for (; nthreads_ < want; ++nthreads_) thread_[nthreads_] = std::thread([this] { work(); });
    } catch (...) {  // no thread to be had: the ones there are do the work
    }
}

hipError_t HostReader::add(void *dst, const void *dev, size_t bytes)
{
    std::unique_lock<std::mutex> lk(mu_);  // (a worker of an earlier array may be writing err_)
    if (err_ != hipSuccess || bytes == 0)
        return err_;
    char *d = (char *)dst;
    if (lo_ && d < hi_ && d + bytes > lo_) {  // arrays that may overlap arrive in order
        while (taken_ < issued_) {
            spawn(lk);
            if (taken_ < issued_)
                take(lk);
        }
        cv_.wait(lk, [&] { return done_ == issued_; });
    }
    hi_ = lo_ ? std::max(hi_, d + bytes) : d + bytes;
    lo_ = lo_ ? std::min(lo_, d) : d;
    if (!pinned_ || known_to_runtime(dst)) {
        hipError_t e = hipMemcpyAsync(dst, dev, bytes, hipMemcpyDeviceToHost, stream_);
        if (e == hipSuccess)  // (pageable copies left to queue up: 1.6 ms for 64^3, waited for one by one 0.5)
            e = hipStreamSynchronize(stream_);
        return err_ == hipSuccess ? err_ = e : err_;
    }
    const size_t n = (bytes + slot_ - 1) / slot_, len = std::min(slot_, ((bytes + n - 1) / n + 4095) / 4096 * 4096);
    for (size_t a = 0; a < bytes; a += len) {
        const int q = (int)(issued_ % slots_);
        while (part_[q].busy) {
            spawn(lk);
            if (!part_[q].busy)
                break;
            if (taken_ < issued_)
                take(lk);
            else
                cv_.wait(lk);
        }
        const size_t m = std::min(len, bytes - a);
        hipError_t e = hipMemcpyAsync(pinned_ + (size_t)q * slot_, (const char *)dev + a, m, hipMemcpyDeviceToHost,
                                      stream_);
        if (e == hipSuccess)
            e = hipEventRecord(ev_[q], stream_);
        if (e != hipSuccess && err_ == hipSuccess)
            err_ = e;
        if (err_ != hipSuccess)
            return err_;
        part_[q] = Part{d + a, m, true};
        pending_ += m;
        ++issued_;
        cv_.notify_one();
    }
    return hipSuccess;
}

hipError_t HostReader::finish()
{
    std::unique_lock<std::mutex> lk(mu_);
    closed_ = true;
    cv_.notify_all();
    if (taken_ < issued_)
        spawn(lk);
    while (taken_ < issued_) take(lk);
    cv_.wait(lk, [&] { return done_ == issued_; });
    lk.unlock();
    for (; nthreads_ > 0; --nthreads_) thread_[nthreads_ - 1].join();
    if (err_ != hipSuccess)
        (void)hipStreamSynchronize(stream_);  // nothing enqueued here outlives the call
    return err_;
}

}  // namespace fdtd
