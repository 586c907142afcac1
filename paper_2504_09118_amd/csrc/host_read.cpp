#include "host_read.h"

#include <sys/mman.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <new>

namespace fdtd {
namespace {

#ifndef MADV_POPULATE_WRITE
#define MADV_POPULATE_WRITE 23
#endif

// Map the whole pages of a buffer that is about to be written, unless its first and last are (a kernel that
// cannot leaves it to the copy).
void map_pages(char *p, size_t n)
{
    const uintptr_t page = 4096, a = ((uintptr_t)p + page - 1) / page * page, b = ((uintptr_t)p + n) / page * page;
    unsigned char first = 0, last = 0;
    if (a >= b)
        return;
    if (mincore((void *)a, page, &first) == 0 && mincore((void *)(b - page), page, &last) == 0 && (first & last & 1))
        return;
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

// What the readers of a device share. Nothing is freed when the process ends: the runtime may be gone by then.
struct Shared {
    size_t read = 0;  // bytes read so far
    int sets = 0;     // made and not freed, leased ones among them
    PinnedSlots *idle[kSlotSets] = {};
    int nidle = 0;
};
constexpr size_t kWorth = 32 << 20;
constexpr int kDevices = 64;
Shared g_shared[kDevices];
std::mutex g_mu;
int g_readers = 0;  // objects

void destroy(PinnedSlots *p)
{
    RelaxedCapture relaxed;
    for (hipEvent_t e : p->ev)
        if (e)
            (void)hipEventDestroy(e);
    if (p->mem)
        (void)hipHostFree(p->mem);
    delete p;
}

PinnedSlots *create(size_t slot, int slots)
{
    RelaxedCapture relaxed;
    auto *p = new (std::nothrow) PinnedSlots{nullptr, slot, slots, {}};
    if (!p)
        return nullptr;
    hipError_t e = hipHostMalloc((void **)&p->mem, slot * slots, hipHostMallocDefault);
    if (e != hipSuccess)
        p->mem = nullptr;
    for (int q = 0; q < slots && e == hipSuccess; ++q) e = hipEventCreateWithFlags(&p->ev[q], hipEventDisableTiming);
    if (e == hipSuccess)
        return p;
    (void)hipGetLastError();
    destroy(p);
    return nullptr;
}

// Slots for a read of n arrays of at most largest bytes, or null: the runtime copies. Making them takes one
// to two milliseconds and saves 27 us for a MiB in mapped pages, more in fresh ones, so the first set waits
// until kWorth has been read, the next ones (readers at the same time) for as much each. One array alone is
// worth a set of its size at once (0.9 MiB in fresh pages: 0.5 ms by the runtime, 0.2). A set there is serves
// every size: six arrays of 16^3 or less arrive in 70 to 90 us, not 146, of 48^3 in 140, not 255; a gradient
// of 24^3 by 24 steps takes 180, not 249.
PinnedSlots *lease(int device, int n, size_t largest)
{
    size_t slot = std::min(kSlot, (largest + 4095) / 4096 * 4096);
    int slots = (int)std::min<size_t>(kSlots, ((size_t)n * ((largest + kSlot - 1) / kSlot) + 1) / 2);
    if (slots < 1 || device < 0 || device >= kDevices)
        return nullptr;
    Shared &d = g_shared[device];
    PinnedSlots *small = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (int q = d.nidle - 1; q >= 0; --q) {
            PinnedSlots *p = d.idle[q];
            if (p->slot >= slot && p->slots >= slots) {
                d.idle[q] = d.idle[--d.nidle];
                return p;
            }
        }
        const bool worth = d.read >= kWorth;
        if (d.nidle > 0 && (worth || n == 1)) {  // too small for this read: once more only
            small = d.idle[--d.nidle];
        } else if (d.sets < kSlotSets && (d.read >= kWorth * (d.sets + 1) || n == 1)) {
            ++d.sets;
        } else {
            return nullptr;
        }
        if (small || worth) {
            slot = kSlot;
            slots = kSlots;
        }
    }
    if (small)
        destroy(small);
    PinnedSlots *p = create(slot, slots);
    if (!p) {
        std::lock_guard<std::mutex> lk(g_mu);
        --d.sets;
    }
    return p;
}

}  // namespace

HostReader::HostReader()
{
    std::lock_guard<std::mutex> lk(g_mu);
    ++g_readers;
}

// The last object leaves one set to the next.
HostReader::~HostReader()
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (--g_readers > 0)
        return;
    for (Shared &d : g_shared)
        for (; d.nidle > 1; --d.sets) destroy(d.idle[--d.nidle]);
}

void HostReader::begin(int device, hipStream_t s, int n, size_t largest)
{
    device_ = device;
    stream_ = s;
    n_ = n;
    largest_ = largest;
    slots_ = nullptr;
    tried_ = false;
    closed_ = false;
    lo_ = hi_ = nullptr;
    pending_ = 0;
    issued_ = taken_ = done_ = 0;
    err_ = hipSuccess;
    std::lock_guard<std::mutex> lk(g_mu);
    if (device >= 0 && device < kDevices)
        g_shared[device].read += (size_t)n * largest;
}

// Take the next filled slot and copy it out (lk held on entry and on return).
void HostReader::take(std::unique_lock<std::mutex> &lk)
{
    const int q = (int)(taken_++ % slots_->slots);
    const Part p = part_[q];
    pending_ -= p.bytes;
    lk.unlock();
    map_pages(p.dst, p.bytes);  // in one call, not a fault a page: 96^3 FP32 fields 1.75 -> 1.27 ms
    const hipError_t e = hipEventSynchronize(slots_->ev[q]);
    if (e == hipSuccess)
        memcpy(p.dst, slots_->mem + (size_t)q * slots_->slot, p.bytes);
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
        for (long long c = 0; c < issued_ && hipEventQuery(slots_->ev[0]) == hipErrorNotReady; ++c)
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
    const bool known = (slots_ || !tried_) && ((uintptr_t)dev % 16 != 0 || known_to_runtime(dst));
    if (!known && !tried_) {
        slots_ = lease(device_, n_, largest_);
        tried_ = true;
    }
    if (known || !slots_) {
        hipError_t e = hipMemcpyAsync(dst, dev, bytes, hipMemcpyDeviceToHost, stream_);
        if (e == hipSuccess)  // (pageable copies left to queue up: 1.6 ms for 64^3, waited for one by one 0.5)
            e = hipStreamSynchronize(stream_);
        return err_ == hipSuccess ? err_ = e : err_;
    }
    const size_t slot = slots_->slot, n = (bytes + slot - 1) / slot;
    const size_t len = std::min(slot, ((bytes + n - 1) / n + 4095) / 4096 * 4096);
    for (size_t a = 0; a < bytes; a += len) {
        const int q = (int)(issued_ % slots_->slots);
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
        hipError_t e = launch_host_copy(slots_->mem + q * slot, (const char *)dev + a, m, stream_);
        if (e == hipSuccess)
            e = hipEventRecord(slots_->ev[q], stream_);
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
    // Every event has been waited for, so nothing enqueued here outlives the call; after an error the stream is,
    // and where that fails the slots are not used again. (A wait for the stream each time costs 30 us a read: it
    // has a marker of its own to send; without it the solver's end pays them once.)
    const hipError_t e = err_ != hipSuccess ? hipStreamSynchronize(stream_) : hipSuccess;
    if (slots_ && e == hipSuccess) {
        std::lock_guard<std::mutex> shared_lk(g_mu);
        Shared &sh = g_shared[device_];
        sh.idle[sh.nidle++] = slots_;
    }
    slots_ = nullptr;
    return err_ != hipSuccess ? err_ : e;
}

}  // namespace fdtd
