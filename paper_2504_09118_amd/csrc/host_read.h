// Device arrays into pageable host memory.
//
// The runtime's own copy into fresh pageable memory pins the caller's pages chunk by chunk: 4.4 GB/s from 1
// MiB on, 17 into mapped pages, where the link carries 57. Here a kernel fills pinned slots and up to kThreads
// threads (the caller is one) copy them out, so that the pages are mapped by all of them; while the stream is
// still busy with earlier work the caller maps pages ahead. Fresh pages and mapped ones, the runtime's copy
// in brackets: all FP32 fields of 256^3 (404 MB) 11.3 and 8.5 ms (40 and 23), of 128^3 2.1 and 1.2 (6.1 and
// 3.0). Memory that the runtime knows (pinned, managed) still takes one copy of its own.
//
// The slots belong to the device and are leased for a read: made by each object, a first read of 96^3 FP32
// fields took 2.9 ms (the runtime's copy 1.4), and its end 0.3 ms more.
#pragma once

#include <hip/hip_runtime.h>

#include <condition_variable>
#include <cstddef>
#include <mutex>
#include <thread>

namespace fdtd {

// slots of 2 MiB and four threads: 256^3 FP32 fields arrived in 19 ms with 512 KiB slots, 11 with 2 MiB; in 31
// by one thread, 12 by four, 11 by six (slots filled by the runtime's copies)
constexpr size_t kSlot = 2 << 20;
constexpr int kSlots = 8;
constexpr int kSlotSets = 4;  // of a device

struct PinnedSlots {
    char *mem;
    size_t slot;  // bytes of each
    int slots;
    hipEvent_t ev[kSlots];
};

// A kernel that copies device memory to pinned memory, both on 16-byte boundaries (k_host_copy.hip).
hipError_t launch_host_copy(void *dst, const void *src, size_t bytes, hipStream_t s);

// One read at a time: begin, add for each array in stream order (a source may be rewritten by work enqueued
// after its add), finish. After an error finish is still called.
class HostReader {
public:
    HostReader();
    HostReader(const HostReader &) = delete;
    HostReader &operator=(const HostReader &) = delete;
    ~HostReader();
    // A read of n arrays of at most largest bytes each, in order on s; the device is current.
    void begin(int device, hipStream_t s, int n, size_t largest);
    hipError_t add(void *dst, const void *dev, size_t bytes);
    hipError_t finish();  // every array has arrived

private:
    static constexpr int kThreads = 4;
    static constexpr size_t kPerThread = 2 << 20;  // a thread costs about 20 us to start, 2 MiB 140 to copy

    struct Part {
        char *dst;
        size_t bytes;
        bool busy;
    };
    void take(std::unique_lock<std::mutex> &lk);
    void work();
    void spawn(std::unique_lock<std::mutex> &lk);

    int device_ = 0, n_ = 0;
    size_t largest_ = 0;
    hipStream_t stream_ = nullptr;
    PinnedSlots *slots_ = nullptr;  // leased from the first pageable array on; null: the runtime copies
    bool tried_ = false;
    char *lo_ = nullptr, *hi_ = nullptr;  // hull of the destinations of this read
    size_t pending_ = 0;                  // bytes in slots that no thread has taken
    std::mutex mu_;
    std::condition_variable cv_;
    Part part_[kSlots] = {};
    long long issued_ = 0, taken_ = 0, done_ = 0;
    bool closed_ = false;
    hipError_t err_ = hipSuccess;
    std::thread thread_[kThreads - 1];
    int nthreads_ = 0;
};

}  // namespace fdtd
