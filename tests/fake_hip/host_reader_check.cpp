// Checks of the host reader against the HIP calls of hip/hip_runtime.h here, one per argument; prints "ok".
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <utility>
#include <vector>

#include "host_read.h"

#define CHECK(c)                                                                                                     \
    do {                                                                                                             \
        if (!(c)) {                                                                                                  \
            printf("line %d: %s\n", __LINE__, #c);                                                                   \
            exit(1);                                                                                                 \
        }                                                                                                            \
    } while (0)

namespace fdtd {
hipError_t launch_host_copy(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    if ((uintptr_t)dst % 16 != 0 || (uintptr_t)src % 16 != 0)
        return hipErrorInvalidValue;
    s->push([=] { memcpy(dst, src, bytes); });
    return hipSuccess;
}
}  // namespace fdtd

using fdtd::HostReader;
static const size_t MiB = 1 << 20;

// A worker's wait fails after add has returned: the next add sees the error without a race.
static void error_of_a_worker()
{
    std::vector<char> dev(18 * MiB, 1), dst(18 * MiB);
    static std::atomic<bool> go;
    static std::atomic<int> failed;
    const std::thread::id me = std::this_thread::get_id();
    fake::on_sync = [me] {
        if (std::this_thread::get_id() == me)
            return hipSuccess;
        while (!go.load(std::memory_order_relaxed)) std::this_thread::yield();
        return failed.fetch_add(1, std::memory_order_relaxed) == 0 ? hipErrorUnknown : hipSuccess;
    };
    fake::Stream s;
    HostReader r;
    r.begin(0, &s, 2, 18 * MiB);
    CHECK(r.add(dst.data(), dev.data(), 18 * MiB) == hipSuccess);  // one part more than slots: workers hold three
    go.store(true, std::memory_order_relaxed);
    std::this_thread::sleep_for(std::chrono::milliseconds(200));
    std::vector<char> more(100);
    CHECK(r.add(more.data(), dev.data(), 100) == hipErrorUnknown);
    CHECK(r.finish() == hipErrorUnknown);
    fake::on_sync = [] { return hipSuccess; };
}

// Making and freeing pinned memory leaves another thread's capture alone, also where larger slots take the
// place of smaller ones.
static void capture_mode()
{
    std::vector<char> dev(6 * MiB, 1), dst(6 * MiB);
    fake::Stream s;
    {
        HostReader r;
        for (size_t n : {MiB, 6 * MiB}) {
            r.begin(0, &s, 1, n);
            CHECK(r.add(dst.data(), dev.data(), n) == hipSuccess);
            CHECK(r.finish() == hipSuccess);
        }
        CHECK(fake::allocations >= 1);
        CHECK(memcmp(dst.data(), dev.data(), 6 * MiB) == 0);
    }
    CHECK(fake::unrelaxed == 0);
    CHECK(fake::mode == hipStreamCaptureModeGlobal);
}

// n arrays of bytes each into fresh memory, by one object; the values arrive.
static hipError_t read(HostReader &r, int n, size_t bytes, bool runtime_knows = false)
{
    std::vector<std::vector<char>> dev(n), dst(n);
    fake::Stream s;
    r.begin(0, &s, n, bytes);
    for (int q = 0; q < n; ++q) {
        dev[q].assign(bytes, (char)(q + 1));
        dst[q].resize(bytes);
        if (runtime_knows)
            fake::known.insert(dst[q].data());
        if (r.add(dst[q].data(), dev[q].data(), bytes) != hipSuccess)
            break;
    }
    const hipError_t e = r.finish();
    if (runtime_knows)
        fake::known.clear();
    if (e == hipSuccess)
        CHECK(dst == dev);
    return e;
}

// Slots outlive the object that they were made for, and only slots that were leased are given back.
static void slots_are_shared()
{
    for (int q = 0; q < 3; ++q) {
        HostReader r;
        CHECK(read(r, 6, 8 * MiB) == hipSuccess);
        CHECK(fake::allocations == 1);
    }
    CHECK(fake::live == 1);
}

// Memory that the runtime knows takes no slots, and makes none.
static void known_memory_makes_no_slots()
{
    HostReader r;
    for (int q = 0; q < 3; ++q) CHECK(read(r, 6, 8 * MiB, true) == hipSuccess);
    CHECK(fake::allocations == 0);
}

// Slots wait until the objects together have read enough, by reads of any size, and then serve any size.
static void small_reads()
{
    for (int q = 0; q < 3; ++q) {
        HostReader r;
        CHECK(read(r, 6, MiB) == hipSuccess);
    }
    CHECK(fake::allocations == 0);
    for (int q = 0; q < 20; ++q) {
        HostReader r;
        CHECK(read(r, 6, MiB / 2) == hipSuccess);
    }
    CHECK(fake::allocations == 1);
    HostReader r;
    int copies = fake::runtime_copies;
    CHECK(read(r, 6, 100) == hipSuccess);
    CHECK(fake::allocations == 1 && fake::runtime_copies == copies);
    CHECK(read(r, 1, 100) == hipSuccess);
    CHECK(fake::allocations == 1 && fake::runtime_copies == copies);
}

// Slots are filled by the kernel, whatever the sizes; a source off its 16-byte boundary is the runtime's.
static void filled_by_the_kernel()
{
    HostReader r;
    for (size_t odd : {0, 4, 4095}) CHECK(read(r, 6, 8 * MiB + odd) == hipSuccess);
    CHECK(fake::allocations == 1 && fake::runtime_copies == 0);
    std::vector<char> dev(6 * MiB + 4, 7), dst(6 * MiB);
    fake::Stream s;
    r.begin(0, &s, 1, 6 * MiB);
    CHECK(r.add(dst.data(), dev.data() + 4, 6 * MiB) == hipSuccess);
    CHECK(r.finish() == hipSuccess);
    CHECK(fake::runtime_copies == 1 && memcmp(dst.data(), dev.data() + 4, 6 * MiB) == 0);
}

// Readers at the same time: a bounded number of slot sets, of which one stays when the last object goes.
static void readers_at_once()
{
    {
        HostReader r[8];
        std::vector<std::thread> t;
        for (auto &x : r)
            t.emplace_back([&x] {
                for (int q = 0; q < 6; ++q) CHECK(read(x, 3, 5 * MiB) == hipSuccess);
            });
        for (auto &x : t) x.join();
        CHECK(fake::live >= 1 && fake::live <= 4);
    }
    CHECK(fake::live == 1);
}

// No pinned memory to be had: the runtime copies.
static void no_pinned_memory()
{
    fake::fail_alloc = true;
    HostReader r;
    for (int q = 0; q < 3; ++q) CHECK(read(r, 6, 8 * MiB) == hipSuccess);
    fake::fail_alloc = false;
    CHECK(read(r, 6, 8 * MiB) == hipSuccess);
    CHECK(fake::allocations == 1);
}

// After a stream that cannot be waited for, its copies may still be to come: their slots are not used again.
static void slots_of_a_failed_stream()
{
    HostReader r;
    CHECK(read(r, 6, 8 * MiB) == hipSuccess);
    fake::on_sync = [] { return hipErrorUnknown; };
    fake::stream_fails = true;
    CHECK(read(r, 6, 8 * MiB) == hipErrorUnknown);
    fake::on_sync = [] { return hipSuccess; };
    fake::stream_fails = false;
    CHECK(fake::allocations == 1 && fake::live == 1);
    for (int q = 0; q < 3; ++q) CHECK(read(r, 6, 8 * MiB) == hipSuccess);
    CHECK(fake::allocations == 2);
}

int main(int argc, char **argv)
{
    for (int a = 1; a < argc; ++a) {
        const std::string what = argv[a];
        bool known = false;
        for (const auto &c : std::initializer_list<std::pair<const char *, void (*)()>>{
                 {"error_of_a_worker", error_of_a_worker},
                 {"capture_mode", capture_mode},
                 {"slots_are_shared", slots_are_shared},
                 {"known_memory_makes_no_slots", known_memory_makes_no_slots},
                 {"small_reads", small_reads},
                 {"filled_by_the_kernel", filled_by_the_kernel},
                 {"readers_at_once", readers_at_once},
                 {"no_pinned_memory", no_pinned_memory},
                 {"slots_of_a_failed_stream", slots_of_a_failed_stream}})
            if (what == c.first) {
                known = true;
                c.second();
            }
        CHECK(known);
    }
    printf("ok\n");
}
