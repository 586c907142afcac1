// Checks of the host reader against the HIP calls of hip/hip_runtime.h here, one per argument; prints "ok".
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "host_read.h"

#define CHECK(c)                                                                                                     \
    do {                                                                                                             \
        if (!(c)) {                                                                                                  \
            printf("line %d: %s\n", __LINE__, #c);                                                                   \
            exit(1);                                                                                                 \
        }                                                                                                            \
    } while (0)

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
    CHECK(r.begin(0, &s, 2, 18 * MiB) == hipSuccess);
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
            CHECK(r.begin(0, &s, 1, n) == hipSuccess);
            CHECK(r.add(dst.data(), dev.data(), n) == hipSuccess);
            CHECK(r.finish() == hipSuccess);
        }
        CHECK(fake::allocations >= 1);
        CHECK(memcmp(dst.data(), dev.data(), 6 * MiB) == 0);
    }
    CHECK(fake::unrelaxed == 0);
    CHECK(fake::mode == hipStreamCaptureModeGlobal);
}

int main(int argc, char **argv)
{
    for (int a = 1; a < argc; ++a) {
        const std::string what = argv[a];
        if (what == "error_of_a_worker")
            error_of_a_worker();
        else if (what == "capture_mode")
            capture_mode();
        else
            CHECK(!"known check");
    }
    printf("ok\n");
}
