// Copy of a device array into pinned host memory by a kernel.
//
// The runtime's copies run on engines that it picks by itself when several are queued: 50 MB of 128^3 fields
// arrived in 1.45, 3.4 or 5.2 ms, one program going from one to the other (a pool's fetch of six such
// requests: 8.7, 19 or 31 ms; one copy waited for after the other, 18). A kernel's stores take 1.20 ms (7.3)
// each time. Bound by the link and the threads that empty the slots: 16, 64 and 256 workgroups take 1.25,
// 1.22 and 1.20 ms, and the fewer leave more of the chip to a sweep beside them.
#include "host_read.h"

namespace fdtd {
namespace {

constexpr int kBlock = 256, kUnroll = 4, kGrid = 64;

__global__ void __launch_bounds__(kBlock) k_host_copy(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n,
                                                      int tail)
{
    const size_t T = (size_t)gridDim.x * kBlock, t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    size_t q = t;
    for (; q + (kUnroll - 1) * T < n; q += kUnroll * T) {
        uint4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) v[u] = src[q + u * T];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) dst[q + u * T] = v[u];
    }
    for (; q < n; q += T) dst[q] = src[q];
    if (t < (size_t)tail)
        ((unsigned char *)(dst + n))[t] = ((const unsigned char *)(src + n))[t];
}

}  // namespace

// src and dst on 16-byte boundaries
hipError_t launch_host_copy(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16, blocks = (n + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_host_copy, dim3(blocks < 1 ? 1 : blocks < kGrid ? (unsigned)blocks : kGrid), dim3(kBlock), 0, s,
                       (const uint4 *)src, (uint4 *)dst, n, (int)(bytes % 16));
    return hipGetLastError();
}

}  // namespace fdtd
