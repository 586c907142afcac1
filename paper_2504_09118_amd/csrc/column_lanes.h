// What the column sweeps share: loads and stores that drop cells, neighbours in x by wave shifts, and the
// slots of the register rings.
#pragma once

#include <hip/hip_runtime.h>

namespace fdtd {
namespace {

constexpr unsigned kDrop = 0x80000000u;      // an offset past every plane: reads 0, stores nothing
constexpr int kRawBufferWord3 = 0x00020000;  // gfx9 raw buffer: 32-bit data format, no swizzle

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, kRawBufferWord3);
}

// Value of the lane one column to the right / left; 0 at the window's edge (every lane is active).
__device__ __forceinline__ float right_of(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x130, 0xf, 0xf, true));
}

__device__ __forceinline__ float left_of(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x138, 0xf, 0xf, true));
}

// Slot of role r at phase ph in a ring of m values whose first role is -first.
constexpr int ring_slot(int r, int ph, int first, int m) { return ((r + first + ph) % m + m) % m; }

}  // namespace
}  // namespace fdtd
