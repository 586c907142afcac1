// Tile numbering and the tile queue shared by the temporal sweeps.
#pragma once

#include "fdtd_internal.h"

namespace fdtd {
namespace {

constexpr int kXcds = 8;

// Tile number of virtual block v (with one workgroup per tile, v is the
// hardware block number, and block b runs on XCD b % 8).
// remap 1: XCD x owns tiles [x * nper, (x + 1) * nper).
// remap 2: one workgroup per CU is resident, so blocks 8 cpx w .. 8 cpx (w + 1) - 1
// run together; they take the contiguous tile range starting at 8 cpx w, XCD x
// the x-th part of it, so the halo rows two neighbouring parts share are read
// at about the same time (the last, partial range is split the same way).
__device__ __forceinline__ int tile_of_block(int v, int ntiles, int remap, int cpx)
{
    if (remap == 0)
        return v;
    const int x = v % kXcds, k = v / kXcds;
    if (remap == 1)
        return x * ((ntiles + kXcds - 1) / kXcds) + k;
    const int w = k / cpx, base = w * kXcds * cpx;
    const int rem = min(kXcds * cpx, ntiles - base);
    return base + x * ((rem + kXcds - 1) / kXcds) + (k - w * cpx);
}

// Tile queue: one workgroup per CU takes virtual blocks until none is left.
// Virtual block v (v < nvb, a multiple of 8) sits in list v % 8, in the
// remap-2 order above; the workgroups on XCD x (hardware register XCC_ID) take
// list x in order, so the tiles that share halo lines run together in one L2,
// then help the other lists, so every block is taken exactly once wherever the
// workgroups run. A CU that ends a tile early starts the next at once, instead
// of waiting for the dispatcher, which hands out blocks in order round the
// XCDs and so holds every XCD to the slowest. No workgroup ever waits for
// another. q[0..7]: next index of each list; q[8]: workgroups done; q[9]: lists
// seen empty. The one that finishes last has seen every take and zeroes the
// counters for the next launch (launches sharing them are ordered by their stream).
constexpr int kQueueWords = kXcds + 2;

struct TileQueue {
    unsigned *q;
    int per;   // blocks per list (nvb / 8)
    int list;  // list taken now

    __device__ explicit TileQueue(unsigned *q_, int nvb) : q(q_), per(nvb / kXcds)
    {
        unsigned xcc;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
        list = (int)(xcc & (kXcds - 1));
    }
    // Next virtual block, or -1 when every list is empty (lead lane only). A take
    // that finds its list empty sets the list's bit in q[9], which then names the
    // lists every workgroup has seen empty: the workgroup moves to one without a
    // bit, and leaves when all eight are set. Each list sends a workgroup on at
    // most once, so the loop ends.
    __device__ int take()
    {
        for (;;) {
            const int j = (int)atomicAdd(&q[list], 1u);
            if (j < per)
                return j * kXcds + list;
            const unsigned empty = atomicOr(&q[kXcds + 1], 1u << list) | (1u << list);
            if (empty == 0xffu)
                return -1;
            list = __ffs(~empty) - 1;
        }
    }
    __device__ void finish()
    {
        if (atomicAdd(&q[kXcds], 1u) == gridDim.x - 1)
            for (int i = 0; i < kQueueWords; ++i)
                atomicExch(&q[i], 0u);
    }
};

}  // namespace
}  // namespace fdtd
