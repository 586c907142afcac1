// Index arithmetic of the kernels that walk the dense staggered arrays plane by plane.
#pragma once

#include "fdtd_internal.h"

namespace fdtd {

constexpr int kPlaneBlock = 256, kPlaneUnroll = 4;

// Exact division of n < 2^31 by a fixed d >= 2: (mulhi(m, n) + n) >> s with s = ceil(log2 d) and
// m = floor(2^32 (2^s - d) / d) + 1 (Granlund and Montgomery, PLDI 1994, figure 4.1; the sum stays below
// 2^32 for such n).
struct FastDiv {
    unsigned m, s;
    __device__ __forceinline__ unsigned div(unsigned n) const { return (__umulhi(m, n) + n) >> s; }
};

inline FastDiv fast_div(unsigned d)
{
    FastDiv f{0, 0};
    while ((1ull << f.s) < d) ++f.s;
    f.m = (unsigned)(((1ull << 32) * ((1ull << f.s) - d)) / d + 1);
    return f;
}

// Row of an index into a plane of X columns, X = nx or nx + 1 (planes stay below 2^31 bytes).
struct PlaneIndex {
    FastDiv by[2];  // X = nx, nx + 1
    __device__ __forceinline__ unsigned row(unsigned q, int X, int nx) const { return by[X != nx].div(q); }
};

inline PlaneIndex plane_index(const Geom &g)
{
    return PlaneIndex{{fast_div((unsigned)g.nx), fast_div((unsigned)g.nx + 1)}};
}

// A workgroup's threads: runs of a plane by planes. Many planes of a few nodes (long thin cavities) share
// workgroups; with one each, most threads are idle (2x2x50000 FP32: unpack 131 us, 18 so; diagnostics 105 and 46;
// 4x4x20000 55 and 15, 58 and 41; 12x12x400 3.5 and 3.3). Fewer planes fill the chip as they are (10x10x200 2.9 us,
// shared 3.2; 16^3 2.6 and 3.1).
constexpr int kManyPlanes = 512;
inline dim3 plane_block(const Geom &g, int unroll)
{
    const long long n = (long long)(g.nx + 1) * (g.ny + 1);
    unsigned w = kPlaneBlock;
    while (g.nz >= kManyPlanes && w > 1 && (long long)(w / 2) * unroll >= n) w /= 2;
    return dim3(w, kPlaneBlock / w);
}

// Workgroups for every plane of nf components: runs of block.x * unroll elements, planes, components.
inline dim3 plane_grid(const Geom &g, int nf, int unroll)
{
    const dim3 b = plane_block(g, unroll);
    const long long n = (long long)(g.nx + 1) * (g.ny + 1), run = (long long)b.x * unroll;
    const unsigned groups = ((unsigned)g.nz + b.y) / b.y;  // of nz + 1 planes
    return dim3((unsigned)((n + run - 1) / run), groups < 65535 ? groups : 65535, (unsigned)nf);
}

// A thread's walk: threads of a run, planes at a time, the first plane, the distance to the next. Where a
// workgroup has one plane at a time (not THIN) all are uniform and in scalar registers (a seeded state of 128^3
// takes 29 us, 38 without).
template <bool THIN>
struct PlaneWalk {
    static __device__ __forceinline__ unsigned width() { return THIN ? blockDim.x : (unsigned)kPlaneBlock; }
    static __device__ __forceinline__ unsigned planes() { return THIN ? blockDim.y : 1u; }  // of a workgroup
    static __device__ __forceinline__ unsigned plane() { return THIN ? threadIdx.y : 0u; }  // a thread's among them
    static __device__ __forceinline__ int first() { return (int)(blockIdx.y * planes() + plane()); }
    // (unsigned: a signed step has the compiler prepare a loop that most threads run once)
    static __device__ __forceinline__ unsigned step() { return gridDim.y * planes(); }
};

// Calls launch(walk) with the walk of plane_block(g, unroll).
template <typename F>
void by_walk(const Geom &g, int unroll, F &&launch)
{
    if (plane_block(g, unroll).y > 1)
        launch(PlaneWalk<true>{});
    else
        launch(PlaneWalk<false>{});
}

}  // namespace fdtd
