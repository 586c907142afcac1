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

// Workgroups for every plane of nf components: runs of kPlaneBlock * unroll elements, planes, components.
inline dim3 plane_grid(const Geom &g, int nf, int unroll)
{
    const long long n = (long long)(g.nx + 1) * (g.ny + 1);
    const int planes = g.nz + 1;
    return dim3((unsigned)((n + (long long)kPlaneBlock * unroll - 1) / ((long long)kPlaneBlock * unroll)),
                (unsigned)(planes < 65535 ? planes : 65535), (unsigned)nf);
}

}  // namespace fdtd
