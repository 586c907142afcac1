// The driven column sweep: 1, 2 or 4 steps of the adjoint's forward and recompute passes in one launch. Each
// step adds the point source to its E node, the probes record E after it, and H^{n+1/2} of every step
// goes to its history slot; the state crosses memory once per launch.
// What bounds it: at 128^3 the history (25 MB per step written once) and a plane's chain of barriers;
// 200 steps with 2 probes take 3.85 ms, 27 us per single slab sweep before (5.4 ms).
#include "column.h"

namespace fdtd {
namespace {

struct Drive : ColumnDrive {
    static constexpr bool on = true;
};

// 12 waves where four stages, the coefficients and the drive do not fit 128 registers.
template <int TS, bool CH_ARR>
constexpr int driven_waves()
{
    return driven_waves_of(TS, CH_ARR);
}

template <int TS, bool CH_ARR>
__global__ void __launch_bounds__((64 * driven_waves<TS, CH_ARR>()))
    k_column_driven(Geom g, ColumnBoxes b, int kchunk, int ntx, int nty, int ntiles, int cpx, Drive drive)
{
    const int t = tile_of_block(blockIdx.x, ntiles, 2, cpx);
    if (t >= ntiles)
        return;  // the whole workgroup leaves before any barrier
    column_tile<float, TS, true, CH_ARR, driven_waves<TS, CH_ARR>()>(g, b, kchunk, ntx, nty, t % ntx,
                                                                     (t / ntx) % nty, t / (ntx * nty), drive);
}

template <int TS>
hipError_t launch_driven(const Geom &g, const Fields<float> &src, const Fields<float> &dst, const Coefs<float> &c,
                         int zchunk, hipStream_t s, const Drive &drive)
{
    const bool cha = c.ch[0] != nullptr;
    const int kchunk = (g.nz + zchunk - 1) / zchunk, nzc = (g.nz + kchunk - 1) / kchunk;
    const int waves = driven_waves_of(TS, cha);
    int ntx, nty;
    column_windows(g.nx, g.ny, TS, waves, &ntx, &nty);
    const int ntiles = ntx * nty * nzc, nblocks = (ntiles + kXcds - 1) / kXcds * kXcds;
    const dim3 block(64, waves), grid(nblocks);
    ColumnBoxes b;
    if (!column_boxes(src, dst, c, &b))
        return hipErrorInvalidValue;
    if (cha)
        hipLaunchKernelGGL((k_column_driven<TS, true>), grid, block, 0, s, g, b, kchunk, ntx, nty, ntiles,
                           cus_per_xcd(), drive);
    else
        hipLaunchKernelGGL((k_column_driven<TS, false>), grid, block, 0, s, g, b, kchunk, ntx, nty, ntiles,
                           cus_per_xcd(), drive);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_column_driven(const Geom &g, const Fields<float> &src, const Fields<float> &dst, const Coefs<float> &c,
                                int zchunk, int ts, hipStream_t s, const ColumnDrive &cd)
{
    if (!c.ce[0])
        return hipErrorInvalidValue;
    Drive drive;
    static_cast<ColumnDrive &>(drive) = cd;
    zchunk = zchunk < 1 ? 1 : zchunk;
    switch (ts) {
    case 1: return launch_driven<1>(g, src, dst, c, zchunk, s, drive);
    case 2: return launch_driven<2>(g, src, dst, c, zchunk, s, drive);
    case 4: return launch_driven<4>(g, src, dst, c, zchunk, s, drive);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fdtd
