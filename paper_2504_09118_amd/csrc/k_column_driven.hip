// The driven column sweep: 1, 2 or 4 steps of the adjoint's forward and recompute passes in one launch. Each
// step adds the point source to its E node, the probes record E after it, and H^{n+1/2} of every step
// goes to its history slot; the state crosses memory once per launch.
// What bounds it: at 128^3 the history (25 MB per step written once) and a plane's chain of barriers;
// 200 steps with 2 probes take 3.9 ms, 27 us per single slab sweep before (5.4 ms). 48x40x56, 150 steps in
// narrow workgroups: 0.74 ms, in full ones 0.97, slab sweeps 2.1.
#include "column.h"

namespace fdtd {
namespace {

struct Drive : ColumnDrive {
    static constexpr bool on = true;
};

template <int TS, bool CH_ARR, int kNW>
__global__ void __launch_bounds__(64 * kNW, (kNW != kNarrowWaves ? 1 : driven_narrow_pairs(TS) ? 4 : 2))
    k_column_driven(Geom g, ColumnBoxes b, int kchunk, int ntx, int nty, int ntiles, int cpx, Drive drive)
{
    const int t = tile_of_block(blockIdx.x, ntiles, 2, cpx);
    if (t >= ntiles)
        return;  // the whole workgroup leaves before any barrier
    column_tile<float, TS, true, CH_ARR, kNW>(g, b, kchunk, ntx, nty, t % ntx, (t / ntx) % nty, t / (ntx * nty), drive);
}

// Full workgroups (12 waves where four stages, the coefficients and the drive do not fit 128 registers) or
// narrow ones, by the cost of a sweep as in the undriven step.
template <int TS>
hipError_t launch_driven(const Geom &g, const Fields<float> &src, const Fields<float> &dst, const Coefs<float> &c,
                         int zchunk, hipStream_t s, const Drive &drive)
{
    const int kchunk = (g.nz + zchunk - 1) / zchunk, nzc = (g.nz + kchunk - 1) / kchunk, cpx = cus_per_xcd();
    ColumnBoxes b;
    if (!column_boxes(src, dst, c, &b))
        return hipErrorInvalidValue;
    auto go = [&](auto kernel, int waves) {
        int ntx, nty;
        column_windows(g.nx, g.ny, TS, waves, &ntx, &nty);
        const int ntiles = ntx * nty * nzc, nblocks = (ntiles + kXcds - 1) / kXcds * kXcds;
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(64, waves), 0, s, g, b, kchunk, ntx, nty, ntiles, cpx, drive);
        return hipGetLastError();
    };
    auto pick = [&](auto ch) {
        constexpr bool CH = decltype(ch)::value;
        constexpr int wide = driven_waves_of(TS, CH);
        if (column_waves_for(g, TS, wide, driven_narrow_pairs(TS), nzc, kXcds * cpx) == kNarrowWaves)
            return go(k_column_driven<TS, CH, kNarrowWaves>, kNarrowWaves);
        return go(k_column_driven<TS, CH, wide>, wide);
    };
    return c.ch[0] ? pick(std::true_type{}) : pick(std::false_type{});
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
