// FP64 diagnostics of a stored state (E^n, H^{n-1/2}), off the timed path.
//
//   W       = sum_E E^2/Ce + sum_H H^{n-1/2} H^{n+1/2} / Ch   (H^{n+1/2} formed
//             here in FP64 from the stored E and H); the leapfrog of Eq. 2
//             conserves it exactly in exact arithmetic because the E curl is
//             minus the transpose of the H curl
//   sum E^2, sum H^2, max |div (H/Ch)| per cell, max |tangential E| on the
//   PEC walls, count of non-finite values.
// A fixed grid of workgroups walks the nodes in a fixed order, so the sums
// do not depend on scheduling.
#include "fdtd_internal.h"
#include "plane_index.h"
#include "storage.h"

namespace fdtd {
namespace {

constexpr int kBlock = kPlaneBlock;
constexpr int kGrid = 1024;
constexpr int kQ = 6;  // W, sumE2, sumH2, maxdivB, maxEtan, nonfinite

__device__ __forceinline__ bool e_tan(int f, int i, int j, int k, int nx, int ny, int nz)
{
    if (f == 0) return j == 0 || j == ny || k == 0 || k == nz;
    if (f == 1) return i == 0 || i == nx || k == 0 || k == nz;
    return i == 0 || i == nx || j == 0 || j == ny;
}

__device__ __forceinline__ bool h_normal(int f, int i, int j, int k, int nx, int ny, int nz)
{
    if (f == 3) return i == 0 || i == nx;
    if (f == 4) return j == 0 || j == ny;
    return k == 0 || k == nz;
}

template <typename T>
__device__ __forceinline__ double coef_at(const T *arr, T s, long long o)
{
    return arr ? (double)arr[o] : (double)s;
}

template <typename T>
__device__ __forceinline__ double val(const T *a, long long o, long long lo_off)
{
    return (double)get_elem(a, lo_off, o);
}

// Sums the workgroup's values over its threads, in red[][0].
__device__ __forceinline__ void reduce(double (*red)[kBlock], const double *v)
{
    const int t = threadIdx.y * blockDim.x + threadIdx.x;
    for (int q = 0; q < kQ; ++q) red[q][t] = v[q];
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if (t < s) {
            for (int q = 0; q < 3; ++q) red[q][t] += red[q][t + s];
            red[3][t] = fmax(red[3][t], red[3][t + s]);
            red[4][t] = fmax(red[4][t], red[4][t + s]);
            red[5][t] += red[5][t + s];
        }
        __syncthreads();
    }
}

// Workgroup b walks the runs b, b + kGrid, ... of kBlock nodes within a plane, or within a few small planes
// (the index of a run is uniform, a node's row comes from a multiplication). What bounds it: the latency of a
// run's loads, which are all in flight at once, and twelve FP64 divisions a node. 133 x 40 x 71, both media: 11.5 us, 22.4 with
// each load behind the test that needs it; 256^3 with the second kernel and the copy 244 us, 685 before. A
// second small kernel adds up the partial results: doing that in the workgroup that finishes last needs a
// fence in each of the 1024, and took 92 us when the two kernels took 28.
template <typename T, typename Walk>
__global__ void __launch_bounds__(kBlock)
    k_diag(Geom g, PlaneIndex ix, Fields<T> f, Coefs<typename Store<T>::C> c, double *partial)
{
    __shared__ double red[kQ][kBlock];
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int X = nx + 1;
    const unsigned n = (unsigned)X * (unsigned)(ny + 1);
    const unsigned runs = (n + Walk::width() - 1) / Walk::width();             // of one plane
    const unsigned groups = ((unsigned)nz + Walk::planes()) / Walk::planes();  // of the nz + 1 planes
    const long long P = g.plane;
    const int px = g.px;
    double w = 0, se = 0, sh = 0, mdiv = 0, mtan = 0, bad = 0;
    for (unsigned long long item = blockIdx.x; item < (unsigned long long)runs * groups; item += kGrid) {
        const unsigned z = (unsigned)(item / runs);
        const int k = (int)(z * Walk::planes() + Walk::plane());
        const unsigned q0 = (unsigned)(item - (unsigned long long)z * runs) * Walk::width() + threadIdx.x;
        if (q0 >= n || (Walk::planes() > 1 && k > nz))
            continue;
        const int j = (int)ix.row(q0, X, nx), i = (int)q0 - j * X;
        const long long o = g.at(i, j, k);
        // every value that the node may need, before the first that depends on one: a load behind each of
        // the tests below is a memory latency of its own (at a far wall a neighbour is the node itself)
        const long long ox = o + (i < nx), oy = o + (j < ny ? px : 0), oz = o + (k < nz ? P : 0);
        double v[6], ce[3], ch[3], chn[3];
#pragma unroll
        for (int q = 0; q < 6; ++q) v[q] = val(f.f[q], o, g.lo_rec(q));
        const double exy = val(f.f[0], oy, g.lo_rec(0)), exz = val(f.f[0], oz, g.lo_rec(0)),
                     eyx = val(f.f[1], ox, g.lo_rec(1)), eyz = val(f.f[1], oz, g.lo_rec(1)),
                     ezx = val(f.f[2], ox, g.lo_rec(2)), ezy = val(f.f[2], oy, g.lo_rec(2));
        const double hn1[3] = {val(f.f[3], ox, g.lo_rec(3)), val(f.f[4], oy, g.lo_rec(4)),
                               val(f.f[5], oz, g.lo_rec(5))};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            ce[q] = coef_at(c.ce[q], c.ce_s, o);
            ch[q] = coef_at(c.ch[q], c.ch_s, o);
            chn[q] = coef_at(c.ch[q], c.ch_s, q == 0 ? ox : q == 1 ? oy : oz);
        }
        bool ex[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            int a, b, d;
            extents(g, q, a, b, d);
            ex[q] = i < a && j < b && k < d;
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (!ex[q]) continue;
            const double e = v[q];
            if (!isfinite(e)) bad += 1;
            se += e * e;
            const bool wall = e_tan(q, i, j, k, nx, ny, nz);
            if (wall) {
                mtan = fmax(mtan, fabs(e));
            } else if (ce[q] != 0.0) {
                w += e * e / ce[q];
            }
        }
        const double Ex0 = ex[0] ? v[0] : 0.0, Ey0 = ex[1] ? v[1] : 0.0, Ez0 = ex[2] ? v[2] : 0.0;
        const double curl[3] = {(eyz - Ey0) - (ezy - Ez0), (ezx - Ez0) - (exz - Ex0), (exy - Ex0) - (eyx - Ey0)};
#pragma unroll
        for (int q = 3; q < 6; ++q) {
            if (!ex[q]) continue;
            const double h = v[q];
            if (!isfinite(h)) bad += 1;
            sh += h * h;
            if (h_normal(q, i, j, k, nx, ny, nz)) continue;
            if (ch[q - 3] == 0.0) continue;
            const double hn = h + ch[q - 3] * curl[q - 3];
            w += h * hn / ch[q - 3];
        }
        if (i < nx && j < ny && k < nz) {
            // B = H/Ch, taken as 0 on wall-normal nodes (constant in time)
            auto b = [&](bool normal, double h, double coef) { return !normal && coef != 0.0 ? h / coef : 0.0; };
            const double dv = (b(i + 1 == nx, hn1[0], chn[0]) - b(i == 0, v[3], ch[0])) +
                              (b(j + 1 == ny, hn1[1], chn[1]) - b(j == 0, v[4], ch[1])) +
                              (b(k + 1 == nz, hn1[2], chn[2]) - b(k == 0, v[5], ch[2]));
            mdiv = fmax(mdiv, fabs(dv));
        }
    }
    const double own[kQ] = {w, se, sh, mdiv, mtan, bad};
    reduce(red, own);
    const unsigned t = threadIdx.y * blockDim.x + threadIdx.x;
    if (t < kQ)
        partial[(long long)blockIdx.x * kQ + t] = red[t][0];
}

__global__ void __launch_bounds__(kBlock) k_diag_final(const double *partial, double *out)
{
    __shared__ double red[kQ][kBlock];
    double acc[kQ] = {0, 0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < kGrid; b += kBlock) {
        for (int q = 0; q < 3; ++q) acc[q] += partial[b * kQ + q];
        acc[3] = fmax(acc[3], partial[b * kQ + 3]);
        acc[4] = fmax(acc[4], partial[b * kQ + 4]);
        acc[5] += partial[b * kQ + 5];
    }
    reduce(red, acc);
    if (threadIdx.x < kQ)
        out[threadIdx.x] = red[threadIdx.x][0];
}

}  // namespace

size_t diag_partial_doubles() { return (size_t)kGrid * kQ; }

template <typename T>
hipError_t launch_diag(const Geom &g, const Fields<T> &f, const Coefs<typename Store<T>::C> &c, double *partial,
                       double *out_dev, hipStream_t s)
{
    by_walk(g, 1, [&](auto walk) {
        hipLaunchKernelGGL((k_diag<T, decltype(walk)>), dim3(kGrid), plane_block(g, 1), 0, s, g, plane_index(g), f, c,
                           partial);
    });
    hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(kBlock), 0, s, partial, out_dev);
    return hipGetLastError();
}

template hipError_t launch_diag<float>(const Geom &, const Fields<float> &, const Coefs<float> &, double *,
                                       double *, hipStream_t);
template hipError_t launch_diag<double>(const Geom &, const Fields<double> &, const Coefs<double> &, double *,
                                        double *, hipStream_t);
template hipError_t launch_diag<f16>(const Geom &, const Fields<f16> &, const Coefs<float> &, double *, double *,
                                     hipStream_t);
template hipError_t launch_diag<f16c>(const Geom &, const Fields<f16c> &, const Coefs<float> &, double *,
                                      double *, hipStream_t);
template hipError_t launch_diag<bf16c>(const Geom &, const Fields<bf16c> &, const Coefs<float> &, double *,
                                       double *, hipStream_t);
template hipError_t launch_diag<bf16>(const Geom &, const Fields<bf16> &, const Coefs<float> &, double *, double *,
                                      hipStream_t);

}  // namespace fdtd
