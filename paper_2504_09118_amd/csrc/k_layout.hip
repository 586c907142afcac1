// Layout conversion and the FP64 coefficient precompute.
//
//   pack    dense staggered array (host layout) -> padded device box, with the
//           PEC boundary (Fig. 1b caption, Sec. 4: tangential E = 0 on walls)
//   unpack  padded device box -> dense staggered array
//   coef    per-node Ce = dt/(dx * eps_edge), Ch = dt/(dx * mu_face) in FP64,
//           rounded once to the storage type (Eq. 2 coefficients dt/eps and
//           dt/mu with the cubic-cell 1/dx folded in)
#include "fdtd_internal.h"
#include "plane_index.h"
#include "storage.h"

namespace fdtd {
namespace {

constexpr int kBlock = kPlaneBlock;

__device__ __forceinline__ bool e_wall(int field, int i, int j, int k, int nx, int ny, int nz)
{
    switch (field) {
    case 0: return j == 0 || j == ny || k == 0 || k == nz;
    case 1: return i == 0 || i == nx || k == 0 || k == nz;
    case 2: return i == 0 || i == nx || j == 0 || j == ny;
    default: return false;
    }
}

// Wall-normal H node: its update reads only wall-tangential E, so it never changes.
__device__ __forceinline__ bool h_wall_normal(int field, int i, int j, int k, int nx, int ny, int nz)
{
    switch (field) {
    case 3: return i == 0 || i == nx;
    case 4: return j == 0 || j == ny;
    case 5: return k == 0 || k == nz;
    default: return false;
    }
}

// The components a launch converts: component f0 + blockIdx.z, its dense array and its box (pack: both
// state buffers' boxes, the second may be null).
template <typename S, typename T>
struct Boxes {
    S *dense[6];
    T *box[6], *box2[6];
    double scale[3];
};

// A plane of a component is contiguous in the dense array, so a workgroup takes a run of it: one launch
// for all components, an index by 32-bit multiplication instead of 64-bit divisions per element.
// Bound by HBM: 512^3 FP32, six components: unpack 1.12 ms (6.45 GB: 5.8 TB/s), pack 1.94 ms (9.7 GB,
// 5.0 TB/s), from 2.37 and 3.0 ms with a launch per component and 64-bit divisions per element; 16^3:
// one launch instead of six (4 us each).
// SCALED: rectangular cells; the cubic scale is exactly 1.
template <typename S, typename T, bool SCALED, typename Walk>
__global__ void __launch_bounds__(kBlock) k_pack(Geom g, PlaneIndex ix, Boxes<const S, T> b, int f0)
{
    const int f = f0 + blockIdx.z;
    int X, Y, Z;
    extents(g, f, X, Y, Z);
    const unsigned n = (unsigned)X * (unsigned)Y;
    const double scale = b.scale[f % 3];
    for (int k = Walk::first(); k < Z; k += Walk::step()) {
        const S *src = b.dense[f] + (long long)k * n;
        const long long ok = (long long)k * g.plane;
        // every load before the first store, which the compiler may not move them over
        S in[kPlaneUnroll];
#pragma unroll
        for (int u = 0; u < kPlaneUnroll; ++u) {
            const unsigned q = (blockIdx.x * kPlaneUnroll + u) * Walk::width() + threadIdx.x;
            if (q >= n)
                break;
            in[u] = src[q];
        }
#pragma unroll
        for (int u = 0; u < kPlaneUnroll; ++u) {
            const unsigned q = (blockIdx.x * kPlaneUnroll + u) * Walk::width() + threadIdx.x;
            if (q >= n)
                break;
            const int j = (int)ix.row(q, X, g.nx), i = (int)q - j * X;
            // scaled in FP64; 16-bit storage: rounded to FP32, then to the 16-bit type
            typename Store<T>::C v = to_compute<T>(SCALED ? (double)in[u] * scale : (double)in[u]);
            if (e_wall(f, i, j, k, g.nx, g.ny, g.nz))
                v = 0;
            // a wall-normal H of -0 is stored as +0 (equal values): sweeps that add the zero curl to
            // every H node then keep every bit
            if (h_wall_normal(f, i, j, k, g.nx, g.ny, g.nz) && v == 0)
                v = 0;
            const long long o = ok + (long long)(i + g.px * j);
            put_elem(b.box[f], g.lo_rec(f), o, v);
            if (b.box2[f])
                put_elem(b.box2[f], g.lo_rec(f), o, v);
        }
    }
}

template <typename T, typename S, bool SCALED, typename Walk>
__global__ void __launch_bounds__(kBlock) k_unpack(Geom g, PlaneIndex ix, Boxes<S, const T> b, int f0)
{
    const int f = f0 + blockIdx.z;
    int X, Y, Z;
    extents(g, f, X, Y, Z);
    const unsigned n = (unsigned)X * (unsigned)Y;
    const double scale = b.scale[f % 3];
    for (int k = Walk::first(); k < Z; k += Walk::step()) {
        S *dst = b.dense[f] + (long long)k * n;
        const long long ok = (long long)k * g.plane;
        typename Store<T>::C v[kPlaneUnroll];
#pragma unroll
        for (int u = 0; u < kPlaneUnroll; ++u) {
            const unsigned q = (blockIdx.x * kPlaneUnroll + u) * Walk::width() + threadIdx.x;
            if (q >= n)
                break;
            const int j = (int)ix.row(q, X, g.nx), i = (int)q - j * X;
            v[u] = get_elem(b.box[f], g.lo_rec(f), ok + (long long)(i + g.px * j));
        }
#pragma unroll
        for (int u = 0; u < kPlaneUnroll; ++u) {
            const unsigned q = (blockIdx.x * kPlaneUnroll + u) * Walk::width() + threadIdx.x;
            if (q < n)
                dst[q] = SCALED ? (S)((double)v[u] / scale) : (S)v[u];
        }
    }
}

__device__ __forceinline__ double mat(const double *m, int nx, int ny, int i, int j, int k)
{
    return m ? m[(long long)i + (long long)nx * ((long long)j + (long long)ny * k)] : 1.0;
}

struct CoefOut {
    void *out[6];
    double fac[6];
};

// One thread per node of component f0 + blockIdx.z (0..2 E edges, 3..5 H faces).
template <typename T, typename Walk>
__global__ void __launch_bounds__(kBlock) k_coef(Geom g, PlaneIndex ix, int f0, double dx, double dt,
                                                 const double *__restrict__ m, CoefOut co)
{
    const int field = f0 + blockIdx.z;
    int X, Y, Z;
    extents(g, field, X, Y, Z);
    const unsigned q = blockIdx.x * Walk::width() + threadIdx.x;
    if (q >= (unsigned)X * (unsigned)Y)
        return;
    const int j = (int)ix.row(q, X, g.nx), i = (int)q - j * X;
    for (int k = Walk::first(); k < Z; k += Walk::step()) {
        const int nx = g.nx, ny = g.ny, nz = g.nz;
        double c = 0.0;
        switch (field) {
        case 0:  // x-edge: cells (i, j-1..j, k-1..k)
            if (j > 0 && j < ny && k > 0 && k < nz) {
                double a = (mat(m, nx, ny, i, j - 1, k - 1) + mat(m, nx, ny, i, j, k - 1)) +
                           (mat(m, nx, ny, i, j - 1, k) + mat(m, nx, ny, i, j, k));
                c = dt / (dx * (a * 0.25));
            }
            break;
        case 1:  // y-edge: cells (i-1..i, j, k-1..k)
            if (i > 0 && i < nx && k > 0 && k < nz) {
                double a = (mat(m, nx, ny, i - 1, j, k - 1) + mat(m, nx, ny, i - 1, j, k)) +
                           (mat(m, nx, ny, i, j, k - 1) + mat(m, nx, ny, i, j, k));
                c = dt / (dx * (a * 0.25));
            }
            break;
        case 2:  // z-edge: cells (i-1..i, j-1..j, k)
            if (i > 0 && i < nx && j > 0 && j < ny) {
                double a = (mat(m, nx, ny, i - 1, j - 1, k) + mat(m, nx, ny, i, j - 1, k)) +
                           (mat(m, nx, ny, i - 1, j, k) + mat(m, nx, ny, i, j, k));
                c = dt / (dx * (a * 0.25));
            }
            break;
        case 3:  // x-face between cells (i-1, j, k) and (i, j, k)
            if (i > 0 && i < nx)
                c = dt / (dx * ((mat(m, nx, ny, i - 1, j, k) + mat(m, nx, ny, i, j, k)) * 0.5));
            break;
        case 4:
            if (j > 0 && j < ny)
                c = dt / (dx * ((mat(m, nx, ny, i, j - 1, k) + mat(m, nx, ny, i, j, k)) * 0.5));
            break;
        default:
            if (k > 0 && k < nz)
                c = dt / (dx * ((mat(m, nx, ny, i, j, k - 1) + mat(m, nx, ny, i, j, k)) * 0.5));
            break;
        }
        ((T *)co.out[field])[g.at(i, j, k)] = (T)(c * co.fac[field]);  // exact for factor 1; one rounding
    }
}

}  // namespace

template <typename S, typename T>
hipError_t launch_pack(const Geom &g, int f0, int nf, const S *const *src, T *const *dst, T *const *dst2, hipStream_t s,
                       const double *scale)
{
    Boxes<const S, T> b{};
    for (int f = f0; f < f0 + nf; ++f) {
        b.dense[f] = src[f];
        b.box[f] = dst[f];
        b.box2[f] = dst2 ? dst2[f] : nullptr;
    }
    const bool scaled = scale && (scale[0] != 1.0 || scale[1] != 1.0 || scale[2] != 1.0);
    for (int a = 0; a < 3; ++a) b.scale[a] = scale ? scale[a] : 1.0;
    const dim3 grid = plane_grid(g, nf, kPlaneUnroll), block = plane_block(g, kPlaneUnroll);
    by_walk(g, kPlaneUnroll, [&](auto walk) {
        if (scaled)
            hipLaunchKernelGGL((k_pack<S, T, true, decltype(walk)>), grid, block, 0, s, g, plane_index(g), b, f0);
        else
            hipLaunchKernelGGL((k_pack<S, T, false, decltype(walk)>), grid, block, 0, s, g, plane_index(g), b, f0);
    });
    return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_unpack(const Geom &g, int f0, int nf, const T *const *src, S *const *dst, hipStream_t s,
                         const double *scale)
{
    Boxes<S, const T> b{};
    for (int f = f0; f < f0 + nf; ++f) {
        b.dense[f] = dst[f];
        b.box[f] = src[f];
    }
    const bool scaled = scale && (scale[0] != 1.0 || scale[1] != 1.0 || scale[2] != 1.0);
    for (int a = 0; a < 3; ++a) b.scale[a] = scale ? scale[a] : 1.0;
    const dim3 grid = plane_grid(g, nf, kPlaneUnroll), block = plane_block(g, kPlaneUnroll);
    by_walk(g, kPlaneUnroll, [&](auto walk) {
        if (scaled)
            hipLaunchKernelGGL((k_unpack<T, S, true, decltype(walk)>), grid, block, 0, s, g, plane_index(g), b, f0);
        else
            hipLaunchKernelGGL((k_unpack<T, S, false, decltype(walk)>), grid, block, 0, s, g, plane_index(g), b, f0);
    });
    return hipGetLastError();
}

template <typename T>
hipError_t launch_coef(const Geom &g, double dx, double dt, const double *eps, const double *mu, T *ce[3],
                       T *ch[3], hipStream_t s, const double *fac)
{
    CoefOut co;
    for (int f = 0; f < 6; ++f) {
        co.out[f] = f < 3 ? ce[f] : ch[f - 3];
        co.fac[f] = fac ? fac[f] : 1.0;
    }
    for (int f0 = 0; f0 < 6; f0 += 3) {
        if (!co.out[f0])
            continue;
        by_walk(g, 1, [&](auto walk) {
            hipLaunchKernelGGL((k_coef<T, decltype(walk)>), plane_grid(g, 3, 1), plane_block(g, 1), 0, s, g,
                               plane_index(g), f0, dx, dt, f0 == 0 ? eps : mu, co);
        });
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

#define FDTD_LAYOUT(S, T)                                                                                            \
    template hipError_t launch_pack<S, T>(const Geom &, int, int, const S *const *, T *const *, T *const *,          \
                                          hipStream_t, const double *);                                             \
    template hipError_t launch_unpack<T, S>(const Geom &, int, int, const T *const *, S *const *, hipStream_t,      \
                                            const double *);
FDTD_LAYOUT(float, float)
FDTD_LAYOUT(double, float)
FDTD_LAYOUT(float, double)
FDTD_LAYOUT(double, double)
FDTD_LAYOUT(float, f16)
FDTD_LAYOUT(double, f16)
FDTD_LAYOUT(float, bf16)
FDTD_LAYOUT(double, bf16)
FDTD_LAYOUT(float, f16c)
FDTD_LAYOUT(double, f16c)
FDTD_LAYOUT(float, bf16c)
FDTD_LAYOUT(double, bf16c)
#undef FDTD_LAYOUT
template hipError_t launch_coef<float>(const Geom &, double, double, const double *, const double *, float *[3],
                                       float *[3], hipStream_t, const double *);
template hipError_t launch_coef<double>(const Geom &, double, double, const double *, const double *,
                                        double *[3], double *[3], hipStream_t, const double *);

}  // namespace fdtd
