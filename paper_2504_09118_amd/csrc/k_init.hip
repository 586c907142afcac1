// Seeded random initial state generated on the device.
//
// The cavity workloads start from a "random initial state" (Fig. 1b, Sec. 4)
// with PEC walls. E components are drawn from SplitMix64 (Steele, Lea and
// Flood, OOPSLA 2014) used counter-style: output c of seed s is
// mix64(s + (c + 1) * 0x9E3779B97F4A7C15 mod 2^64), u = (output >> 11) 2^-53,
// value 2u - 1 computed in FP64 and rounded once to the storage type (FP32
// first for 16-bit storage). The counter of component f (0, 1, 2 for Ex, Ey,
// Ez) at the x-fastest linear index l of its staggered array is (f << 40) + l.
// Wall-tangential E is 0 (PEC) and H = 0. Generating on the device avoids a
// host round trip when requests are admitted at a high rate.
#include "fdtd_internal.h"
#include "plane_index.h"
#include "storage.h"

namespace fdtd {
namespace {

constexpr int kBlock = kPlaneBlock;

__device__ __forceinline__ unsigned long long mix64(unsigned long long z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

template <typename T>
struct InitOut {
    T *a[6], *b[6];
    double scale[3];
};

// Component blockIdx.z, one thread per node of a plane (PlaneIndex), planes as plane_grid gives them.
template <typename T, typename Walk>
__global__ void __launch_bounds__(kBlock) k_init_random(Geom g, PlaneIndex ix, unsigned long long seed, InitOut<T> out)
{
    const int field = blockIdx.z;
    int X, Y, Z;
    extents(g, field, X, Y, Z);
    const unsigned n = (unsigned)X * (unsigned)Y, q = blockIdx.x * Walk::width() + threadIdx.x;
    if (q >= n)
        return;
    const int j = (int)ix.row(q, X, g.nx), i = (int)q - j * X;
    for (int k = Walk::first(); k < Z; k += Walk::step()) {
        const long long l = (long long)k * n + q;
        typename Store<T>::C v = 0;
        if (field < 3) {
            bool wall;
            if (field == 0)
                wall = j == 0 || j == g.ny || k == 0 || k == g.nz;
            else if (field == 1)
                wall = i == 0 || i == g.nx || k == 0 || k == g.nz;
            else
                wall = i == 0 || i == g.nx || j == 0 || j == g.ny;
            if (!wall) {
                const unsigned long long c = ((unsigned long long)field << 40) + (unsigned long long)l;
                const unsigned long long z = mix64(seed + (c + 1ull) * 0x9E3779B97F4A7C15ull);
                const double u = (double)(z >> 11) * 0x1.0p-53;
                v = to_compute<T>((2.0 * u - 1.0) * out.scale[field]);  // exact for scale 1
            }
        }
        const long long o = g.at(i, j, k);
        put_elem(out.a[field], g.lo_rec(field), o, v);
        if (out.b[field])
            put_elem(out.b[field], g.lo_rec(field), o, v);
    }
}

}  // namespace

template <typename T>
hipError_t launch_init_random(const Geom &g, unsigned long long seed, T *const a[6], T *const b[6], hipStream_t s,
                              const double *scale)
{
    InitOut<T> out;
    for (int f = 0; f < 6; ++f) {
        out.a[f] = a[f];
        out.b[f] = b[f];
    }
    for (int q = 0; q < 3; ++q) out.scale[q] = scale ? scale[q] : 1.0;
    by_walk(g, 1, [&](auto walk) {
        hipLaunchKernelGGL((k_init_random<T, decltype(walk)>), plane_grid(g, 6, 1), plane_block(g, 1), 0, s, g,
                           plane_index(g), seed, out);
    });
    return hipGetLastError();
}

template hipError_t launch_init_random<float>(const Geom &, unsigned long long, float *const[6], float *const[6],
                                              hipStream_t, const double *);
template hipError_t launch_init_random<double>(const Geom &, unsigned long long, double *const[6],
                                               double *const[6], hipStream_t, const double *);
template hipError_t launch_init_random<f16>(const Geom &, unsigned long long, f16 *const[6], f16 *const[6],
                                            hipStream_t, const double *);
template hipError_t launch_init_random<f16c>(const Geom &, unsigned long long, f16c *const[6], f16c *const[6],
                                             hipStream_t, const double *);
template hipError_t launch_init_random<bf16c>(const Geom &, unsigned long long, bf16c *const[6], bf16c *const[6],
                                              hipStream_t, const double *);
template hipError_t launch_init_random<bf16>(const Geom &, unsigned long long, bf16 *const[6], bf16 *const[6],
                                             hipStream_t, const double *);

}  // namespace fdtd
