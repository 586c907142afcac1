// Column form of the temporal sweep: TS full leapfrog steps per pass over memory with the stages,
// the plane lag between them and the arithmetic of k_temporal.hip, hence the same bits, but another
// split of the tile.
//
// A workgroup's window is 64 columns x 32 rows, 24 or 16 where it has 12 or 8 waves. A lane holds one
// column of kNR rows, a wave kNR whole rows of the window, so
//   - the x neighbours of a cell are in the next lanes of the same wave: the differences read them
//     by a wave shift inside the subtraction (a DPP operand), without LDS and without an extra
//     instruction; a lane at the window's edge reads 0 there;
//   - of the y neighbours only one row per wave comes from another wave: (Ex, Ez) of a wave's first
//     row and (Hx, Hz) of its last row pass through LDS, 8 bytes written and read per lane and
//     update;
//   - the E input of each stage is staged for the next plane as soon as it is known (two buffers, by
//     plane parity), so a plane takes TS barriers, and a tile clears only the rows beside its window.
// Own cells are the window less a halo of TS rows and columns on every side that has a neighbour;
// the outermost windows own up to the walls.
//
// What bounds it: neither HBM nor the matrix cores (there is no contraction). On a 128^3 cavity with
// per-node Ce (a state the 256 MB last-level cache holds) a 4-step sweep takes 48 us: 15 planes of
// about 2.8 us, in which the vector units are 40 % busy, the barriers and the chain of dependent
// stages taking the rest; it moves 200 MB past L2, where that cache delivers 11 TB/s (18 us). The form
// of k_temporal.hip, whose cells exchange 52 bytes a stage through LDS where these exchange 16, takes
// 68 us on the same sweep. 64^3: 18 us (58). 16-bit storage, 128^3: FP16 44 us (61), BF16 with
// residuals 59 us (79). Per-node Ce and Ch, 160 x 96 x 128, 3 steps: 42 us (61).
// Larger states keep the other form: there the sweep is bound by what memory serves, and windows whose
// own cells do not end on 128-byte lines make two workgroups write parts of one line (512^3: 2.65 ms
// against 2.08; BF16 with residuals 320^3 0.63 against 0.55, FP16 0.46 and 0.41; FP16 at 394x301x350, whose
// rows and planes divide badly among the other form's tiles, 0.60 and 0.65).
#pragma once

#include <algorithm>

#include <type_traits>

#include "column_lanes.h"
#include "fdtd_internal.h"
#include "storage.h"
#include "tile_queue.h"
#include "yee_update.h"

namespace fdtd {
namespace {

constexpr int kNR = kColumnRows;  // rows per lane
constexpr int kCols = 64;

// Waves of a workgroup: 16 of 128 registers where the rings fit (FP32 with one coefficient array: 51
// values a row at 4 stages), else 12 of 168, or 8 of 256. A spilled register inside the plane loop costs
// more than the smaller window, because its reload waits for every load issued before it (Ce and Ch, 3
// stages: 72 us with 16 waves and 20 spills, 43 us with 12).
template <typename S, int TS, bool CE_ARR, bool CH_ARR>
constexpr int column_waves()
{
    return column_waves_of(sizeof(S) == 2, TS, CE_ARR, CH_ARR);
}

// What a driven sweep does beside its steps; an undriven one carries nothing.
struct NoDrive {
    static constexpr bool on = false;
};

// The boxes of an undriven sweep, a pointer each, with ColumnBoxes' accessors (as base and distance they
// cost the sweep two address additions more per box and plane).
template <typename S>
struct FieldBoxes {
    Fields<S> src, dst;
    Coefs<float> c;
    static constexpr long long step = 0;
    __device__ __forceinline__ const S *read_e(long long, int q) const { return src.f[q]; }
    __device__ __forceinline__ const S *read_h(long long, int q) const { return src.f[3 + q]; }
    __device__ __forceinline__ S *write_e(long long, int q) const { return dst.f[q]; }
    __device__ __forceinline__ S *write_h(long long, int q) const { return dst.f[3 + q]; }
    __device__ __forceinline__ const float *read_ce(long long, int q) const { return c.ce[q]; }
    __device__ __forceinline__ const float *read_ch(long long, int q) const { return c.ch[q]; }
    __device__ __forceinline__ float scalar_ce() const { return c.ce_s; }
    __device__ __forceinline__ float scalar_ch() const { return c.ch_s; }
};

template <typename S, int TS, bool CE_ARR, bool CH_ARR, int kNW, typename Boxes, typename Drive>
__device__ __forceinline__ void column_tile(const Geom &g, const Boxes &b, int kchunk, int ntx, int nty,
                                            int tile_x, int tile_y, int zc, const Drive &drive)
{
    constexpr int kRows = kNR * kNW;
    typedef float f2 __attribute__((ext_vector_type(2)));
    constexpr bool H16 = sizeof(S) == 2, COMP = Store<S>::comp;
    static_assert(kNR == 2 || !H16, "16-bit fields are converted in pairs of rows");
    __shared__ __attribute__((aligned(16))) f2 sE[2][TS][kNW + 1][kCols];  // (Ex, Ez) of each wave's first row
    __shared__ __attribute__((aligned(16))) f2 sH[TS][kNW + 1][kCols];     // (Hx, Hz) of the last row of wave w - 1

    const int nx = g.nx, ny = g.ny, nz = g.nz, px = g.px;
    const long long P = g.plane;
    const int kb = zc * kchunk, ke = min(nz, kb + kchunk);
    const int lane = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int i = tile_x * (kCols - 2 * TS) + lane;
    const int row0 = wave * kNR, j0 = tile_y * (kRows - 2 * TS) + row0;  // first row of the wave
    const bool col_own = i < nx && (lane >= TS || tile_x == 0) && (lane < kCols - TS || tile_x == ntx - 1);
    const bool wall_x = i < 1 || i >= nx;

    // the rows beside the window, which its outermost rows read: never written
    if (wave == 0) {
        const f2 z = {0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < TS; ++s) {
            sE[0][s][kNW][lane] = z;
            sE[1][s][kNW][lane] = z;
            sH[s][0][lane] = z;
        }
    }

    // byte offsets of the lane's cells in a plane of 4-byte elements (16-bit fields: half of it; half of
    // kDrop is past every plane of 2-byte elements as well), and which of them the tile stores
    unsigned vc[kNR];
    bool own[kNR];
#pragma unroll
    for (int r = 0; r < kNR; ++r) {
        const int j = j0 + r, lr = row0 + r;
        const bool in = i < nx && j < ny;
        own[r] = in && col_own && (lr >= TS || tile_y == 0) && (lr < kRows - TS || tile_y == nty - 1);
        vc[r] = in ? (unsigned)(i + px * j) * 4u : kDrop;
    }

    // driven: whether this wave holds the source node (own or halo: every copy of it is driven), and which
    // probes lie in its rows and planes
    bool has_source = false;
    unsigned long long probes = 0;
    int source_plane = 0;
    if constexpr (Drive::on) {
        const auto *t = constant(drive.tab);
        source_plane = t->sk;
        has_source = t->sf >= 0 && t->sj >= j0 && t->sj < j0 + kNR && t->si >= i - lane && t->si < i - lane + kCols;
        const bool here = drive.rec && lane < t->np && t->pj[lane] >= j0 && t->pj[lane] < j0 + kNR &&
                          t->pi[lane] >= i - lane && t->pi[lane] < i - lane + kCols && t->pk[lane] >= kb &&
                          t->pk[lane] < ke;
        probes = __ballot(here);
    }

    // Register rings as in k_temporal.hip: role r at phase ph is slot (r + off + ph) mod M, and the plane
    // loop is unrolled M times, so that a value passes to the next stage by a change of name.
    //   E roles: -2 (E prefetched for plane k+2), -1 (E^n at p_1 + 1), s = 0..TS-1 (E of stage s at p_s);
    //   H roles: -1 (H prefetched for plane k+1), s (H of stage s), TS (the last stage's, one plane down);
    //   coefficients: -1 (prefetched), s.
    // 16-bit fields are prefetched as loaded bits and decoded at the top of the plane that uses them.
    constexpr int M = TS + 2;
    float RE[M][3][kNR], RH[M][3][kNR], RC[M][3][kNR], RK[M][3][kNR];
    unsigned short qe[3][kNR], qh[3][kNR];
    unsigned qre[kNR], qrh[kNR];  // 16-bit: E(k+1), H(k), their residual records
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int r = 0; r < kNR; ++r) {
                RE[m][q][r] = 0.0f;
                RH[m][q][r] = 0.0f;
                RC[m][q][r] = CE_ARR ? 0.0f : b.scalar_ce();
                RK[m][q][r] = CH_ARR ? 0.0f : b.scalar_ch();
            }
#define ES(r, ph) ring_slot(r, ph, 2, M)
#define HS(r, ph) ring_slot(r, ph, 1, M)
    const int k0 = max(0, kb - TS), kend = ke + TS - 2;
    const unsigned fbytes = (unsigned)(P * (long long)sizeof(S)), cbytes = (unsigned)(P * 4);

    auto load32 = [&](float *out, const void *p, unsigned n) {
        const __amdgpu_buffer_rsrc_t d = plane_rsrc(p, n);
#pragma unroll
        for (int r = 0; r < kNR; ++r)
            out[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(d, vc[r], 0, 0));
    };
    auto load16 = [&](unsigned short *out, const void *p, unsigned n) {
        const __amdgpu_buffer_rsrc_t d = plane_rsrc(p, n);
#pragma unroll
        for (int r = 0; r < kNR; ++r)
            out[r] = __builtin_amdgcn_raw_buffer_load_b16(d, vc[r] >> 1, 0, 0);
    };
    auto load_rec = [&](unsigned *out, const S *base, long long pk, unsigned n) {
        const __amdgpu_buffer_rsrc_t d = plane_rsrc((const char *)base + g.lo_off + kRecBytes * pk, n);
#pragma unroll
        for (int r = 0; r < kNR; ++r) out[r] = __builtin_amdgcn_raw_buffer_load_b32(d, vc[r], 0, 0);
    };
    // three components of two rows from loaded bits and residual records
    auto decode = [&](float (*out)[kNR], unsigned short (*q)[kNR], unsigned *w) {
        if constexpr (COMP) {
            Store<S>::template dec2r<0>((unsigned)q[0][0] | ((unsigned)q[0][1] << 16), w[0], w[1], out[0][0], out[0][1]);
            Store<S>::template dec2r<1>((unsigned)q[1][0] | ((unsigned)q[1][1] << 16), w[0], w[1], out[1][0], out[1][1]);
            Store<S>::template dec2r<2>((unsigned)q[2][0] | ((unsigned)q[2][1] << 16), w[0], w[1], out[2][0], out[2][1]);
        } else if constexpr (H16) {
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int r = 0; r < kNR; ++r) {
                    const unsigned short u = q[p][r];
                    S v;
                    __builtin_memcpy(&v, &u, 2);
                    out[p][r] = Store<S>::widen(v);
                }
        }
    };
    {
        const long long pk = (long long)k0 * P;
        const bool up = k0 + 1 < nz;
        const long long pk1 = up ? pk + P : 0;
        const unsigned nf = up ? fbytes : 0u, nc = up ? cbytes : 0u;
        if constexpr (H16) {
            for (int q = 0; q < 3; ++q) load16(qe[q], b.read_e(b.step, q) + pk, fbytes);
            if (COMP)
                load_rec(qre, b.read_e(b.step, 0), pk, cbytes);
            decode(RE[ES(0, 0)], qe, qre);
            for (int q = 0; q < 3; ++q) {
                load16(qe[q], b.read_e(b.step, q) + pk1, nf);
                load16(qh[q], b.read_h(b.step, q) + pk, fbytes);
            }
            if (COMP) {
                load_rec(qre, b.read_e(b.step, 0), pk1, nc);
                load_rec(qrh, b.read_h(b.step, 0), pk, cbytes);
            }
        } else {
            for (int q = 0; q < 3; ++q) {
                load32(RE[ES(0, 0)][q], b.read_e(b.step, q) + pk, fbytes);
                load32(RE[ES(-1, 0)][q], b.read_e(b.step, q) + pk1, nf);
                load32(RH[HS(0, 0)][q], b.read_h(b.step, q) + pk, fbytes);
            }
        }
        for (int q = 0; q < 3; ++q) {
            if (CE_ARR)
                load32(RC[HS(0, 0)][q], b.read_ce(b.step, q) + pk, cbytes);
            if (CH_ARR)
                load32(RK[HS(0, 0)][q], b.read_ch(b.step, q) + pk, cbytes);
        }
    }
    {
        const f2 e = {RE[ES(0, 0)][0][0], RE[ES(0, 0)][2][0]};
        sE[k0 & 1][0][wave][lane] = e;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): else every plane waits for its own prefetch at the loop head
    __syncthreads();

    for (int kk = k0; kk <= kend; kk += M) {
#pragma unroll
        for (int u = 0; u < M; ++u) {
            const int ph = (M - u) % M;  // a constant once unrolled
            const int k = kk + u;
            if (k > kend)
                break;
            const int par = k & 1;
            long long pk0 = (long long)k * P;
            // box addresses are formed anew in each plane: stepped on or kept as loop invariants they would be
            // spilled (128^3, 4 steps: 48.8 us)
            long long fs = b.step;
            if constexpr (Drive::on)
                __asm__ volatile("" : "+s"(fs));
            else
                __asm__ volatile("" : "+s"(pk0));
            // ---- decode the previous prefetch, prefetch the inputs of plane k+1 (E of k+2) ----
            {
                const bool pv = k + 1 <= kend && k + 1 < nz;
                const bool pv2 = pv && k + 2 < nz;
                const long long pk1 = pk0 + P, pk2 = pk1 + P;  // (planes that do not exist have no bytes)
                const unsigned nc1 = pv ? cbytes : 0u, nc2 = pv2 ? cbytes : 0u;
                if constexpr (H16) {
                    decode(RE[ES(-1, ph)], qe, qre);
                    decode(RH[HS(0, ph)], qh, qrh);
                    const unsigned nf1 = pv ? fbytes : 0u, nf2 = pv2 ? fbytes : 0u;
#pragma unroll
                    for (int q = 0; q < 3; ++q) load16(qe[q], b.read_e(fs, q) + pk2, nf2);
#pragma unroll
                    for (int q = 0; q < 3; ++q) load16(qh[q], b.read_h(fs, q) + pk1, nf1);
                    if (COMP) {
                        load_rec(qre, b.read_e(fs, 0), pk2, nc2);
                        load_rec(qrh, b.read_h(fs, 0), pk1, nc1);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 3; ++q) load32(RE[ES(-2, ph)][q], b.read_e(fs, q) + pk2, nc2);
#pragma unroll
                    for (int q = 0; q < 3; ++q) load32(RH[HS(-1, ph)][q], b.read_h(fs, q) + pk1, nc1);
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if (CE_ARR)
                        load32(RC[HS(-1, ph)][q], b.read_ce(fs, q) + pk1, nc1);
                    if (CH_ARR)
                        load32(RK[HS(-1, ph)][q], b.read_ch(fs, q) + pk1, nc1);
                }
            }
#pragma unroll
            for (int s = 0; s <= TS; ++s) {
                // both LDS reads of the phase leave first; what needs them comes last
                f2 upr = {0.0f, 0.0f};
                if (s < TS)
                    upr = sE[par][s][wave + 1][lane];  // (Ex, Ez) of row j0 + kNR
                if (s > 0) {
                    // ---- E update of stage s-1 (its H was staged before the last barrier) ----
                    const int sp = s - 1;
                    const int pp = k - sp;
                    const int lop = sp == TS - 1 ? max(0, kb - 1) : max(0, kb - TS + sp);
                    const int hip = sp == TS - 1 ? ke - 1 : min(nz - 1, ke + TS - 2 - sp);
                    const bool livep = pp >= lop && pp <= hip;
                    auto &E = RE[ES(sp, ph)];
                    const auto &Hn = RH[HS(sp, ph)];      // H^{n+sp+1/2}(p_sp), just updated
                    const auto &Hd = RH[HS(sp + 1, ph)];  // the same one plane down
                    const auto &Cs = RC[HS(sp, ph)];
                    if (livep) {
                        const f2 dn = sH[sp][wave][lane];  // (Hx, Hz) of row j0 - 1
                        int jv = j0;
                        if constexpr (Drive::on)
                            __asm__ volatile("" : "+s"(jv));
                        __builtin_amdgcn_sched_barrier(0);
                        // the row next to another wave's comes last, and of it the parts that read dn
#pragma unroll
                        for (int r = kNR - 1; r >= 0; --r) {
                            float cy = (Hn[0][r] - Hd[0][r]) - (Hn[2][r] - left_of(Hn[2][r]));
                            // Driven: walls and outside take no curl, for 0 * curl is NaN where a curl is not
                            // finite, and the forward's state is that of single slab sweeps (2 to 3 % of a
                            // sweep; by rows from scalars, or the masks are spilled: 5 %). Rows and columns
                            // beyond the wall follow: their H stays 0.
                            if constexpr (Drive::on)
                                cy = pp >= 1 && !wall_x ? cy : 0.0f;
                            const float ey = __builtin_fmaf(Cs[1][r], cy, E[1][r]);
                            const float hyl = Hn[1][r] - left_of(Hn[1][r]), hyd = Hn[1][r] - Hd[1][r];
                            if (r == 0)
                                __builtin_amdgcn_sched_barrier(0);
                            const float hxj = r > 0 ? Hn[0][r - 1] : dn.x, hzj = r > 0 ? Hn[2][r - 1] : dn.y;
                            float cx = (Hn[2][r] - hzj) - hyd, cz = hyl - (Hn[0][r] - hxj);
                            if constexpr (Drive::on) {
                                const bool jw = jv + r >= 1 && jv + r < ny;
                                cx = jw && pp >= 1 ? cx : 0.0f;
                                cz = jw && !wall_x ? cz : 0.0f;
                            }
                            const float ex = __builtin_fmaf(Cs[0][r], cx, E[0][r]);
                            const float ez = __builtin_fmaf(Cs[2][r], cz, E[2][r]);
                            if (CE_ARR) {
                                // coefficients are 0 on the walls and outside: E + 0 * curl = E
                                E[0][r] = ex;
                                E[1][r] = ey;
                                E[2][r] = ez;
                            } else {
                                const int j = j0 + r;
                                const bool in = i < nx && j < ny;
                                E[0][r] = in && j >= 1 && pp >= 1 ? ex : E[0][r];
                                E[1][r] = in && i >= 1 && pp >= 1 ? ey : E[1][r];
                                E[2][r] = in && i >= 1 && j >= 1 ? ez : E[2][r];
                            }
                        }
                    }
                    if constexpr (Drive::on) {
                        // the point source joins its node right after the update, then the probes read E
                        if (has_source && livep && pp == source_plane) {
                            const auto *t = constant(drive.tab);
                            const int f = t->sf, si = t->si, sj = t->sj;
                            const float w = constant(drive.w)[sp];
#pragma unroll
                            for (int r = 0; r < kNR; ++r)
#pragma unroll
                                for (int q = 0; q < 3; ++q)
                                    E[q][r] = f == q && i == si && j0 + r == sj ? E[q][r] + w : E[q][r];
                        }
                        const bool mine = livep && pp >= kb && pp < ke;
                        if (probes && mine) {
                            for (unsigned long long m = probes; m; m &= m - 1) {
                                const int q = __builtin_ctzll(m);
                                const auto *t = constant(drive.tab);
                                if (t->pk[q] != pp)
                                    continue;
                                const int f = t->pf[q], pi = t->pi[q], pj = t->pj[q];
                                double *rec = drive.rec + (long long)sp * t->np + q;
#pragma unroll
                                for (int r = 0; r < kNR; ++r)
                                    if (own[r] && i == pi && j0 + r == pj)
                                        *rec = (double)(f == 0 ? E[0][r] : f == 1 ? E[1][r] : E[2][r]);
                            }
                        }
                        // H^{n+sp+1/2} of this plane into its history slot
                        if (sp < drive.nhist) {
                            const unsigned n = mine ? fbytes : 0u;
                            const long long pk = pk0 - sp * P;
#pragma unroll
                            for (int q = 0; q < 3; ++q) {
                                const __amdgpu_buffer_rsrc_t d = plane_rsrc(box_at(drive.hist, fs, 3 * sp + q) + pk, n);
#pragma unroll
                                for (int r = 0; r < kNR; ++r)
                                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, Hn[q][r]), d,
                                                                          own[r] ? vc[r] : kDrop, 0, 0);
                            }
                        }
                    }
                    if (sp < TS - 1) {
                        const f2 e = {E[0][0], E[2][0]};
                        sE[par ^ 1][sp + 1][wave][lane] = e;
                    } else {
                        // every lane issues every store: lanes and planes that write nothing drop it
                        const bool wr = livep && pp >= kb;
                        const unsigned nf = wr ? fbytes : 0u;
                        const long long pk = pk0 - sp * P;
                        unsigned vr[kNR], vs[kNR];
#pragma unroll
                        for (int r = 0; r < kNR; ++r) {
                            vr[r] = own[r] ? vc[r] : kDrop;
                            vs[r] = H16 ? vr[r] >> 1 : vr[r];
                        }
                        if constexpr (COMP) {
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                unsigned short q[3];
#pragma unroll
                                for (int p = 0; p < 3; ++p) {
                                    unsigned hh;
                                    Store<S>::enc2(h ? Hn[p][0] : E[p][0], h ? Hn[p][1] : E[p][1], hh, q[p]);
                                    const __amdgpu_buffer_rsrc_t d =
                                        plane_rsrc((h ? b.write_h(fs, p) : b.write_e(fs, p)) + pk, nf);
                                    __builtin_amdgcn_raw_buffer_store_b16((short)hh, d, vs[0], 0, 0);
                                    __builtin_amdgcn_raw_buffer_store_b16((short)(hh >> 16), d, vs[1], 0, 0);
                                }
                                const unsigned w0 = (q[0] & 0xffu) | ((q[1] & 0xffu) << 8) | ((q[2] & 0xffu) << 16);
                                const unsigned w1 = (unsigned)(q[0] >> 8) | ((unsigned)(q[1] >> 8) << 8) |
                                                    ((unsigned)(q[2] >> 8) << 16);
                                const __amdgpu_buffer_rsrc_t d = plane_rsrc(
                                    (const char *)(h ? b.write_h(fs, 0) : b.write_e(fs, 0)) + g.lo_off + kRecBytes * pk,
                                    wr ? cbytes : 0u);
                                __builtin_amdgcn_raw_buffer_store_b32(w0, d, vr[0], 0, 0);
                                __builtin_amdgcn_raw_buffer_store_b32(w1, d, vr[1], 0, 0);
                            }
                        } else {
#pragma unroll
                            for (int q = 0; q < 6; ++q) {
                                const __amdgpu_buffer_rsrc_t d = plane_rsrc(
                                    (q < 3 ? b.write_e(fs, q) : b.write_h(fs, q - 3)) + pk, nf);
                                const float *x = q < 3 ? E[q % 3] : Hn[q % 3];
                                if constexpr (H16) {
                                    const unsigned hh = Store<S>::pack2(x[0], x[1]);
                                    __builtin_amdgcn_raw_buffer_store_b16((short)hh, d, vs[0], 0, 0);
                                    __builtin_amdgcn_raw_buffer_store_b16((short)(hh >> 16), d, vs[1], 0, 0);
                                } else {
#pragma unroll
                                    for (int r = 0; r < kNR; ++r)
                                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x[r]), d,
                                                                              vs[r], 0, 0);
                                }
                            }
                        }
                    }
                }
                if (s == TS)
                    break;
                // ---- H update of stage s, in place ----
                const int p = k - s;
                const int lo = max(0, kb - TS + s), hi = min(nz - 1, ke + TS - 2 - s);
                const auto &en = RE[ES(s - 1, ph)];  // E input at plane p+1: role -1 or stage s-1's output
                const auto &Es = RE[ES(s, ph)];
                const auto &Ks = RK[HS(s, ph)];
                auto &H = RH[HS(s, ph)];
                if (p >= lo && p <= hi) {
#pragma unroll
                    for (int r = 0; r < kNR; ++r) {
                        const float ezr = right_of(Es[2][r]) - Es[2][r], eyr = right_of(Es[1][r]) - Es[1][r];
                        const float eyu = en[1][r] - Es[1][r];
                        H[1][r] = __builtin_fmaf(Ks[1][r], ezr - (en[0][r] - Es[0][r]), H[1][r]);
                        if (r == kNR - 1)
                            __builtin_amdgcn_sched_barrier(0);
                        const float exj = r + 1 < kNR ? Es[0][r + 1] : upr.x, ezj = r + 1 < kNR ? Es[2][r + 1] : upr.y;
                        H[0][r] = __builtin_fmaf(Ks[0][r], eyu - (ezj - Es[2][r]), H[0][r]);
                        H[2][r] = __builtin_fmaf(Ks[2][r], (exj - Es[0][r]) - eyr, H[2][r]);
                    }
                }
                const f2 h = {H[0][kNR - 1], H[2][kNR - 1]};
                sH[s][wave + 1][lane] = h;
                if (s == 0) {
                    const f2 e = {en[0][0], en[2][0]};
                    sE[par ^ 1][0][wave][lane] = e;
                }
                __syncthreads();
            }
            if (TS == 1)
                __syncthreads();  // the next plane's H update rewrites sH[0], which this E update read
        }
    }
#undef ES
#undef HS
}

// One workgroup per tile (queue null, in the order remap names), or one workgroup per CU taking tiles
// from the queue.
template <typename S, int TS, bool CE_ARR, bool CH_ARR, int kNW>
__global__ void __launch_bounds__(64 * kNW, (kNW != kNarrowWaves ? 1 : column_narrow_pairs(sizeof(S) == 2, TS, CE_ARR, CH_ARR) ? 4 : 2))
    k_column(Geom g, FieldBoxes<S> b, int kchunk, int ntx, int nty, int ntiles, int nvb, int remap, int cpx,
             unsigned *queue)
{
    __shared__ int s_v;
    const bool lead = threadIdx.x == 0 && threadIdx.y == 0;
    TileQueue tq(queue, nvb);
    for (;;) {
        int v = blockIdx.x;
        if (queue) {
            if (lead)
                s_v = tq.take();
            __syncthreads();
            v = __builtin_amdgcn_readfirstlane(s_v);
            __syncthreads();  // every lane has read s_v before the next take rewrites it
            if (v < 0)
                break;  // the same for the whole workgroup
        }
        const int t = tile_of_block(v, ntiles, remap, cpx);
        if (t < ntiles)
            column_tile<S, TS, CE_ARR, CH_ARR, kNW>(
                g, b, kchunk, ntx, nty, t % ntx, (t / ntx) % nty, t / (ntx * nty), NoDrive{});
        if (!queue)
            return;
        __syncthreads();  // the next tile rewrites the LDS this one read last
    }
    if (lead)
        tq.finish();
}

template <typename S, int TS>
hipError_t launch_column(const Geom &g, const Fields<S> &src, const Fields<S> &dst, const Coefs<float> &c, int zchunk,
                         hipStream_t s, unsigned *queue)
{
    const int cpx = cus_per_xcd();
    const int kchunk = (g.nz + zchunk - 1) / zchunk, nzc = (g.nz + kchunk - 1) / kchunk;
    auto go = [&](auto kernel, int waves) {
        int ntx, nty;
        column_windows(g.nx, g.ny, TS, waves, &ntx, &nty);
        const int ntiles = ntx * nty * nzc, nvb = (ntiles + kXcds - 1) / kXcds * kXcds;
        // with a CU for every tile there is nothing to hand out: a workgroup per tile saves the queue's
        // serial atomics (64^3: 27 us a sweep through the queue, 24 without); narrow workgroups are handed out by the
        // dispatcher, two a CU where their registers allow it
        const bool direct = !queue || temporal_sched() == 0 || ntiles <= kXcds * cpx || waves == kNarrowWaves;
        const dim3 block(64, waves), grid(direct ? nvb : std::min(ntiles, kXcds * cpx));
        hipLaunchKernelGGL(kernel, grid, block, 0, s, g, FieldBoxes<S>{src, dst, c}, kchunk, ntx, nty, ntiles, nvb,
                           temporal_sched() == 0 ? xcd_remap() : 2, cpx, direct ? nullptr : queue);
        return hipGetLastError();
    };
    const bool cea = c.ce[0] != nullptr, cha = c.ch[0] != nullptr;
    auto pick = [&](auto ce, auto ch) {
        constexpr bool CE = decltype(ce)::value, CH = decltype(ch)::value;
        constexpr int wide = column_waves<S, TS, CE, CH>();
        const bool pairs = column_narrow_pairs(sizeof(S) == 2, TS, CE, CH);
        if (column_waves_for(g, TS, wide, pairs, nzc, kXcds * cpx) == kNarrowWaves)
            return go(k_column<S, TS, CE, CH, kNarrowWaves>, kNarrowWaves);
        return go(k_column<S, TS, CE, CH, wide>, wide);
    };
    using yes = std::true_type;
    using no = std::false_type;
    return cea && cha ? pick(yes{}, yes{}) : cha ? pick(no{}, yes{}) : cea ? pick(yes{}, no{}) : pick(no{}, no{});
}

}  // namespace

template <typename S>
hipError_t launch_column_step(const Geom &g, const Fields<S> &src, const Fields<S> &dst, const Coefs<float> &c,
                              int zchunk, int ts, hipStream_t s, unsigned *queue)
{
    switch (ts) {
    case 1: return launch_column<S, 1>(g, src, dst, c, zchunk, s, queue);
    case 2: return launch_column<S, 2>(g, src, dst, c, zchunk, s, queue);
    case 3: return launch_column<S, 3>(g, src, dst, c, zchunk, s, queue);
    case 4: return launch_column<S, 4>(g, src, dst, c, zchunk, s, queue);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fdtd
