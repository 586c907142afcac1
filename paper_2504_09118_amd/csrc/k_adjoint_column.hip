// Column form of the reverse sweep (k_adjoint.hip): TS reverse steps n, n-1, ... in one pass, FP32 storage
// with one scalar Ch. The stages follow each other one plane behind, as the forward column sweep's do
// (column.h): stage s takes step n - s on plane k - s,
//   mu' = mu - K(Ce lam),  gCe += lam (L h),  lam' = lam - L(Ch mu'),  lam' += 2 E at the probes,
// with h = H^{n-s+1/2} from its history slot. A lane holds one column of two rows; x neighbours come from
// the next lanes, one row per wave crosses LDS in y for each of Ce lam, Ch mu' and h. lam, mu, Ce and the
// FP32 group sums of gCe cross memory once for TS steps. Products are rounded on their own and every
// operand is that of k_adj_slab: the same bits.
//
// What bounds it: at 128^3 (two steps, 81 us; the slab sweep 43 us for one) 310 MB cross the last-level
// cache's edge at 3.8 TB/s, the window's halo among them (60 of 64 columns, 20 of 24 rows own); a plane's
// two barriers and its scalar address work keep it from the 11 TB/s that a copy there reaches. A sweep of
// one step takes 71 us. 128^3, 200 steps with 2 probes: 8.7 ms, slab sweeps 10.0; 48x40x56, 150 steps:
// 1.06 (narrow workgroups; 1.28 full) and 2.2 ms.
#include "column_lanes.h"
#include "fdtd_internal.h"
#include "tile_queue.h"
#include "yee_update.h"

#pragma clang fp contract(off)

namespace fdtd {
namespace {

constexpr int kNR = kColumnRows, kCols = 64;

__device__ __forceinline__ float rmul(float a, float b) { return a * b; }

template <int TS, int kNW>
__global__ void __launch_bounds__(64 * kNW, (kNW != kNarrowWaves ? 1 : adjoint_narrow_pairs(TS) ? 4 : 2))
    k_adj_column(Geom g, ColumnBoxes b, AdjointColumn ac, int kchunk, int ntx, int nty, int ntiles, int cpx)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    constexpr int kRows = kNR * kNW;
    __shared__ __attribute__((aligned(16))) f2 sE[2][TS][kNW + 1][kCols];  // (Ce lam)_(x, z) of each wave's first row
    __shared__ __attribute__((aligned(16))) f2 sB[TS][kNW + 1][kCols];     // (Ch mu')_(x, z) of wave w - 1's last row
    __shared__ __attribute__((aligned(16))) f2 sF[TS][kNW + 1][kCols];     // h_(x, z) of wave w - 1's last row

    const int t = tile_of_block(blockIdx.x, ntiles, 2, cpx);
    if (t >= ntiles)
        return;  // the whole workgroup leaves before any barrier
    const int tile_x = t % ntx, tile_y = (t / ntx) % nty, zc = t / (ntx * nty);
    const int nx = g.nx, ny = g.ny, nz = g.nz, px = g.px;
    const long long P = g.plane;
    const int kb = zc * kchunk, ke = min(nz, kb + kchunk);
    const int lane = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int i = tile_x * (kCols - 2 * TS) + lane;
    const int row0 = wave * kNR, j0 = tile_y * (kRows - 2 * TS) + row0;
    const bool col_own = i < nx && (lane >= TS || tile_x == 0) && (lane < kCols - TS || tile_x == ntx - 1);

    if (wave == 0) {  // the rows beside the window: never written
        const f2 z = {0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < TS; ++s) {
            sE[0][s][kNW][lane] = z;
            sE[1][s][kNW][lane] = z;
            sB[s][0][lane] = z;
            sF[s][0][lane] = z;
        }
    }

    // byte offset of the lane's cells in a plane, the cells the tile owns, and those whose h their gCe terms
    // read: the own cells and one row and column before them
    unsigned vc[kNR];
    bool own[kNR], needs_h[kNR];
#pragma unroll
    for (int r = 0; r < kNR; ++r) {
        const int j = j0 + r, lr = row0 + r;
        const bool in = i < nx && j < ny;
        const bool below = lr < kRows - TS || tile_y == nty - 1;
        own[r] = in && col_own && (lr >= TS || tile_y == 0) && below;
        needs_h[r] = in && below && (lr >= TS - 1 || tile_y == 0) && (lane >= TS - 1 || tile_x == 0) &&
                     (lane < kCols - TS || tile_x == ntx - 1);
        vc[r] = in ? (unsigned)(i + px * j) * 4u : kDrop;
    }
    // the probes in this wave's rows and planes (own or halo: every copy takes the probe's term)
    unsigned long long probes = 0;
    if (ac.rec[0] || ac.rec[TS - 1]) {
        const auto *d = constant(ac.tab);
        probes = __ballot(lane < d->np && d->pj[lane] >= j0 && d->pj[lane] < j0 + kNR && d->pi[lane] >= i - lane &&
                          d->pi[lane] < i - lane + kCols && d->pk[lane] >= kb - TS && d->pk[lane] < ke + TS);
    }

    // Rings as in column.h. lam and Ce roles: -2 (prefetched for plane k+2), -1 (plane k+1), s; mu roles: -1
    // (prefetched for k+1), s, TS (the last stage's, one plane down); group sums: -1 (prefetched), s.
    // h of stage s: hc (plane k-s; loaded for the next plane as soon as this one's terms are formed), hp ((x,
    // y) one plane down).
    constexpr int M = TS + 2;
    float RL[M][3][kNR], RC[M][3][kNR], RM[M][3][kNR], RG[M][3][kNR];
    float hc[TS][3][kNR], hp[TS][2][kNR];
#pragma unroll
    for (int r = 0; r < kNR; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
            for (int m = 0; m < M; ++m) RL[m][q][r] = RC[m][q][r] = RM[m][q][r] = RG[m][q][r] = 0.0f;
#pragma unroll
            for (int s = 0; s < TS; ++s) {
                hc[s][q][r] = 0.0f;
                if (q < 2)
                    hp[s][q][r] = 0.0f;
            }
        }
#define ES(r, ph) ring_slot(r, ph, 2, M)
#define HS(r, ph) ring_slot(r, ph, 1, M)
    const int k0 = max(0, kb - TS), kend = ke + TS - 2;
    const unsigned bytes = (unsigned)(P * 4);
    const float ch = b.ch_s, m1 = -1.0f;
    const int hlo = max(0, kb - 1);  // h: the own planes and one before them

    // a plane of a box (no bytes: zeros) for the cells of mask (null: all of the lane's)
    auto load = [&](float *out, const float *p, bool exists, const bool *mask) {
        const __amdgpu_buffer_rsrc_t d = plane_rsrc(p, exists ? bytes : 0u);
#pragma unroll
        for (int r = 0; r < kNR; ++r)
            out[r] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(d, !mask || mask[r] ? vc[r] : kDrop, 0, 0));
    };
    const long long pk = (long long)k0 * P;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const long long fs = b.step;
        load(RL[ES(0, 0)][q], b.read_e(fs, q) + pk, true, nullptr);
        load(RL[ES(-1, 0)][q], b.read_e(fs, q) + pk + P, k0 + 1 < nz, nullptr);
        load(RC[ES(0, 0)][q], b.read_ce(fs, q) + pk, true, nullptr);
        load(RC[ES(-1, 0)][q], b.read_ce(fs, q) + pk + P, k0 + 1 < nz, nullptr);
        load(RM[HS(0, 0)][q], b.read_h(fs, q) + pk, true, nullptr);
        load(RG[HS(0, 0)][q], box_at(ac.gpart, fs, q) + pk, k0 >= kb, own);
#pragma unroll
        for (int s = 0; s < TS; ++s) {
            const float *h = box_at(ac.hist, fs, q - 3 * s) + (pk - s * P);
            load(hc[s][q], h, k0 - s >= hlo && k0 - s < ke, needs_h);
            if (q < 2)
                load(hp[s][q], h - P, k0 - s - 1 >= hlo && k0 - s - 1 < ke, needs_h);
        }
    }
    {
        const f2 e = {rmul(RC[ES(0, 0)][0][0], RL[ES(0, 0)][0][0]), rmul(RC[ES(0, 0)][2][0], RL[ES(0, 0)][2][0])};
        sE[k0 & 1][0][wave][lane] = e;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();

    for (int kk = k0; kk <= kend; kk += M) {
#pragma unroll
        for (int u = 0; u < M; ++u) {
            const int ph = (M - u) % M;
            const int k = kk + u;
            if (k > kend)
                break;
            const int par = k & 1;
            long long fs = b.step;  // (box addresses formed anew, as in column.h)
            __asm__ volatile("" : "+s"(fs));
            const bool more = k + 1 <= kend;
            const long long pk0 = (long long)k * P;  // (planes that do not exist have no bytes)
            // ---- prefetch ----
            {
                const bool e1 = more && k + 1 < nz, e2 = more && k + 2 < nz, g1 = e1 && k + 1 >= kb && k + 1 < ke;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    load(RL[ES(-2, ph)][q], b.read_e(fs, q) + (pk0 + 2 * P), e2, nullptr);
                    load(RC[ES(-2, ph)][q], b.read_ce(fs, q) + (pk0 + 2 * P), e2, nullptr);
                    load(RM[HS(-1, ph)][q], b.read_h(fs, q) + (pk0 + P), e1, nullptr);
                    load(RG[HS(-1, ph)][q], box_at(ac.gpart, fs, q) + (pk0 + P), g1, own);
                }
            }
#pragma unroll
            for (int s = 0; s <= TS; ++s) {
                f2 upr = {0.0f, 0.0f};
                if (s < TS)
                    upr = sE[par][s][wave + 1][lane];  // Ce lam of row j0 + kNR
                if (s > 0) {
                    // ---- gCe and lam' of stage s-1 ----
                    const int sp = s - 1;
                    const int pp = k - sp;
                    const int lop = sp == TS - 1 ? max(0, kb - 1) : max(0, kb - TS + sp);
                    const int hip = sp == TS - 1 ? ke - 1 : min(nz - 1, ke + TS - 2 - sp);
                    const bool livep = pp >= lop && pp <= hip;
                    auto &L = RL[ES(sp, ph)];
                    auto &G = RG[HS(sp, ph)];
                    const auto &Mn = RM[HS(sp, ph)];      // mu' of this plane
                    const auto &Md = RM[HS(sp + 1, ph)];  // one plane down
                    if (livep) {
                        const f2 dn = sB[sp][wave][lane];       // (Ch mu')_(x, z) of row j0 - 1
                        const f2 fd = sF[sp][wave][lane];       // h_(x, z) of row j0 - 1
                        __builtin_amdgcn_sched_barrier(0);
                        const auto &h = hc[sp];
                        float bm[3][kNR];
#pragma unroll
                        for (int q = 0; q < 3; ++q)
#pragma unroll
                            for (int r = 0; r < kNR; ++r) bm[q][r] = rmul(ch, Mn[q][r]);
#pragma unroll
                        for (int r = kNR - 1; r >= 0; --r) {
                            const int j = j0 + r;
                            const bool in = i < nx && j < ny;
                            const float l0 = L[0][r], l1 = L[1][r], l2 = L[2][r];
                            const float hzl = h[2][r] - left_of(h[2][r]), hyl = h[1][r] - left_of(h[1][r]);
                            const float bzl = bm[2][r] - left_of(bm[2][r]), byl = bm[1][r] - left_of(bm[1][r]);
                            const float bdx = rmul(ch, Md[0][r]), bdy = rmul(ch, Md[1][r]);
                            const float hxj = r > 0 ? h[0][r - 1] : fd.x, hzj = r > 0 ? h[2][r - 1] : fd.y;
                            const float bxj = r > 0 ? bm[0][r - 1] : dn.x, bzj = r > 0 ? bm[2][r - 1] : dn.y;
                            // a node that never changes has lam = 0, so its gCe term is 0
                            const float lh0 = (h[2][r] - hzj) - (h[1][r] - hp[sp][1][r]);
                            const float lh1 = (h[0][r] - hp[sp][0][r]) - hzl;
                            const float lh2 = hyl - (h[0][r] - hxj);
                            const bool ok0 = in && j >= 1 && pp >= 1, ok1 = in && i >= 1 && pp >= 1,
                                       ok2 = in && i >= 1 && j >= 1;
                            G[0][r] = ok0 ? G[0][r] + rmul(l0, lh0) : G[0][r];
                            G[1][r] = ok1 ? G[1][r] + rmul(l1, lh1) : G[1][r];
                            G[2][r] = ok2 ? G[2][r] + rmul(l2, lh2) : G[2][r];
                            const float x = __builtin_fmaf(m1, (bm[2][r] - bzj) - (bm[1][r] - bdy), l0);
                            const float y = __builtin_fmaf(m1, (bm[0][r] - bdx) - bzl, l1);
                            const float z = __builtin_fmaf(m1, byl - (bm[0][r] - bxj), l2);
                            L[0][r] = ok0 ? x : l0;
                            L[1][r] = ok1 ? y : l1;
                            L[2][r] = ok2 ? z : l2;
                        }
                    }
                    // the next plane's h takes the place of this one's
#pragma unroll
                    for (int r = 0; r < kNR; ++r) {
                        hp[sp][0][r] = hc[sp][0][r];
                        hp[sp][1][r] = hc[sp][1][r];
                    }
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        load(hc[sp][q], box_at(ac.hist, fs, q - 3 * sp) + (pk0 + P - sp * P),
                             more && k + 1 - sp >= hlo && k + 1 - sp < ke, needs_h);
                    // probe terms of this step, in probe order (duplicates add in turn)
                    if (probes && livep && ac.rec[sp]) {
                        for (unsigned long long m = probes; m; m &= m - 1) {
                            const int q = __builtin_ctzll(m);
                            if (constant(ac.tab)->pk[q] != pp)
                                continue;
                            const float add = (float)(2.0 * ac.rec[sp][q]);
                            const auto *t = constant(ac.tab);
                            const int f = t->pf[q], pi = t->pi[q], pj = t->pj[q];
#pragma unroll
                            for (int r = 0; r < kNR; ++r)
#pragma unroll
                                for (int e = 0; e < 3; ++e)
                                    L[e][r] = e == f && i == pi && j0 + r == pj ? L[e][r] + add : L[e][r];
                        }
                    }
                    if (sp < TS - 1) {
                        const auto &Cs = RC[ES(sp, ph)];
                        const f2 e = {rmul(Cs[0][0], L[0][0]), rmul(Cs[2][0], L[2][0])};
                        sE[par ^ 1][sp + 1][wave][lane] = e;
                    } else {
                        const bool wr = livep && pp >= kb;
                        const unsigned n = wr ? bytes : 0u;
                        const long long pk = pk0 - sp * P;
                        if (ac.close && wr) {
                            // the step that closes a group: its sums join the FP64 total
#pragma unroll
                            for (int q = 0; q < 3; ++q)
#pragma unroll
                                for (int r = 0; r < kNR; ++r)
                                    if (own[r]) {
                                        auto *p = (__attribute__((address_space(1))) double *)(
                                            box_at(ac.gce, ac.gstep, q) + pk + (vc[r] >> 2));
                                        *p = *p + (double)G[q][r];
                                        G[q][r] = 0.0f;
                                    }
                        }
                        unsigned vs[kNR];
#pragma unroll
                        for (int r = 0; r < kNR; ++r) vs[r] = own[r] ? vc[r] : kDrop;
#pragma unroll
                        for (int q = 0; q < 9; ++q) {
                            const __amdgpu_buffer_rsrc_t d =
                                plane_rsrc((q < 3   ? b.write_e(fs, q)
                                            : q < 6 ? b.write_h(fs, q - 3)
                                                    : box_at(ac.gpart, fs, q - 6)) + pk, n);
                            const float *x = q < 3 ? L[q] : q < 6 ? Mn[q - 3] : G[q - 6];
#pragma unroll
                            for (int r = 0; r < kNR; ++r)
                                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x[r]), d, vs[r], 0, 0);
                        }
                    }
                }
                if (s == TS)
                    break;
                // ---- mu' of stage s ----
                const int p = k - s;
                const int lo = max(0, kb - TS + s), hi = min(nz - 1, ke + TS - 2 - s);
                const auto &Ln = RL[ES(s - 1, ph)], &Ls = RL[ES(s, ph)];
                const auto &Cn = RC[ES(s - 1, ph)], &Cs = RC[ES(s, ph)];
                auto &Mu = RM[HS(s, ph)];
                if (p >= lo && p <= hi) {
                    float a[3][kNR];
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int r = 0; r < kNR; ++r) a[q][r] = rmul(Cs[q][r], Ls[q][r]);
#pragma unroll
                    for (int r = 0; r < kNR; ++r) {
                        const float azr = right_of(a[2][r]) - a[2][r], ayr = right_of(a[1][r]) - a[1][r];
                        const float ayu = rmul(Cn[1][r], Ln[1][r]) - a[1][r], axu = rmul(Cn[0][r], Ln[0][r]) - a[0][r];
                        Mu[1][r] = __builtin_fmaf(m1, azr - axu, Mu[1][r]);
                        const float axj = r + 1 < kNR ? a[0][r + 1] : upr.x, azj = r + 1 < kNR ? a[2][r + 1] : upr.y;
                        Mu[0][r] = __builtin_fmaf(m1, ayu - (azj - a[2][r]), Mu[0][r]);
                        Mu[2][r] = __builtin_fmaf(m1, (axj - a[0][r]) - ayr, Mu[2][r]);
                    }
                }
                const f2 bw = {rmul(ch, Mu[0][kNR - 1]), rmul(ch, Mu[2][kNR - 1])};
                sB[s][wave + 1][lane] = bw;
                const f2 f = {hc[s][0][kNR - 1], hc[s][2][kNR - 1]};
                sF[s][wave + 1][lane] = f;
                if (s == 0) {
                    const f2 e = {rmul(Cn[0][0], Ln[0][0]), rmul(Cn[2][0], Ln[2][0])};
                    sE[par ^ 1][0][wave][lane] = e;
                }
                __syncthreads();
            }
            if (TS == 1)
                __syncthreads();  // the next plane's mu' rewrites sB[0] and sF[0], which this lam' read
        }
    }
#undef ES
#undef HS
}

template <int TS>
hipError_t launch_ts(const Geom &g, const Fields<float> &src, const Fields<float> &dst, const Coefs<float> &c,
                     const AdjointColumn &ac, int zchunk, hipStream_t s)
{
    const int kchunk = (g.nz + zchunk - 1) / zchunk, nzc = (g.nz + kchunk - 1) / kchunk;
    constexpr int wide = adjoint_column_waves(TS);
    const int cpx = cus_per_xcd();
    ColumnBoxes b;
    if (!column_boxes(src, dst, c, &b))
        return hipErrorInvalidValue;
    auto go = [&](auto kernel, int waves) {
        int ntx, nty;
        column_windows(g.nx, g.ny, TS, waves, &ntx, &nty);
        const int ntiles = ntx * nty * nzc, nblocks = (ntiles + kXcds - 1) / kXcds * kXcds;
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(64, waves), 0, s, g, b, ac, kchunk, ntx, nty, ntiles, cpx);
        return hipGetLastError();
    };
    // (as the forward's workgroups)
    if (column_waves_for(g, TS, wide, adjoint_narrow_pairs(TS), nzc, kXcds * cpx) == kNarrowWaves)
        return go(k_adj_column<TS, kNarrowWaves>, kNarrowWaves);
    return go(k_adj_column<TS, wide>, wide);
}

}  // namespace

hipError_t launch_adj_column(const Geom &g, const Fields<float> &src, const Fields<float> &dst, const Coefs<float> &c,
                             const AdjointColumn &ac, int ts, int zchunk, hipStream_t s)
{
    if (!c.ce[0] || c.ch[0] || !ac.gpart)
        return hipErrorInvalidValue;
    zchunk = zchunk < 1 ? 1 : zchunk;
    switch (ts) {
    case 1: return launch_ts<1>(g, src, dst, c, ac, zchunk, s);
    case 2: return launch_ts<2>(g, src, dst, c, ac, zchunk, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fdtd
