// One iteration of Alg. 1 (problem (20)) as one HBM-streaming sweep for gfx950.
//
// FP32 duals:
//   passes   (fallback.hip): the thresholds tau_s, tau_t of this iteration
//            whose search missed at the end of the last one; a no-op otherwise.
//   sweep    (LDS-tiled): steps 1-14, with the thresholds and the factor
//            a4 of y4 known from the end of the last iteration; the FP64 partial
//            sums of the stopping rule (eq. (28)) and of the l2-ball distance of
//            step 15; and what the search of the next thresholds needs of the
//            new state (search.hip).
//   search   (search.hip): the l2-ball factor of step 15 (applied lazily when
//            y4 is next read), the stopping test, the iteration counter, and
//            the next thresholds.
//
// Every state word is read and written once per iteration (172 bytes per
// voxel with FP32 duals). What bounds the sweep is HBM streaming: 287 us for
// 256 x 256 x 128 and 1866 us for 512 x 512 x 224 are 5.03 and 5.41 TB/s on those
// bytes, 0.94 and more of what a plain copy reaches. In two sweeps with the search
// between them (the second read s, t, y3, y4 and an intermediate again, 36
// bytes) the iteration took 354 and 2350 us, now 301 and 1898. Cubes of few tiles
// are bound by the instructions of a band (4.7 us) and a tile's start and end
// instead: 64 x 64 x 16 17 us.
//
// Two things let the loads of a band stay in flight for a whole band. They go
// through the buffer path (common.hpp: band_of), so no branch stands between a
// load and its use and the compiler waits for exactly that load; with branches
// it waited for everything outstanding, at four points of a band. And the edge
// masks of y are applied when it is stored to LDS, not when it is loaded. (The
// BF16 sweep, the same otherwise: 400 -> 352 us at 256 x 256 x 190.)
//
// The sweep keeps the w1/w2 extrapolations (12 of the 21 state words per voxel)
// out of HBM: a workgroup owns a TI x TJ pixel tile and marches through a
// chunk of bands. Per band it stages the masked dual edge fields y1, y2 with
// a 2-pixel halo in LDS, recomputes w' on a 1-pixel ring, u' on the
// (i+1, j+1) ring and t' on the rows above and below, and updates y1, y2, y3
// from LDS; the D_s coupling of neighbouring bands is carried in LDS. Global
// loads of bands k+1 (w), k+2 (u, v, y4, s, t, y3) and k+3 (y) are issued while
// band k is computed, so the memory latency overlaps the arithmetic.
//
// Every state array is ping-ponged: iteration k reads side (k & 1) and writes
// side ((k + 1) & 1), so halo reads never race with writes. The side comes
// from the device iteration counter, which makes one iteration's launches a
// fixed sequence; once the stopping rule holds a device flag turns the
// remaining launches into no-ops, so iteration counts stay exact.
#include <string.h>

#include <type_traits>

#include "radix.hpp"

namespace geo {

namespace {

// LDS planes of a tile of TI x TJ pixels, TI * TJ <= NT, TI + TJ <= SPAN and TJ <=
// COLS: y with a 2-pixel halo, w' on a 1-pixel ring, u' with the (+1, +1) ring, t'
// with the rows above and below. A tile of fewer than NT pixels leaves the last word
// of each free: idle threads write there.
template <int THREADS, int SPAN, int COLS>
struct Planes {
    static constexpr int NT = THREADS;
    static constexpr int S2 = NT + 4 * SPAN + 16, S1 = NT + 2 * SPAN + 4, SU = NT + SPAN + 1;
    static constexpr int ST = NT + 2 * COLS;
    static constexpr int NY = (S2 + NT - 1) / NT;  // y points per thread
    static constexpr int T0 = NT / 2;              // first thread of the t' ring
    static_assert(2 * SPAN + 4 <= NT && SPAN + 1 <= T0 && T0 + 2 * COLS <= NT && T0 % 64 == 0,
                  "at most one ring point of a kind per thread, one of u' and t' per wavefront");
};
using Wide = Planes<kSweepThreads, kTileSpan, kTileCols>;  // 8 x 128 fills them
using Small = Planes<kSmallThreads, kSmallSpan, kSmallCols>;
static_assert((uint64_t)kMaxTiles * kSweepThreads <= 1u << 22 && 1u << 22 <= kNoPix - (1u << 22),
              "a missing pixel and its neighbours lie past a band");
static_assert(kTileRows * kTileCols == Wide::NT && kTileRows + kTileCols == kTileSpan, "the fixed tile fills the planes");
template <int S>
using PlanesOf = std::conditional_t<S == kSmallForm, Small, Wide>;
constexpr int NPT = 256;  // threads of the pointwise kernels
using lds_f = __attribute__((address_space(3))) float;

template <typename DT>
using Table = const CubeArgs<DT> *__restrict__;

// XCD-aware persistent tile order: the 8 XCDs take contiguous tile ranges so
// that the halos shared by neighbouring tiles meet in the same L2.
__device__ __forceinline__ int tile_at(int b, int G, int T, int r)
{
    if (G >= 8 && (G & 7) == 0) {
        const int x = b & 7, slot = b >> 3, per = G >> 3;
        const int lo = (int)(((int64_t)x * T) >> 3), hi = (int)(((int64_t)(x + 1) * T) >> 3);
        const int t = lo + slot + r * per;
        return t < hi ? t : -1;
    }
    const int t = b + r * G;
    return t < T ? t : -1;
}

// The tiles of many cubes in one launch: each cube's are dealt to the XCDs in
// contiguous eighths, and an XCD's blocks take its parts of one cube after another
// in turn. Of the tiles before number P of the list, XCD x has those whose number
// is x modulo 8, as many as it would have in turn, so the XCDs' shares differ by
// one at most. (With the list as a whole in eighths, the cubes of a mixed batch met
// different XCDs, and the XCDs with the deep tiles of a large cube kept the
// launch: an iteration of 512 x 512 x 224 and 256 x 256 x 128 took 3123 us, now 2165;
// of 256 x 256 x 128 and six of 128 x 128 x 64 1361, now 527; of 32 uneven cubes
// 5170, now 4690.)
struct TileList {
    int x, first, step;  // XCD (< 0: the list is not split), a block's first position, to its next
    __device__ __forceinline__ TileList(int b, int G)
    {
        const bool split = G >= 8 && (G & 7) == 0;
        x = split ? b & 7 : -1;
        first = split ? b >> 3 : b;
        step = split ? G >> 3 : G;
    }
    // positions of this XCD before tile P of the list
    __device__ __forceinline__ int before(int P) const { return x < 0 ? P : (P >> 3) + ((P & 7) > x ? 1 : 0); }
    // positions of the XCDs before this one
    __device__ __forceinline__ int below(int P) const { return x < 0 ? 0 : (P >> 3) * x + min(P & 7, x); }
};

// FUSED (FP32 duals): the whole iteration, thresholds known beforehand.
// Otherwise (BF16 duals) the first of two sweeps: steps 1, 4, 5, 11, 12 and the
// u' part of step 14, the inputs z_s, z_t of steps 2 and 3 with their window
// statistics; the search and sweep B (sweep_b.hip) follow in the same slot.
// With BF16 duals a change of 1e-10 in a threshold (the search-ahead form sums
// |z| by its slope in a4, not the rounded values) grows to 4e-4 of s within 40
// iterations, so that storage keeps the form whose sums are over the values
// themselves.
// S 0: tiles of 8 x 128 pixels, the geometry known to the compiler (256 x 256 x
// 128: 289 us, in the other form 293); 1: the cube's own rows x cols; kSmallForm: the
// same in workgroups of kSmallThreads, for cubes whose bands are one such tile.
template <typename DT, int S, bool FUSED>
__global__ __launch_bounds__(PlanesOf<S>::NT, 4) void k_sweep(Table<DT> cubes, LaunchShape sh)
{
    using P = typename PairOf<DT>::type;
    using PL = PlanesOf<S>;
    constexpr int NT = PL::NT, S2 = PL::S2, S1 = PL::S1, SU = PL::SU, ST = PL::ST, NY = PL::NY, T0 = PL::T0;
    // three bands of masked [y1v, y1h, y2v, y2h] | u' by band parity | w1', w2'
    // planes read by neighbours (ud_h, lr_v, c_v, c_h)
    __shared__ __align__(16) float smem[3 * 4 * S2 + 2 * SU + 2 * 4 * S1];
    // u' and w' start here
    constexpr int U0 = 3 * 4 * S2, W0 = U0 + 2 * SU;
    // t' with the rows above and below the tile; what a point keeps between the
    // phases of a band (t+, q+, y3, y3 of the row above)
    __shared__ float sT[FUSED ? ST : 1];
    __shared__ float4 keep[FUSED ? NT : 1];
    constexpr int NS = 8;  // FP64 partials of a tile
    __shared__ double red[(FUSED ? 10 : NS) * (NT / 64)];
    __shared__ uint32_t ncand[2];
    __shared__ int tile0[kMaxBatch + 1];

    // The tiles of the cubes of this form that work in this slot, one
    // cube after another: a cube that idles takes none, so the persistent
    // blocks, and the XCDs, share the working cubes' tiles evenly (with the
    // full list, a batch in which a few cubes still run would leave most
    // blocks without work). Every block reads the same flags, written before
    // this launch.
    // A single cube needs no list.
    static_assert(kMaxBatch <= 64, "one wavefront scans the cubes");
    const bool many = sh.ncubes > 1;
    if (!many) {
        const const4<CubeCommon> &cc = ((const4<CubeArgs<DT>> *)cubes)->c;
        DevScalars *sc = cc.sc;
        const bool idle_now = idle(sc);
        if (FUSED && blockIdx.x == 0 && threadIdx.x == 0) {
            sc->view = {sc->in.a_lo, sc->in.a_hi, sc->in.a_c, idle_now ? 1u : 0u};
            passes_over(slot_flags(cubes, 1));
        }
        if (idle_now) return;
    } else if (threadIdx.x < 64) {
        const int c = threadIdx.x;
        int x = c < sh.ncubes && cubes[c].c.g.form == S && !idle(cubes[c].c.sc) ? cubes[c].c.ntiles : 0;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (c >= o) x += y;
        }
        if (c < sh.ncubes) tile0[c + 1] = x;
        if (c == 0) tile0[0] = 0;
        // the first block copies what the search of this slot reads of the
        // state it rewrites, and lowers the flag of the histogram passes
        if (FUSED && blockIdx.x == 0) {
            if (c < sh.ncubes) {
                DevScalars *sc = cubes[c].c.sc;
                sc->view = {sc->in.a_lo, sc->in.a_hi, sc->in.a_c, idle(sc) ? 1u : 0u};
            }
            if (c == 0) passes_over(slot_flags(cubes, sh.ncubes));
        }
    }
    if (many) __syncthreads();
    const int tid = threadIdx.x;

    for (int r = 0;; ++r) {
        // (the working cubes' tile count is read from LDS at each tile rather
        // than kept live through the march)
        int cube = 0, lt;  // tile within the cube
        if (many) {
            const TileList list(blockIdx.x, sh.form_grid[S]);
            const int p = list.first + r * list.step;
            if (p >= list.before(tile0[sh.ncubes])) break;
            while (list.before(tile0[cube + 1]) <= p) ++cube;
            lt = p - list.before(tile0[cube]) + list.below(tile0[cube + 1]) - list.below(tile0[cube]);
        } else {
            lt = tile_at(blockIdx.x, sh.form_grid[S], ((const4<CubeArgs<DT>> *)cubes)->c.ntiles, r);
            if (lt < 0) break;
        }
        // uniform across the block: the cube's entry is read with scalar loads
        cube = __builtin_amdgcn_readfirstlane(cube);
        lt = __builtin_amdgcn_readfirstlane(lt);
        const4<CubeArgs<DT>> &a = ((const4<CubeArgs<DT>> *)cubes)[cube];
        const4<DevScalars> &sc = *(const4<DevScalars> *)a.c.sc;  // this launch does not write what it reads of it
        // Each phase reads the pointers and windows it needs with scalar loads
        // of its own: kept live through the march (as the compiler would, since
        // they never change) they overflow the scalar registers, and the spills
        // take vector registers and a fifth of the vector instructions.
        const4<CubeArgs<DT>> *ent = &a;
        const4<DevScalars> *scp = &sc;
        // LDS pointers are formed where they are used, for the same reason: one
        // base, the planes at constant offsets from it.
        auto at = [](float *p) {
            lds_f *q = (lds_f *)p;
            asm volatile("" : "+v"(q));
            return q;
        };
        auto fresh = [&]() {
            asm volatile("" : "+s"(ent), "+s"(scp));
            __builtin_amdgcn_sched_barrier(0);
        };
        const SweepGrid g{a.c.g.tj, a.c.g.ti, a.c.g.tk, a.c.g.kc, S, S ? a.c.g.rows : kTileRows,
                          S ? a.c.g.cols : kTileCols};
        const int TI = g.rows, TJ = g.cols;
        const int W2 = TJ + 4, W1 = TJ + 2, WU = TJ + 1;  // LDS row lengths
        const bool act = S == 0 || tid < TI * TJ;         // the thread has a point of the tile
        const int oti = act ? tid / TJ : 0, otj = act ? tid % TJ : 0;
        // Ring roles: the w' ring (the first threads) and, apart from each other
        // so that each wavefront has one, the u' ring (the first threads) and the
        // t' ring: the rows above and below the tile (threads T0 on).
        int rwi = 0, rwj = 0, rui = 0, ruj = 0;
        const bool ring_w = tid < 2 * (TI + TJ) + 4, ring_u = tid < TI + TJ + 1;
        const bool ring_t = FUSED && tid >= T0 && tid < T0 + 2 * TJ;
        const int wave0 = __builtin_amdgcn_readfirstlane(tid);
        const bool wave_t = FUSED && wave0 >= T0 && wave0 < T0 + 2 * TJ;
        if (ring_w) {
            if (tid < W1) { rwi = 0; rwj = tid; }
            else if (tid < 2 * W1) { rwi = TI + 1; rwj = tid - W1; }
            else { const int s = tid - 2 * W1; rwi = 1 + (s >> 1); rwj = (s & 1) ? W1 - 1 : 0; }
        }
        if (ring_u) {
            if (tid < WU) { rui = TI; ruj = tid; }
            else { rui = tid - WU; ruj = TJ; }
        }
        if (ring_t) {
            rui = tid - T0 < TJ ? -1 : TI;
            ruj = tid - T0 < TJ ? tid - T0 : tid - T0 - TJ;
        }
        // Offsets into the LDS planes: of the own point in y (one row up), w' and
        // u' (where an idle thread writes to the free word), of the ring points.
        const int oy = (oti + 1) * W2 + (otj + 2), ow = oti * W1 + otj, ou = oti * WU + otj;
        const int ow_w = act ? ow + W1 + 1 : S1 - 1, ou_w = act ? ou : SU - 1, ot_w = act ? TJ + tid : ST - 1;
        const int ry = (rui + 1) * W2 + (ruj + 2), ru = rui * WU + ruj;
        const int rwy = rwi * W2 + (rwj + 1), rww = rwi * W1 + rwj;
        const int tj = lt % g.tj, rest = lt / g.tj;
        const int j0 = tj * TJ, i0 = (rest % g.ti) * TI, kb = (rest / g.ti) * g.kc;
        const int n1 = a.c.d.n1, n2 = a.c.d.n2, n3 = a.c.d.n3;
        const int ke = min(kb + g.kc, n3);
        const int64_t N = a.c.d.plane;
        const uint32_t np = (uint32_t)n1 * (uint32_t)n2;  // pixels of a band

        if (tid < 2) ncand[tid] = 0u;  // published by the first barrier of the march
        const int par = (int)(sc.iter & 1u);
        const float a4 = FUSED ? sc.in.a4 : (float)sc.a4;
        const bool zst = !FUSED && sc.zstore != 0u;
        double du2 = 0.0, u2 = 0.0, r2 = 0.0;
        Gathered ga;
        SlopeRegs sl;
        // otherwise (by field): |z| above the window, sum and count (of the
        // wavefront), and sum of all |z|
        double sum[2] = {0.0, 0.0}, all[2] = {0.0, 0.0};
        uint32_t cnt[2] = {0u, 0u};

        // pixels of this thread in a band (kNoPix outside the cube)
        auto pixel = [&](int i, int j) {
            return i >= 0 && i < n1 && j >= 0 && j < n2 ? (uint32_t)i * (uint32_t)n2 + (uint32_t)j : kNoPix;
        };
        const int oi = i0 + oti, oj = j0 + otj;
        const uint32_t po = act ? pixel(oi, oj) : kNoPix;
        const bool own_in = po != kNoPix;
        const uint32_t pr = ring_u || ring_t ? pixel(i0 + rui, j0 + ruj) : kNoPix;
        const uint32_t pw = ring_w ? pixel(i0 - 1 + rwi, j0 - 1 + rwj) : kNoPix;
        uint32_t py[NY];
        // masks of the staged y: bit 2n vertical, 2n + 1 horizontal of point n;
        // of the own point: bits 16, 17; of the w' ring point: 18, 19
        uint32_t keepm = 0u;
#pragma unroll
        for (int n = 0; n < NY; ++n) {
            const int p = tid + NT * n, i = i0 - 2 + p / W2, j = j0 - 2 + p % W2;
            py[n] = p < (TI + 4) * W2 ? pixel(i, j) : kNoPix;
            keepm |= (i <= n1 - 2 ? 1u : 0u) << (2 * n) | (j <= n2 - 2 ? 2u : 0u) << (2 * n);
        }
        const float mv = mask_le(oi, n1), mh = mask_le(oj, n2);
        const float rmv = mask_le(i0 - 1 + rwi, n1), rmh = mask_le(j0 - 1 + rwj, n2);

        // ---------------- register staging of global loads ----------------
        // band k of an array; no bytes when the band is not wanted
        auto band = [&](auto *p, int k, bool want) { return band_of(p, (int64_t)k * np, want ? np : 0u); };
#define SRC (ent->side[par])
#define DST (ent->side[par ^ 1])
        using Raw = decltype(bld_raw((const P *)nullptr, BandRsrc(), 0u));
        auto loadY = [&](int k, bool want, Raw (&q1)[NY], Raw (&q2)[NY]) {
            const BandRsrc b1 = band(SRC.y1, k, want), b2 = band(SRC.y2, k, want);
#pragma unroll
            for (int n = 0; n < NY; ++n) {
                q1[n] = bld_raw((const P *)nullptr, b1, py[n]);
                q2[n] = bld_raw((const P *)nullptr, b2, py[n]);
            }
        };
        auto storeY = [&](float *buf, const Raw (&q1)[NY], const Raw (&q2)[NY]) {
            lds_f *o = at(buf + tid);
#pragma unroll
            for (int n = 0; n < NY; ++n) {
                const bool v = keepm >> (2 * n) & 1u, h = keepm >> (2 * n + 1) & 1u;
                const float2 y1 = pair_of(q1[n]), y2 = pair_of(q2[n]);
                if (NT * (n + 1) <= S2 || tid + NT * n < S2) {
                    o[NT * n] = v ? y1.x : 0.f;           // masked: last row (vertical)
                    o[NT * n + S2] = h ? y1.y : 0.f;      // last column (horizontal)
                    o[NT * n + 2 * S2] = v ? y2.x : 0.f;
                    o[NT * n + 3 * S2] = h ? y2.y : 0.f;
                }
            }
        };
        Raw ry1[NY], ry2[NY];
        // u, y4 (stored), v, s, t, y3 (row and row above) at the own point; u
        // and y4 at the u' ring point, or t, y4 and both y3 at the t' ring point
        float ru_u, ru_y4, ru_v, ru_s, ru_t, ru_y3c, ru_y3m, rr_u, rr_y4, rr_y3c = 0.f, rr_y3m = 0.f;
        auto loadRU = [&](int k, bool want, bool own) {
            const BandRsrc bu = band(SRC.u, k, want), b4 = band(SRC.y4, k, want);
            const BandRsrc bt = band(SRC.t, k, own), b3 = band(SRC.y3, k, own);
            ru_u = bld((const float *)nullptr, bu, po);
            ru_y4 = bld((const DT *)nullptr, b4, po);
            ru_s = bld<kNT>((const float *)nullptr, band(SRC.s, k, own), po);
            ru_t = bld<FUSED ? 0 : kNT>((const float *)nullptr, bt, po);
            ru_y3c = bld((const DT *)nullptr, b3, po);
            ru_y3m = bld((const DT *)nullptr, b3, po - (uint32_t)n2);  // row -1: past the band, 0
            ru_v = bld<kNT>((const float *)nullptr, band(ent->c.v, k, own), po);
            rr_u = bld((const float *)nullptr, wave_t ? bt : bu, pr);
            rr_y4 = bld((const DT *)nullptr, wave_t ? band(SRC.y4, k, own) : b4, pr);
            if constexpr (FUSED) {
                const BandRsrc br = band(SRC.y3, k, own && wave_t);
                rr_y3c = bld((const DT *)nullptr, br, pr);
                rr_y3m = bld((const DT *)nullptr, br, pr - (uint32_t)n2);
            }
        };
        // w1, w2 (3 pairs each) at the own point and the w' ring point
        u32x4 rwa[2][2];  // [own, ring][field]: ud, lr
        u32x2 rwc[2][2];  // c
        auto loadW = [&](int k, bool want) {
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    const float2 *w = f ? SRC.w2 : SRC.w1;
                    rwa[o][f] = bld_raw((const float4 *)nullptr, band(w_udlr(w), k, want), o ? pw : po);
                    rwc[o][f] = bld_raw((const float2 *)nullptr, band(w_c(w, N), k, want), o ? pw : po);
                }
        };

        auto won = [&](int f) { return scp->sel[f].win_on != 0u; };
        auto wlo = [&](int f) { return scp->sel[f].win_lo; };
        auto whi = [&](int f) { return scp->sel[f].win_hi; };

        // ---------------- phases ----------------
        // D^T of planes pv (vertical) and pv + 1 of a staged band, at the point
        // below `up` (LDS pointers: immediate offsets are unsigned)
        auto dT = [&](const lds_f *up, int pv) {
            const lds_f *yv = up + pv * S2, *yh = yv + S2 + W2 - 1;
            return (yv[0] - yv[W2]) + (yh[0] - yh[1]);
        };
        // u+ of step 1 at one point of band kk (yc: its y; yp: the band before;
        // o: the offset of the point above it)
        auto u_at = [&](int kk, float *yc, float *yp, int o, float uo, float y4s) {
            const lds_f *y = at(yc + o);
            float g = dT(y, 0);                          // D^T y1
            if (kk <= n3 - 2) g -= dT(y, 2);             // D_s^T D^T y2
            if (kk >= 1) g += dT(at(yp + o), 2);
            const float x = __builtin_fmaf(-kStepU, __builtin_fmaf(a4, y4s, g), uo);
            return x < ent->c.mu_lo ? ent->c.mu_lo : (x > ent->c.mu_hi ? ent->c.mu_hi : x);
        };
        // FUSED: one value of the next search, z = x - g (e + a4 q)
        auto gather = [&](int f, bool in, float x, float e, float g, float q) {
            gather_ahead(ga, sl, scp->in, f, in, x, e, g, q, ent->c.cand + ((int64_t)f * ent->c.ntiles + lt) * ent->c.capt,
                         &ncand[f], ent->c.capt);
        };
        // otherwise: one value of this slot's search
        auto collect = [&](int f, bool in, float z) {
            const float av = fabsf(z);
            const bool above = in && won(f) && av > whi(f);
            all[f] += in ? (double)av : 0.0;
            cnt[f] += (uint32_t)__popcll(__ballot(above));
            sum[f] += above ? (double)av : 0.0;
            wave_append(in && won(f) && !above && av >= wlo(f), av,
                        ent->c.vcand + ((int64_t)f * ent->c.ntiles + lt) * ent->c.capt, &ncand[f], ent->c.capt);
        };
        // step 1 and u' for band kk; for an own band also (FUSED) steps 2, 3, 6, 7,
        // 8, 14 and the s values of the next search: u+, s+, t+ and
        // q+ = 5 y4' - v (step 15: r = ||q+||); otherwise z_s, z_t and the
        // intermediate of step 14
        auto uphase = [&](int kk, bool own, float *yc, float *yp) {
            float *su = smem + U0 + (kk & 1) * SU;
            const float y4 = y4_of(ru_y4, a4);
            const float un = u_at(kk, yc, yp, oy, ru_u, ru_y4);
            const float up = 2.f * un - ru_u;
            *at(su + ou_w) = up;
            bst_nt((const float *)nullptr, band(DST.u, kk, own), po, un);
            const bool wr = own && own_in;
            const double dl = (double)un - (double)ru_u, uo = (double)ru_u;
            if (wr) {
                du2 += dl * dl;
                u2 += uo * uo;
            }
            const float zs = zs_of(ru_s, y4);
            const float zt = zt_of(ru_t, ru_y3m, oi <= n1 - 2 ? ru_y3c : 0.f, y4, kStepT);
            // 5 (y4 + u'/5) - v, rounded as the duals are stored
            const float y4p = as_stored((const DT *)nullptr, (5.f * y4 + up) - ru_v);
            if constexpr (FUSED) {
                const float sn = soft(zs, scp->in.tau[0]), tn = soft(zt, scp->in.tau[1]);
                bst_nt((const float *)nullptr, band(DST.s, kk, own), po, sn);
                bst_nt((const float *)nullptr, band(DST.t, kk, own), po, tn);
                const float sp = 2.f * sn - ru_s, tp = 2.f * tn - ru_t;
                const float qn = as_stored((const DT *)nullptr, y4p + (sp + tp));
                bst_nt((const DT *)nullptr, band(DST.y4, kk, own), po, qn);
                if (wr) r2 += (double)qn * (double)qn;
                *at(sT + ot_w) = tp;  // the own point: TJ * (oti + 1) + otj
                keep[tid] = make_float4(tn, qn, ru_y3c, ru_y3m);
                if (S ? ring_t : wave_t) {
                    const float x = soft(zt_of(rr_u, rr_y3m, i0 + rui <= n1 - 2 ? rr_y3c : 0.f, y4_of(rr_y4, a4), kStepT),
                                         scp->in.tau[1]);
                    *at(sT + (rui + 1) * TJ + ruj) = 2.f * x - rr_u;
                }
                if (own) gather(0, wr, sn, 0.f, 1.f, qn);
            } else {
                bst_nt((const DT *)nullptr, band(ent->y4p, kk, own), po, y4p);
                if (zst) {
                    bst((const float *)nullptr, band(ent->c.zbuf, kk, own), po, zs);
                    bst((const float *)nullptr, band(ent->c.zbuf + N, kk, own), po, zt);
                }
                if (own) {
                    collect(0, wr, zs);
                    collect(1, wr, zt);
                }
            }
            if (ring_u) *at(su + ru) = 2.f * u_at(kk, yc, yp, ry, rr_u, rr_y4) - rr_u;
        };
        // steps 4, 5 and the w extrapolations (9, 10) at one point of band k; the
        // own point also writes w+ and keeps the own-only planes ud_v', lr_h'
        float wk[2][2];
        // (oy_, ow_: offsets of the point above it in y and of the point in w')
        auto w_at = [&](int k, float *yb, int o, int oy_, int ow_, float v, float h) {
            const lds_f *y = at(yb + oy_) + W2;
            lds_f *wo_at = at(smem + W0 + ow_);
            constexpr int c = 0;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const lds_f *yv = y + 2 * f * S2, *yh = yv + S2;
                float L[6], wo[6], wn[6], o6[6];
                L[0] = v * yv[c];
                L[1] = v * 0.25f * ((yh[c] + yh[c - 1]) + (yh[c + W2] + yh[c + W2 - 1]));
                L[2] = h * 0.25f * ((yv[c] + yv[c - W2]) + (yv[c + 1] + yv[c - W2 + 1]));
                L[3] = h * yh[c];
                L[4] = 0.5f * (yv[c] + yv[c - W2]);
                L[5] = 0.5f * (yh[c] + yh[c - 1]);
                const float thr = f ? kStepW : ent->c.thr1;
                const u32x4 wa = rwa[o][f];
                const u32x2 wc = rwc[o][f];
                wo[0] = __uint_as_float(wa.x);
                wo[1] = __uint_as_float(wa.y);
                wo[2] = __uint_as_float(wa.z);
                wo[3] = __uint_as_float(wa.w);
                wo[4] = __uint_as_float(wc.x);
                wo[5] = __uint_as_float(wc.y);
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) wn[cc] = wo[cc] + kStepW * L[cc];
                shrink2(wn[0], wn[1], thr);
                shrink2(wn[2], wn[3], thr);
                shrink2(wn[4], wn[5], thr);
                if (o == 0) {
                    float2 *wd = f ? DST.w2 : DST.w1;
                    bst_nt((const float4 *)nullptr, band(w_udlr(wd), k, true), po, make_float4(wn[0], wn[1], wn[2], wn[3]));
                    bst_nt((const float2 *)nullptr, band(w_c(wd, N), k, true), po, make_float2(wn[4], wn[5]));
                }
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) o6[cc] = 2.f * wn[cc] - wo[cc];
                o6[0] *= v;
                o6[1] *= v;
                o6[2] *= h;
                o6[3] *= h;
                wo_at[(4 * f + 0) * S1] = o6[1];
                wo_at[(4 * f + 1) * S1] = o6[2];
                wo_at[(4 * f + 2) * S1] = o6[4];
                wo_at[(4 * f + 3) * S1] = o6[5];
                if (o == 0) {
                    wk[f][0] = o6[0];
                    wk[f][1] = o6[3];
                }
            }
        };
        // steps 11, 12 for band k at the own point
        auto yphase = [&](int k, float *yb) {
            const float msk = k <= n3 - 2 ? 1.f : 0.f;
            const int c1 = W1 + 1;
            constexpr int c2 = 0, cu = 0;
            const lds_f *w0 = at(smem + W0 + ow), *yc = at(yb + oy + W2);
            const lds_f *u0 = at(smem + U0 + (k & 1) * SU + ou);
            const lds_f *u1 = at(smem + U0 + ((k & 1) ^ 1) * SU + ou);
            const float du_v = mv * (u0[cu + WU] - u0[cu]), du_h = mh * (u0[cu + 1] - u0[cu]);
            const float dn_v = mv * (u1[cu + WU] - u1[cu]), dn_h = mh * (u1[cu + 1] - u1[cu]);
            // A masked entry (vertical component on the last row, horizontal on
            // the last column) keeps its value, and both sides hold the same
            // one: it is not written at all.
            const bool mx = oi > n1 - 2, my = oj > n2 - 2;
            const uint32_t pp = mx || my ? kNoPix : po;
            const bool edge = __ballot(own_in && (mx != my)) != 0ull;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const lds_f *A = w0 + 4 * f * S1, *B = A + S1, *C = B + S1, *E = C + S1;  // ud_h, lr_v, c_v, c_h
                const float pv = mv * (wk[f][0] + 0.25f * ((B[c1] + B[c1 + W1]) + (B[c1 - 1] + B[c1 + W1 - 1]))
                                       + 0.5f * (C[c1] + C[c1 + W1]));
                const float ph = mh * (wk[f][1] + 0.25f * ((A[c1] + A[c1 + 1]) + (A[c1 - W1] + A[c1 - W1 + 1]))
                                       + 0.5f * (E[c1] + E[c1 + 1]));
                const float2 y = make_float2(yc[2 * f * S2 + c2], yc[(2 * f + 1) * S2 + c2]);
                const float gv = f ? msk * (dn_v - du_v) : du_v;
                const float gh = f ? msk * (dn_h - du_h) : du_h;
                const float2 yn = make_float2(y.x + kStepY * (gv - pv), y.y + kStepY * (gh - ph));
                const BandRsrc b = band(f ? DST.y2 : DST.y1, k, true);
                bst_nt((const P *)nullptr, b, pp, yn);
                if (edge) {
                    bst_comp_nt((const P *)nullptr, b, !mx && my ? po : kNoPix, 0, yn.x);
                    bst_comp_nt((const P *)nullptr, b, mx && !my ? po : kNoPix, 1, yn.y);
                }
            }
        };
        // FUSED: step 13 (y3+ = y3 + D_v t'/5) and the t values of the next search
        // for band kk, once the t' of the rows next to a point are in LDS
        auto tphase = [&](int kk) {
            if constexpr (FUSED) {
                const float4 o = keep[tid];
                // t' of the row above, this one, the row below
                const lds_f *tr = at(sT + (S ? oti * TJ + otj : tid));
                const float tp = tr[TJ];
                const bool ei = oi <= n1 - 2;
                const float yc = as_stored((const DT *)nullptr, ei ? __builtin_fmaf(kStepY, tr[2 * TJ] - tp, o.z) : o.z);
                bst_nt((const DT *)nullptr, band(DST.y3, kk, true), po, yc);
                const float ym = as_stored((const DT *)nullptr, __builtin_fmaf(kStepY, tp - tr[0], o.w));
                gather(1, own_in, o.x, (oi >= 1 ? ym : 0.f) - (ei ? yc : 0.f), kStepT, o.y);
            }
        };

        // ---------------- march through the band chunk ----------------
        // Bands b - 1, b, b + 1, b + 2 of y sit in three buffers in turn; band
        // k + 2 goes from registers to LDS in the interval in which band k is
        // finished, and band k + 3 is requested then.
        float *yA = smem, *yB = smem + 4 * S2, *yC = smem + 8 * S2;  // bands k, k + 1, k + 2 (and k - 1)
        {
            Raw p1[NY], p2[NY], q1[NY], q2[NY];
            loadY(kb - 1, kb >= 1, p1, p2);
            loadY(kb, true, q1, q2);
            loadY(kb + 1, kb + 1 <= ke && kb + 1 < n3, ry1, ry2);
            loadRU(kb, true, true);
            storeY(yC, p1, p2);
            storeY(yA, q1, q2);
            storeY(yB, ry1, ry2);
        }
        __syncthreads();
        uphase(kb, true, yA, yC);
        loadY(kb + 2, kb + 2 <= ke && kb + 2 < n3, ry1, ry2);
        loadRU(kb + 1, kb + 1 < n3, kb + 1 < ke);
        loadW(kb, true);
        __syncthreads();
        tphase(kb);
        __syncthreads();
        int k = kb;
        do {
            const bool more = k + 1 < ke;
            storeY(yC, ry1, ry2);  // band k + 2
            fresh();
            loadY(k + 3, k + 3 <= ke && k + 3 < n3, ry1, ry2);
            fresh();
            uphase(k + 1, more, yB, yA);
            fresh();
            loadRU(k + 2, k + 2 <= ke && k + 2 < n3, k + 2 < ke);
            fresh();
            w_at(k, yA, 0, oy, ow_w, mv, mh);
            fresh();
            if (ring_w) w_at(k, yA, 1, rwy, rww, rmv, rmh);
            fresh();
            loadW(k + 1, more);
            __syncthreads();
            fresh();
            yphase(k, yA);
            fresh();
            if (more) tphase(k + 1);
            __syncthreads();
            float *const y = yA;
            yA = yB;
            yB = yC;
            yC = y;
        } while (++k < ke);

#undef SRC
#undef DST
        // the tile's FP64 partials: stopping sums; the residual's norm and the
        // values above the windows, or the window statistics of the search
        fresh();
        const int nt = ent->c.ntiles;
        if constexpr (FUSED) {
            tile_sums<NT>(du2, u2, r2, ga, sl, red, ent->c.part + 3 * lt, ent->c.winpart + 4 * lt,
                          ent->c.winpart + 4 * (nt + lt));
        } else {
            const bool one = (tid & 63) == 0;
            double acc[NS] = {du2, u2, one ? (double)cnt[0] : 0.0, sum[0], all[0],
                              one ? (double)cnt[1] : 0.0, sum[1], all[1]};
            block_sums<NS, NT>(acc, red);
            if (tid == 0) {
                ent->c.part[2 * lt] = acc[0];
                ent->c.part[2 * lt + 1] = acc[1];
                for (int f = 0; f < 2; ++f)
                    for (int q = 0; q < 3; ++q) ent->c.winpart[((int64_t)f * nt + lt) * 3 + q] = acc[2 + 3 * f + q];
            }
        }
        if (tid == 0) {
            ent->c.ccount[lt] = ncand[0];
            ent->c.ccount[nt + lt] = ncand[1];
        }
        if constexpr (!FUSED) __syncthreads();  // red is reused by the next tile
    }
}

template <typename DT>
__global__ __launch_bounds__(NPT) void k_init(Dims d, const float *v, Side<DT> s0, Side<DT> s1,
                                              DevScalars *sc, double eps, double tol, double alpha,
                                              double beta)
{
    using P = typename PairOf<DT>::type;
    const int64_t N = d.plane;
    const int64_t stride = (int64_t)gridDim.x * NPT;
    const float2 z2 = make_float2(0.f, 0.f);
    for (int64_t q = (int64_t)blockIdx.x * NPT + threadIdx.x; q < N; q += stride) {
        s0.u[q] = v[q];
        s0.s[q] = 0.f;
        s0.t[q] = 0.f;
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            s0.w1[g * N + q] = z2;
            s0.w2[g * N + q] = z2;
        }
        // y1, y2 on both sides: their masked entries are never rewritten
        st2((P *)s0.y1 + q, z2);
        st2((P *)s0.y2 + q, z2);
        st2((P *)s1.y1 + q, z2);
        st2((P *)s1.y2 + q, z2);
        st(s0.y3 + q, 0.f);
        st(s0.y4 + q, 0.f);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        init_scalars(sc, eps, tol, alpha, beta, 0.2);  // the y4 step printed after eq. (24)
    }
}

// State copy in/out between separate FP32 planes (the ABI layout) and the
// workspace layout. var: GEO_VAR_*; planes: 1, 6 or 2.
template <typename DT>
__global__ __launch_bounds__(NPT) void k_state_io(Dims d, Side<DT> s0, Side<DT> s1, DevScalars *sc,
                                                  int var, const float *v, float *out,
                                                  const float *in)
{
    using P = typename PairOf<DT>::type;
    const int64_t N = d.plane;
    const int par = (int)(sc->iter & 1u);
    const Side<DT> s = par ? s1 : s0;
    const int planes = (var == GEO_VAR_W1 || var == GEO_VAR_W2) ? 6
                       : (var == GEO_VAR_Y1 || var == GEO_VAR_Y2) ? 2 : 1;
    const int64_t total = N * planes;
    const int64_t stride = (int64_t)gridDim.x * NPT;
    const float a4 = (float)sc->a4;
    for (int64_t g = (int64_t)blockIdx.x * NPT + threadIdx.x; g < total; g += stride) {
        const int pl = (int)(g / N);
        const int64_t q = g - (int64_t)pl * N;
        float2 *wp = var == GEO_VAR_W1 ? s.w1 : s.w2;
        P *yp = var == GEO_VAR_Y1 ? s.y1 : s.y2;
        if (out) {
            float x = 0.f;
            switch (var) {
            case GEO_VAR_U: x = s.u[q]; break;
            case GEO_VAR_S: x = s.s[q]; break;
            case GEO_VAR_T: x = s.t[q]; break;
            case GEO_VAR_W1:
            case GEO_VAR_W2: {
                const float2 w = *w_pair(wp, N, pl >> 1, q);
                x = (pl & 1) ? w.y : w.x;
            } break;
            case GEO_VAR_Y1:
            case GEO_VAR_Y2: {
                const float2 y = ld2(yp + q);
                x = pl ? y.y : y.x;
            } break;
            case GEO_VAR_Y3: x = ld(s.y3 + q); break;
            default: x = y4_of(ld(s.y4 + q), a4); break;
            }
            out[g] = x;
        } else {
            switch (var) {
            case GEO_VAR_U: s.u[q] = in[q]; break;
            case GEO_VAR_S: s.s[q] = in[q]; break;
            case GEO_VAR_T: s.t[q] = in[q]; break;
            case GEO_VAR_W1:
            case GEO_VAR_W2:
                if ((pl & 1) == 0) *w_pair(wp, N, pl >> 1, q) = make_float2(in[g], in[g + N]);
                break;
            case GEO_VAR_Y1:
            case GEO_VAR_Y2:
                // both sides: the sweep never rewrites the masked entries
                if (pl == 0) {
                    const float2 y = make_float2(in[q], in[q + N]);
                    st2((var == GEO_VAR_Y1 ? s0.y1 : s0.y2) + q, y);
                    st2((var == GEO_VAR_Y1 ? s1.y1 : s1.y2) + q, y);
                }
                break;
            case GEO_VAR_Y3: st(s.y3 + q, in[q]); break;
            default: st(s.y4 + q, in[q]); break;
            }
        }
    }
}

// After a state load: y4 loaded as-is is read back with the factor 1, and
// the threshold predictions are dropped (the loaded state does not continue
// the previous run).
__global__ void k_state_loaded(DevScalars *sc, int var)
{
    if (threadIdx.x == 0) {
        if (var == GEO_VAR_Y4) sc->a4 = 1.0;
        for (int f = 0; f < 2; ++f) {
            sc->sel[f].win_on = 0u;
            sc->sel[f].tau_prev = 0.0;
            sc->sel[f].tau_prev2 = 0.0;
            sc->sel[f].tau_prev3 = 0.0;
            sc->sel[f].done = 1u;
        }
        sc->zstore = 1u;
        sc->calm = 0u;
    }
}

template <typename DT>
Side<DT> side_of(void *ws, const Layout &L, int p)
{
    char *b = (char *)ws;
    Side<DT> s;
    s.u = (float *)(b + L.u[p]);
    s.s = (float *)(b + L.s[p]);
    s.t = (float *)(b + L.t[p]);
    s.w1 = (float2 *)(b + L.w1[p]);
    s.w2 = (float2 *)(b + L.w2[p]);
    s.y1 = (typename Side<DT>::P *)(b + L.y1[p]);
    s.y2 = (typename Side<DT>::P *)(b + L.y2[p]);
    s.y3 = (DT *)(b + L.y3[p]);
    s.y4 = (DT *)(b + L.y4[p]);
    return s;
}

int grid_for(int64_t n)
{
    int64_t b = (n + NPT - 1) / NPT;
    return (int)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

// Resident blocks of the sweep on this device, of the forms in use (BF16: 8 x 128 and
// the small one) the smaller number; queried once per process, storage and size.
template <typename DT, bool SMALL>
int resident_grid()
{
    // (thread-safe initialisation of a local static)
    static const int cached = [] {
        int dev = 0, cus = 256;
        if (hipGetDevice(&dev) == hipSuccess) {
            hipDeviceProp_t prop;
            if (hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
        }
        constexpr bool fused = sizeof(DT) == 4;
        auto per_cu = [](auto kernel, int threads) {
            int p = 1;
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(&p, kernel, threads, 0) == hipSuccess && p >= 1 ? p : 1;
        };
        if constexpr (SMALL) return cus * per_cu(k_sweep<DT, kSmallForm, fused>, Small::NT);
        int p = per_cu(k_sweep<DT, 0, fused>, Wide::NT);
        if constexpr (fused) {
            const int p1 = per_cu(k_sweep<DT, 1, true>, Wide::NT);
            if (p1 < p) p = p1;
        }
        return cus * p;
    }();
    return cached;
}

template <typename DT>
void cube_entry_t(CubeArgs<DT> *a, const Dims &d, const float *v, void *ws, const Layout &L, const geo_params *p,
                  int n_iter, int b0, int *ntiles, int *nb)
{
    char *b = (char *)ws;
    memset(a, 0, sizeof *a);
    CubeCommon &c = a->c;
    c.d = d;
    c.v = v;
    c.sc = (DevScalars *)(b + L.scalars);
    c.part = (double *)(b + L.partials);
    c.winpart = (double *)(b + L.winpart);
    c.hist = (Hist *)(b + L.hist);
    c.rec = (FbRec *)(b + L.rec);
    constexpr bool fused = sizeof(DT) == 4;
    c.ahead = fused ? 1u : 0u;
    if (fused) {
        c.cand = (float4 *)(b + L.cand);
    } else {
        c.vcand = (float *)(b + L.cand);
        c.zbuf = (float *)(b + L.zbuf);
    }
    c.ccount = (uint32_t *)(b + L.ccount);
    c.g = cube_grid(d.n1, d.n2, d.n3, p->band_chunk, sweep_grid_of(sizeof(DT), 0, 1 << 30), (int)sizeof(DT));
    c.ntiles = c.g.blocks();
    c.capt = (int)(L.cap / c.ntiles);
    c.thr1 = (float)(p->omega * 0.25);
    c.zt_step = kStepT;
    c.mu_lo = (float)p->mu_lo;
    c.mu_hi = (float)p->mu_hi;
    c.tol = p->tol;
    c.alpha = p->alpha;
    c.beta = p->beta;
    c.limit = (uint32_t)n_iter;
    a->side[0] = side_of<DT>(ws, L, 0);
    a->side[1] = side_of<DT>(ws, L, 1);
    if (!fused) {
        // sweep B: strips of kSweepBRows rows; never more blocks than the
        // partials hold
        const int64_t items = (int64_t)d.n3 * ((d.n1 + kSweepBRows - 1) / kSweepBRows) * (d.n2 / sweep_b_cpt(d.n2));
        const int pb = point_blocks(items);
        c.nb = pb < kSweepBBlocks ? pb : kSweepBBlocks;
        c.b0 = b0;
        a->y4p = (DT *)(b + L.y4p);
        for (int p = 0; p < 2; ++p) {
            c.bin[p][0] = a->side[p].s;
            c.bin[p][1] = a->side[p].t;
            c.bin[p][2] = a->side[p].y3;
            c.bin[p][3] = a->side[p].y4;
            c.bin[p][4] = a->y4p;
        }
        const size_t N = (size_t)d.plane;
        c.bin_bytes[0] = c.bin_bytes[1] = N * sizeof(float);
        c.bin_bytes[2] = c.bin_bytes[3] = c.bin_bytes[4] = N * sizeof(DT);
    }
    *ntiles = c.ntiles;
    *nb = c.nb;
}

constexpr int kPrefetchBlocks = 240;  // cache prefetch beside the search (BF16)

template <typename DT, int S>
void launch_sweep(const CubeArgs<DT> *cubes, const LaunchShape &sh, hipStream_t st)
{
    if (sh.form_tiles[S] > 0)
        hipLaunchKernelGGL((k_sweep<DT, S, sizeof(DT) == 4>), dim3(sh.form_grid[S]), dim3(PlanesOf<S>::NT), 0, st, cubes, sh);
}

hipError_t slot_fused(const void *table, const LaunchShape &sh, hipStream_t st, hipEvent_t *ev, int nev)
{
    const CubeArgs<float> *cubes = (const CubeArgs<float> *)table;
    if (nev >= 4) (void)hipEventRecord(ev[0], st);
    hipError_t e = launch_fallback(table, 4, sh, st);
    if (e != hipSuccess) return e;
    if (nev >= 2) (void)hipEventRecord(ev[nev >= 4 ? 1 : 0], st);
    // one persistent launch per form present (each takes the tiles of its cubes)
    launch_sweep<float, 0>(cubes, sh, st);
    launch_sweep<float, 1>(cubes, sh, st);
    launch_sweep<float, kSmallForm>(cubes, sh, st);
    if (nev >= 2) (void)hipEventRecord(ev[nev >= 4 ? 2 : 1], st);
    e = launch_search(table, (int)sizeof(CubeEntry), sh.ncubes, st);
    if (nev >= 4) (void)hipEventRecord(ev[3], st);
    return e;
}

hipError_t slot_two(const void *table, const LaunchShape &sh, hipStream_t st, hipEvent_t *ev, int nev)
{
    const CubeArgs<bf16> *cubes = (const CubeArgs<bf16> *)table;
    const int stride = (int)sizeof(CubeEntry);
    if (nev >= 2) (void)hipEventRecord(ev[0], st);
    launch_sweep<bf16, 0>(cubes, sh, st);
    launch_sweep<bf16, kSmallForm>(cubes, sh, st);
    if (nev >= 2) (void)hipEventRecord(ev[1], st);
    hipError_t e = launch_select_window(table, stride, sh.ncubes, kPrefetchBlocks, st);
    if (e == hipSuccess) e = launch_fallback(table, 2, sh, st);
    if (e != hipSuccess) return e;
    if (nev >= 4) (void)hipEventRecord(ev[2], st);
    e = launch_sweep_b(table, sh, st);
    if (e == hipSuccess) e = launch_finalize(table, stride, sh.ncubes, st);
    if (nev >= 4) (void)hipEventRecord(ev[3], st);
    return e;
}

}  // namespace

void cube_entry(CubeEntry *e, const Dims &d, const float *v, void *ws, const Layout &L, const geo_params *p,
                int n_iter, int b0, int *ntiles, int *nb)
{
    if (L.dual_bytes == 2)
        cube_entry_t<bf16>(reinterpret_cast<CubeArgs<bf16> *>(e->bytes), d, v, ws, L, p, n_iter, b0, ntiles, nb);
    else
        cube_entry_t<float>(reinterpret_cast<CubeArgs<float> *>(e->bytes), d, v, ws, L, p, n_iter, b0, ntiles, nb);
}

// Persistent sweep grid of a form: resident blocks, at most one per tile, a multiple
// of the 8 XCDs when it is smaller than the tile count.
int sweep_grid_of(int dual_bytes, int form, int tiles)
{
    const int G = form == kSmallForm ? (dual_bytes == 2 ? resident_grid<bf16, true>() : resident_grid<float, true>())
                                     : (dual_bytes == 2 ? resident_grid<bf16, false>() : resident_grid<float, false>());
    if (G >= tiles) return tiles;
    return G >= 8 ? (G & ~7) : G;
}

hipError_t launch_slot(const void *table, int dual_bytes, const LaunchShape &sh, hipStream_t st,
                       hipEvent_t *ev, int nev)
{
    if (!ev) nev = 0;
    return dual_bytes == 2 ? slot_two(table, sh, st, ev, nev) : slot_fused(table, sh, st, ev, nev);
}

hipError_t launch_state_loaded(DevScalars *sc, int var, hipStream_t st)
{
    hipLaunchKernelGGL(k_state_loaded, dim3(1), dim3(64), 0, st, sc, var);
    return hipGetLastError();
}

hipError_t launch_init(const Dims &d, const float *v, void *ws, const Layout &L, double eps,
                       double tol, double alpha, double beta, hipStream_t st)
{
    DevScalars *sc = (DevScalars *)((char *)ws + L.scalars);
    if (L.dual_bytes == 2)
        hipLaunchKernelGGL(k_init<bf16>, dim3(grid_for(d.plane)), dim3(NPT), 0, st, d, v,
                           side_of<bf16>(ws, L, 0), side_of<bf16>(ws, L, 1), sc, eps, tol, alpha, beta);
    else
        hipLaunchKernelGGL(k_init<float>, dim3(grid_for(d.plane)), dim3(NPT), 0, st, d, v,
                           side_of<float>(ws, L, 0), side_of<float>(ws, L, 1), sc, eps, tol, alpha,
                           beta);
    return hipGetLastError();
}

hipError_t launch_state_io(const Dims &d, void *ws, const Layout &L, int var, const float *v,
                           float *out, const float *in, hipStream_t st)
{
    DevScalars *sc = (DevScalars *)((char *)ws + L.scalars);
    const int planes = (var == GEO_VAR_W1 || var == GEO_VAR_W2) ? 6
                       : (var == GEO_VAR_Y1 || var == GEO_VAR_Y2) ? 2 : 1;
    const int grid = grid_for(d.plane * planes);
    if (L.dual_bytes == 2)
        hipLaunchKernelGGL(k_state_io<bf16>, dim3(grid), dim3(NPT), 0, st, d, side_of<bf16>(ws, L, 0),
                           side_of<bf16>(ws, L, 1), sc, var, v, out, in);
    else
        hipLaunchKernelGGL(k_state_io<float>, dim3(grid), dim3(NPT), 0, st, d,
                           side_of<float>(ws, L, 0), side_of<float>(ws, L, 1), sc, var, v, out, in);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !in) return e;
    return L.dual_bytes == 2 ? launch_state_loaded(sc, var, st)
                             : launch_loaded(sc, (Hist *)((char *)ws + L.hist), var, st);
}

}  // namespace geo
