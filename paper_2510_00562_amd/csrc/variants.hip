// Problem (15) with the GeoSSTV term replaced by one of the regularizers the
// paper compares against (Sec. IV-A), solved by the same P-PDS (eq. (7)):
//   SSTV:   ||D D_s u||_1
//   HSSTV1: ||(D D_s u, omega D u)||_1
//   HSSTV2: sum over voxels of the l2 norm of (D D_s u, omega D u) there
// Primal blocks (u, s, t), dual blocks (y1 for A u, y3 for D_v t, y4 for
// u + s + t); step sizes from eq. (8) with the operator-norm bounds
// ||D D_s||^2 <= 32, ||omega D||^2 <= 8 omega^2, ||D_v||^2 <= 4:
//   u 1/(||A||^2 + 1), s 1, t 1/5, y 1/3.
//
// One launch slot per iteration, on the caller's stream, over a one-entry
// launch table in the workspace, as in the main solver's FP32 form:
//   histogram passes (fallback.hip): thresholds that the last search missed;
//   sweep:  one pass over the state. u+ = P_box(u - g_u (A^T y1 + y4)); s+ and
//           t+ (soft thresholds of z_s = s - y4 and z_t = t - g_t (D_v^T y3 +
//           y4)); the extrapolations x' = 2 x+ - x; y1 += g_y A u' and the
//           conjugate prox of the regularizer (a clip to [-1, 1], or each
//           4-entry group scaled into the unit l2 ball); y3 += g_y D_v t'; the
//           y4 residual; the FP64 partial sums and the inputs of the next search;
//   search (search.hip): the fidelity-ball factor (y4 - g_y P_B(y4/g_y) =
//           c g_y (y4/g_y - v), c = max(0, 1 - eps/r), applied when y4 is next
//           read), the stopping rule, the next thresholds.
//
// What bounds the sweep is HBM: 60 bytes per voxel (SSTV: 7 state words each
// way and v) or 76 (HSSTV). A workgroup owns an 8 x 64 pixel tile and marches
// through a chunk of bands (narrow cubes: other tiles, or none, var_tiles); y1 is staged in LDS with a 1-pixel halo, three bands
// in turn, u' with the row below and the column to the right, t' with the rows
// above and below; the next bands' loads are in flight meanwhile (the buffer
// path, common.hpp: band_of). In two kernels with the search between them, each
// reading s, t, y3, y4 and y1, an iteration of 256 x 256 x 128 took 182 us (SSTV)
// and 226 us (HSSTV2), now 121 and 157 (the sweep 109 and 143: 4.6 and 4.5 TB/s);
// of 64 x 64 x 16 45 us, now 20 (SSTV); of 512 x 512 x 224 1165 and 1435 us, now
// 773 and 973 (the sweep 728 and 930: 4.8 TB/s).
#include <math.h>
#include <string.h>

#include <vector>

#include "host_box.hpp"
#include "radix.hpp"

namespace geo {

namespace {

constexpr int VT = 1024;          // init and copy kernels
constexpr int kVarBlocks = 8192;  // their blocks at most
// The sweep's tile: 512 threads, one per point. Several blocks fit a CU, so one
// block's barriers overlap another's loads, and 64 columns waste little of
// ragged widths. Cubes that fill little of such tiles take others of as many points
// and no larger halo (var_tiles below), or the form without tiles.
constexpr int kTI = 8, kTJ = 64, NT = kTI * kTJ, kSpan = kTI + kTJ;
// LDS planes of a tile of rows x cols <= NT points, rows + cols <= kSpan and cols <=
// kTJ (8 x 64 fills them): y1 with a 1-pixel halo, u' with the (+1, +1) ring, t' with
// the rows above and below. A tile of fewer points leaves the last word of the
// last two free: idle threads write there.
constexpr int S2 = NT + 2 * kSpan + 4, NY = (S2 + NT - 1) / NT;
constexpr int SU = NT + kSpan + 1, ST = NT + 2 * kTJ;
constexpr int T0 = NT / 2;  // first thread of the t' ring
static_assert(T0 >= kSpan + 1 && T0 % 64 == 0 && T0 + 2 * kTJ <= NT, "one ring role per wavefront");
// Wavefronts per SIMD asked of the compiler: three blocks per CU in 80 registers.
// With two (128 registers allowed, 91 taken) the HSSTV2 sweep of 256 x 256 x 128
// takes 140 instead of 143 us, the SSTV sweep of 145 x 141 x 103 50 instead of 43.
constexpr int kVarMinWaves = 6;
// Bands of fewer pixels go through the buffer path (an 8-byte pair of any pixel
// lies below the offset of a missing one); larger ones by 64-bit addresses.
constexpr uint32_t kVarPixels = 1u << 27;
// The index of a missing pixel: kNoPix for the buffer path, and with 64-bit
// addresses, where a large band has a pixel of that index, one that none has
// (N < 2^31).
template <bool BUF>
constexpr uint32_t kNone = BUF ? kNoPix : 0xffffffffu;
static_assert(kVarPixels <= kNone<true> && 1u << 31 <= kNone<false>, "no pixel has the index of a missing one");

struct VarArgs {
    Dims d;
    int variant;
    float gu, gt, gy, omega;  // step sizes, balance
    float mu_lo, mu_hi;
    const float *v;
    DevScalars *sc;
    float *u[2], *t[2], *y3[2], *q[2];  // ping-pong by iteration parity
    float2 *ya[2], *yb[2];              // y1: (D_v, D_h) D_s u, and omega (D_v, D_h) u (HSSTV)
    float *s;                           // in place (a point reads and writes only its own)
    double *part;                       // [3 * slots]
    double *winpart;                    // [2][slots][4]
    float4 *cand;                       // [2][slots][capt]
    uint32_t *ccount;                   // [2][slots]
    uint32_t *flags;                    // of the launch table
    int ti, tj, tk, kc;                 // tiles along i, j, band chunks; bands per chunk
    int slots, per, capt;               // slots of the search, consecutive tiles (voxels) of one, candidates of one
    int rows, cols;                     // points of a tile (0: k_var_flat)
};

// Loads and stores of one band of an array at a pixel (kNone: none): through
// the buffer path, or (bands of kVarPixels pixels and more) by 64-bit addresses.
template <bool BUF, typename T>
struct Band {
    BandRsrc r;
    T *p;
    bool any;
    __device__ __forceinline__ Band(T *base, int k, uint32_t np, bool want)
    {
        if constexpr (BUF) {
            r = band_of(base, (int64_t)k * np, want ? np : 0u);
        } else {
            p = base + (int64_t)k * np;
            any = want;
        }
    }
};
template <bool BUF>
__device__ __forceinline__ float bget(const Band<BUF, const float> &b, uint32_t pix)
{
    if constexpr (BUF) return bld((const float *)nullptr, b.r, pix);
    else return b.any && pix != kNone<BUF> ? b.p[pix] : 0.f;
}
template <bool BUF>
__device__ __forceinline__ float2 bget(const Band<BUF, const float2> &b, uint32_t pix)
{
    if constexpr (BUF) return pair_of(bld_raw((const float2 *)nullptr, b.r, pix));
    else return b.any && pix != kNone<BUF> ? b.p[pix] : make_float2(0.f, 0.f);
}
template <bool BUF, typename T>
__device__ __forceinline__ void bput(const Band<BUF, T> &b, uint32_t pix, T x)
{
    if constexpr (BUF) bst_nt((const T *)nullptr, b.r, pix, x);
    else if (b.any && pix != kNone<BUF>) b.p[pix] = x;
}

// The conjugate prox of the regularizer on one voxel's entries of y1.
template <int P>
__device__ __forceinline__ void dual_prox(int variant, float (&y)[P])
{
    if (P == 4 && variant == GEO_REG_HSSTV2) {
        const float nr = sqrtf((y[0] * y[0] + y[1] * y[1]) + (y[P - 2] * y[P - 2] + y[P - 1] * y[P - 1]));
#pragma unroll
        for (int q = 0; q < P; ++q) y[q] = nr > 1.f ? y[q] / nr : y[q];
    } else {
#pragma unroll
        for (int q = 0; q < P; ++q) y[q] = fminf(fmaxf(y[q], -1.f), 1.f);
    }
}

// P: planes of y1 (2 SSTV, 4 HSSTV). FIT: tiles of a.rows x a.cols, else of 8 x 64.
template <int P, bool BUF, bool FIT>
__global__ __launch_bounds__(NT, kVarMinWaves) void k_var_sweep(VarArgs args)
{
    __shared__ float sY[3 * P * S2];         // three bands of y1, planes one after another
    __shared__ float sU[2 * SU];             // u' by band parity
    __shared__ float sT[ST];                 // t' with the rows above and below
    __shared__ float4 keep[NT];              // t+, q+, y3, y3 of the row above
    __shared__ double red[10 * (NT / 64)];
    // (SSTV: with these sums in registers the sweep spills and takes 2.3% longer;
    // HSSTV: 8 KB more would leave room for two blocks per CU)
    constexpr bool slope_lds = P == 2;
    __shared__ double sSlope[slope_lds ? 2 * NT : 1];
    __shared__ uint32_t ncand[2];
    const int tid = threadIdx.x, lane = tid & 63;
    // Each phase reads the pointers and the window with scalar loads of its own
    // (sweep.hip does, and says why).
    const const4<VarArgs> *ap = (const const4<VarArgs> *)__builtin_amdgcn_kernarg_segment_ptr();
    const const4<VarArgs> &a = *ap;
    const bool idle_now = idle(args.sc);
    if (blockIdx.x == 0 && tid == 0) {
        // what the search of this slot reads of the state it rewrites; the
        // histogram passes are over
        args.sc->view = {args.sc->in.a_lo, args.sc->in.a_hi, args.sc->in.a_c, idle_now ? 1u : 0u};
        passes_over(args.flags);
    }
    if (idle_now) return;
    const const4<DevScalars> &sc = *(const4<DevScalars> *)args.sc;
    const const4<DevScalars> *scp = &sc;
    auto fresh = [&]() {
        asm volatile("" : "+s"(ap), "+s"(scp));
        __builtin_amdgcn_sched_barrier(0);
    };
    const int par = (int)(sc.iter & 1u);
    const int n1 = a.d.n1, n2 = a.d.n2, n3 = a.d.n3;
    const uint32_t np = (uint32_t)n1 * (uint32_t)n2;
    const float a4 = sc.in.a4;
    // blocks of one XCD take consecutive slots, whose halos meet in its L2
    const uint32_t pern = (uint32_t)a.slots >> 3, b0 = blockIdx.x;
    const int slot = (int)(b0 < 8u * pern ? (b0 & 7u) * pern + (b0 >> 3) : b0);
    if (tid < 2) ncand[tid] = 0u;  // published by the first barrier of a march
    const int TI = FIT ? a.rows : kTI, TJ = FIT ? a.cols : kTJ;
    const int W2 = TJ + 2, WU = TJ + 1;          // LDS row lengths
    const bool act = !FIT || tid < TI * TJ;      // the thread has a point of the tile
    const int oti = act ? tid / TJ : 0, otj = act ? tid % TJ : 0;
    const int ou_w = act ? oti * WU + otj : SU - 1, ot_w = act ? TJ + tid : ST - 1;
    // ring roles: u' (the first threads) and t' (T0 on), a wavefront has one
    int rui = 0, ruj = 0;
    const bool ring_u = tid < TI + TJ + 1;
    const int wave0 = __builtin_amdgcn_readfirstlane(tid);
    const bool wave_t = wave0 >= T0 && wave0 < T0 + 2 * TJ;
    const bool ring_t = FIT ? tid >= T0 && tid < T0 + 2 * TJ : wave_t;
    if (ring_u) {
        rui = tid < WU ? TI : tid - WU;
        ruj = tid < WU ? tid : TJ;
    }
    if (ring_t) {
        rui = tid - T0 < TJ ? -1 : TI;
        ruj = FIT ? (tid - T0 < TJ ? tid - T0 : tid - T0 - TJ) : (tid - T0) % TJ;
    }
    double du2 = 0.0, u2 = 0.0, r2 = 0.0;
    Gathered ga;
    std::conditional_t<slope_lds, SlopeLds<NT>, SlopeRegs> sl;
    if constexpr (slope_lds) {
        sl.x = (__attribute__((address_space(3))) double *)sSlope + tid;
        sSlope[tid] = sSlope[NT + tid] = 0.0;
    }

    const int t1 = min((slot + 1) * a.per, a.ti * a.tj * a.tk);
    for (int t = slot * a.per; t < t1; ++t) {
        const int rest = t / a.tj;
        const int j0 = (t % a.tj) * TJ, i0 = (rest % a.ti) * TI, kb = (rest / a.ti) * a.kc;
        const int ke = min(kb + a.kc, n3);
        auto pixel = [&](int i, int j) {
            return i >= 0 && i < n1 && j >= 0 && j < n2 ? (uint32_t)i * (uint32_t)n2 + (uint32_t)j : kNone<BUF>;
        };
        // (the pixel of the row above: 64-bit addresses need its bound checked,
        // the buffer path drops a negative offset)
        auto row_above = [&](uint32_t p, int i) {
            return BUF ? p - (uint32_t)n2 : (p != kNone<BUF> && i >= 1 ? p - (uint32_t)n2 : kNone<BUF>);
        };
        const int oi = i0 + oti, oj = j0 + otj;
        const uint32_t po = act ? pixel(oi, oj) : kNone<BUF>, pom = row_above(po, oi);
        const bool own_in = po != kNone<BUF>;
        const int ri = i0 + rui, rj = j0 + ruj;
        const uint32_t pr = ring_u || ring_t ? pixel(ri, rj) : kNone<BUF>, prm = row_above(pr, ri);
        uint32_t py[NY];
#pragma unroll
        for (int n = 0; n < NY; ++n) {
            const int p = tid + NT * n;
            py[n] = p < (TI + 2) * W2 ? pixel(i0 - 1 + p / W2, j0 - 1 + p % W2) : kNone<BUF>;
        }
        const bool ei = oi <= n1 - 2, ej = oj <= n2 - 2;

        // ---------------- loads ----------------
        struct Y {
            float2 a[NY], b[P == 4 ? NY : 1];
        };
        auto loadY = [&](int k, bool want, Y &y) {
            const Band<BUF, const float2> ba(ap->ya[par], k, np, want);
#pragma unroll
            for (int n = 0; n < NY; ++n) y.a[n] = bget<BUF>(ba, py[n]);
            if constexpr (P == 4) {
                const Band<BUF, const float2> bb(ap->yb[par], k, np, want);
#pragma unroll
                for (int n = 0; n < NY; ++n) y.b[n] = bget<BUF>(bb, py[n]);
            }
        };
        auto storeY = [&](float *buf, const Y &y) {
#pragma unroll
            for (int n = 0; n < NY; ++n) {
                const int p = tid + NT * n;
                if (NT * (n + 1) <= S2 || p < S2) {
                    buf[p] = y.a[n].x;
                    buf[S2 + p] = y.a[n].y;
                    if constexpr (P == 4) {
                        buf[2 * S2 + p] = y.b[n].x;
                        buf[3 * S2 + p] = y.b[n].y;
                    }
                }
            }
        };
        // the own point; u and q at the u' ring point, or t, q and y3 at the t' one
        float lu, lq, lv, ls, lt, l3c, l3m, xu, xq, x3c, x3m;
        auto loadRU = [&](int k, bool want, bool own) {
            const Band<BUF, const float> bu(ap->u[par], k, np, want), bq(ap->q[par], k, np, want);
            const Band<BUF, const float> bt(ap->t[par], k, np, own), b3(ap->y3[par], k, np, own);
            lu = bget<BUF>(bu, po);
            lq = bget<BUF>(bq, po);
            ls = bget<BUF>(Band<BUF, const float>(ap->s, k, np, own), po);
            lt = bget<BUF>(bt, po);
            l3c = bget<BUF>(b3, po);
            l3m = bget<BUF>(b3, pom);
            lv = bget<BUF>(Band<BUF, const float>(ap->v, k, np, own), po);
            const Band<BUF, const float> bx(wave_t ? ap->t[par] : ap->u[par], k, np, wave_t ? own : want);
            const Band<BUF, const float> br(ap->y3[par], k, np, own && wave_t);
            xu = bget<BUF>(bx, pr);
            xq = bget<BUF>(bq, pr);
            x3c = bget<BUF>(br, pr);
            x3m = bget<BUF>(br, prm);
        };

        // ---------------- phases ----------------
        // D^T of a staged pair of planes at the point c (v, h: its edges exist)
        auto dT = [&](const float *y, int c, bool v, bool h) {
            float x = y[c - W2];
            x -= v ? y[c] : 0.f;
            x += y[S2 + c - 1];
            x -= h ? y[S2 + c] : 0.f;
            return x;
        };
        // u+ at one point of band k (yc: its y1, yp: the band before)
        auto u_at = [&](int k, const float *yc, const float *yp, int ui, int uj, bool v, bool h, float uo, float qo) {
            const int c = (ui + 1) * W2 + (uj + 1);
            float g = 0.f;
            if (k >= 1) g += dT(yp, c, v, h);
            if (k <= n3 - 2) g -= dT(yc, c, v, h);
            if constexpr (P == 4) g = __builtin_fmaf(ap->omega, dT(yc + 2 * S2, c, v, h), g);
            const float x = __builtin_fmaf(-ap->gu, g + y4_of(qo, a4), uo);
            return fminf(fmaxf(x, ap->mu_lo), ap->mu_hi);
        };
        auto slice = [&](int f) { return ap->cand + ((int64_t)f * ap->slots + slot) * ap->capt; };
        auto uphase = [&](int k, bool own, const float *yc, const float *yp) {
            float *su = sU + (k & 1) * SU;
            const float un = u_at(k, yc, yp, oti, otj, ei, ej, lu, lq);
            const float u0 = 2.f * un - lu;
            su[ou_w] = u0;
            bput(Band<BUF, float>(ap->u[par ^ 1], k, np, own), po, un);
            const bool wr = own && own_in;
            const double dl = (double)un - (double)lu, ud = (double)lu;
            if (wr) {
                du2 += dl * dl;
                u2 += ud * ud;
            }
            const float y4 = y4_of(lq, a4);
            const float sn = soft(zs_of(ls, y4), scp->in.tau[0]);
            const float tn = soft(zt_of(lt, l3m, ei ? l3c : 0.f, y4, ap->gt), scp->in.tau[1]);
            bput(Band<BUF, float>(ap->s, k, np, own), po, sn);
            bput(Band<BUF, float>(ap->t[par ^ 1], k, np, own), po, tn);
            const float sp = 2.f * sn - ls, tp = 2.f * tn - lt;
            // y4'/g_y - v = (a4/g_y) q + u' + s' + t' - v
            const float qn = (a4 / ap->gy) * lq + ((u0 + sp) + tp) - lv;
            bput(Band<BUF, float>(ap->q[par ^ 1], k, np, own), po, qn);
            if (wr) r2 += (double)qn * (double)qn;
            sT[ot_w] = tp;
            keep[tid] = make_float4(tn, qn, l3c, l3m);
            if (ring_t) {
                const float x = soft(zt_of(xu, x3m, ri <= n1 - 2 ? x3c : 0.f, y4_of(xq, a4), ap->gt), scp->in.tau[1]);
                sT[(rui + 1) * TJ + ruj] = 2.f * x - xu;
            }
            if (ring_u)
                su[rui * WU + ruj] = 2.f * u_at(k, yc, yp, rui, ruj, ri <= n1 - 2, rj <= n2 - 2, xu, xq) - xu;
            if (own) gather_ahead(ga, sl, scp->in, 0, wr, sn, 0.f, 1.f, qn, slice(0), &ncand[0], ap->capt);
        };
        // y1+ of band k at the own point
        auto yphase = [&](int k, const float *yc) {
            const float *u = sU + (k & 1) * SU + oti * WU + otj, *w = sU + ((k & 1) ^ 1) * SU + oti * WU + otj;
            const int c = (oti + 1) * W2 + (otj + 1);
            const bool ek = k <= n3 - 2;
            const float u0 = u[0], ui = ei ? u[WU] : 0.f, uj = ej ? u[1] : 0.f;
            const float s0 = w[0] - u0;
            float av[P], y[P];
            av[0] = ek && ei ? (w[WU] - ui) - s0 : 0.f;
            av[1] = ek && ej ? (w[1] - uj) - s0 : 0.f;
            if constexpr (P == 4) {
                av[2] = ei ? ap->omega * (ui - u0) : 0.f;
                av[3] = ej ? ap->omega * (uj - u0) : 0.f;
            }
#pragma unroll
            for (int q = 0; q < P; ++q) y[q] = __builtin_fmaf(ap->gy, av[q], yc[q * S2 + c]);
            dual_prox<P>(ap->variant, y);
            bput(Band<BUF, float2>(ap->ya[par ^ 1], k, np, true), po, make_float2(y[0], y[1]));
            if constexpr (P == 4)
                bput(Band<BUF, float2>(ap->yb[par ^ 1], k, np, true), po, make_float2(y[2], y[3]));
        };
        // y3+ = y3 + g_y D_v t' (the last row keeps its value) and the t values of
        // the next search
        auto tphase = [&](int k) {
            const float4 o = keep[tid];
            const float tp = sT[TJ + tid];
            const float yc = ei ? __builtin_fmaf(ap->gy, sT[2 * TJ + tid] - tp, o.z) : o.z;
            bput(Band<BUF, float>(ap->y3[par ^ 1], k, np, true), po, yc);
            const float ym = oi >= 1 ? __builtin_fmaf(ap->gy, tp - sT[tid], o.w) : 0.f;
            gather_ahead(ga, sl, scp->in, 1, own_in, o.x, ym - (ei ? yc : 0.f), ap->gt, o.y, slice(1), &ncand[1], ap->capt);
        };

        // ---------------- march ----------------
        float *yA = sY, *yB = sY + P * S2, *yC = sY + 2 * P * S2;  // bands k, k + 1, k + 2 (and k - 1)
        Y ry;
        {
            Y p, q;
            loadY(kb - 1, kb >= 1, p);
            loadY(kb, true, q);
            loadY(kb + 1, kb + 1 <= ke && kb + 1 < n3, ry);
            loadRU(kb, true, true);
            storeY(yC, p);
            storeY(yA, q);
            storeY(yB, ry);
        }
        __syncthreads();
        fresh();
        uphase(kb, true, yA, yC);
        fresh();
        loadY(kb + 2, kb + 2 <= ke && kb + 2 < n3, ry);
        loadRU(kb + 1, kb + 1 < n3, kb + 1 < ke);
        __syncthreads();
        fresh();
        tphase(kb);
        __syncthreads();
        int k = kb;
        do {
            const bool more = k + 1 < ke;
            storeY(yC, ry);  // band k + 2
            fresh();
            loadY(k + 3, k + 3 <= ke && k + 3 < n3, ry);
            fresh();
            uphase(k + 1, more, yB, yA);
            fresh();
            loadRU(k + 2, k + 2 <= ke && k + 2 < n3, k + 2 < ke);
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
    }

    tile_sums<NT>(du2, u2, r2, ga, sl, red, a.part + 3 * slot, a.winpart + 4 * slot, a.winpart + 4 * (a.slots + slot));
    if (tid == 0) {
        a.ccount[slot] = ncand[0];
        a.ccount[a.slots + slot] = ncand[1];
    }
}

// The same iteration for cubes whose bands fill little of any tile (single spectra,
// single rows or columns of pixels): one thread per voxel, which evaluates the u'
// and t' of the neighbours it needs again (6 and 3 points, some 90 loads from the
// caches). What bounds it is those loads, 35 us (SSTV) and 51 us (HSSTV) per million
// voxels, and below a few hundred thousand the search and the launches. A slot is a
// run of `per` consecutive voxels. Every value comes from the operations of
// k_var_sweep in their order.
constexpr int FT = 256;
template <int P>
__global__ __launch_bounds__(FT) void k_var_flat(VarArgs a)
{
    __shared__ double red[10 * (FT / 64)];
    __shared__ uint32_t ncand[2];
    const int tid = threadIdx.x, slot = blockIdx.x;
    DevScalars *sc = a.sc;
    const bool idle_now = idle(sc);
    if (slot == 0 && tid == 0) {
        sc->view = {sc->in.a_lo, sc->in.a_hi, sc->in.a_c, idle_now ? 1u : 0u};
        passes_over(a.flags);
    }
    if (idle_now) return;
    if (tid < 2) ncand[tid] = 0u;
    __syncthreads();
    const const4<DevScalars> &scr = *(const4<DevScalars> *)sc;
    const int par = (int)(scr.iter & 1u);
    const uint32_t n1 = (uint32_t)a.d.n1, n2 = (uint32_t)a.d.n2, n3 = (uint32_t)a.d.n3, np = n1 * n2;
    const float a4 = scr.in.a4;
    const float *u = a.u[par], *t = a.t[par], *y3 = a.y3[par], *qv = a.q[par];
    const float2 *ya = a.ya[par], *yb = a.yb[par];
    double du2 = 0.0, u2 = 0.0, r2 = 0.0;
    Gathered ga;
    SlopeRegs sl;
    const uint32_t N = (uint32_t)a.d.plane, q1 = min(N, (uint32_t)(slot + 1) * (uint32_t)a.per);
    for (uint32_t q0 = (uint32_t)slot * (uint32_t)a.per; q0 < q1; q0 += FT) {
        const bool in = q0 + tid < q1;  // (the others repeat the last voxel)
        const uint32_t q = in ? q0 + tid : q1 - 1u;
        const uint32_t row = q / n2, j = q - row * n2, k = row / n1, i = row - k * n1;
        auto dT = [&](const float2 *y, uint32_t c, uint32_t ci, uint32_t cj) {
            float x = ci >= 1u ? y[c - n2].x : 0.f;
            x -= ci + 2u <= n1 ? y[c].x : 0.f;
            x += cj >= 1u ? y[c - 1u].y : 0.f;
            x -= cj + 2u <= n2 ? y[c].y : 0.f;
            return x;
        };
        // u+ at one point, c its index
        auto u_at = [&](uint32_t c, uint32_t ck, uint32_t ci, uint32_t cj, float uo) {
            float g = 0.f;
            if (ck >= 1u) g += dT(ya, c - np, ci, cj);
            if (ck + 2u <= n3) g -= dT(ya, c, ci, cj);
            if constexpr (P == 4) g = __builtin_fmaf(a.omega, dT(yb, c, ci, cj), g);
            const float x = __builtin_fmaf(-a.gu, g + y4_of(qv[c], a4), uo);
            return fminf(fmaxf(x, a.mu_lo), a.mu_hi);
        };
        auto up_at = [&](uint32_t c, uint32_t ck, uint32_t ci, uint32_t cj) {
            const float uo = u[c];
            return 2.f * u_at(c, ck, ci, cj, uo) - uo;
        };
        // t+ at one point of this band
        auto t_at = [&](uint32_t c, uint32_t ci, float to) {
            const float z = zt_of(to, ci >= 1u ? y3[c - n2] : 0.f, ci + 2u <= n1 ? y3[c] : 0.f, y4_of(qv[c], a4), a.gt);
            return soft(z, scr.in.tau[1]);
        };
        auto tp_at = [&](uint32_t c, uint32_t ci) {
            const float to = t[c];
            return 2.f * t_at(c, ci, to) - to;
        };
        const bool ei = i + 2u <= n1, ej = j + 2u <= n2, ek = k + 2u <= n3;
        const float uo = u[q], qo = qv[q], so = a.s[q], to = t[q], vo = a.v[q];
        const float un = u_at(q, k, i, j, uo), up = 2.f * un - uo;
        const float sn = soft(zs_of(so, y4_of(qo, a4)), scr.in.tau[0]), tn = t_at(q, i, to);
        const float sp = 2.f * sn - so, tp = 2.f * tn - to;
        const float qn = (a4 / a.gy) * qo + ((up + sp) + tp) - vo;
        // y1+
        const float ui = ei ? up_at(q + n2, k, i + 1u, j) : 0.f, uj = ej ? up_at(q + 1u, k, i, j + 1u) : 0.f;
        float av[P], y[P];
        av[0] = av[1] = 0.f;
        if (ek) {
            const float s0 = up_at(q + np, k + 1u, i, j) - up;
            if (ei) av[0] = (up_at(q + np + n2, k + 1u, i + 1u, j) - ui) - s0;
            if (ej) av[1] = (up_at(q + np + 1u, k + 1u, i, j + 1u) - uj) - s0;
        }
        const float2 yo = ya[q];
        y[0] = __builtin_fmaf(a.gy, av[0], yo.x);
        y[1] = __builtin_fmaf(a.gy, av[1], yo.y);
        if constexpr (P == 4) {
            const float2 bo = yb[q];
            av[2] = ei ? a.omega * (ui - up) : 0.f;
            av[3] = ej ? a.omega * (uj - up) : 0.f;
            y[2] = __builtin_fmaf(a.gy, av[2], bo.x);
            y[3] = __builtin_fmaf(a.gy, av[3], bo.y);
        }
        dual_prox<P>(a.variant, y);
        // y3+ here and in the row above, for the t values of the next search
        const float yc = ei ? __builtin_fmaf(a.gy, tp_at(q + n2, i + 1u) - tp, y3[q]) : y3[q];
        const float ym = i >= 1u ? __builtin_fmaf(a.gy, tp - tp_at(q - n2, i - 1u), y3[q - n2]) : 0.f;
        if (in) {
            a.u[par ^ 1][q] = un;
            a.s[q] = sn;
            a.t[par ^ 1][q] = tn;
            a.q[par ^ 1][q] = qn;
            a.y3[par ^ 1][q] = yc;
            a.ya[par ^ 1][q] = make_float2(y[0], y[1]);
            if constexpr (P == 4) a.yb[par ^ 1][q] = make_float2(y[2], y[3]);
            const double dl = (double)un - (double)uo, ud = (double)uo;
            du2 += dl * dl;
            u2 += ud * ud;
            r2 += (double)qn * (double)qn;
        }
        float4 *cand = a.cand + (int64_t)slot * a.capt;
        gather_ahead(ga, sl, scr.in, 0, in, sn, 0.f, 1.f, qn, cand, &ncand[0], a.capt);
        gather_ahead(ga, sl, scr.in, 1, in, tn, ym - (ei ? yc : 0.f), a.gt, qn, cand + (int64_t)a.slots * a.capt, &ncand[1],
                     a.capt);
    }
    tile_sums<FT>(du2, u2, r2, ga, sl, red, a.part + 3 * slot, a.winpart + 4 * slot, a.winpart + 4 * (a.slots + slot));
    if (tid == 0) {  // (every append came before the barrier in the sums)
        a.ccount[slot] = ncand[0];
        a.ccount[a.slots + slot] = ncand[1];
    }
}

__global__ __launch_bounds__(VT) void k_var_init(VarArgs a, int P, double eps, double tol, double alpha,
                                                 double beta, double gy4)
{
    const int64_t N = a.d.plane;
    for (int64_t q = (int64_t)blockIdx.x * VT + threadIdx.x; q < N; q += (int64_t)gridDim.x * VT) {
        a.u[0][q] = a.v[q];
        a.t[0][q] = 0.f;
        a.s[q] = 0.f;
        a.y3[0][q] = 0.f;
        a.q[0][q] = 0.f;
        a.ya[0][q] = make_float2(0.f, 0.f);
        if (P == 4) a.yb[0][q] = make_float2(0.f, 0.f);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) init_scalars(a.sc, eps, tol, alpha, beta, gy4);
}

// Copy a state variable out (out != null) or in, planes as in the C ABI.
__global__ __launch_bounds__(VT) void k_var_io(VarArgs a, int P, int var, float *out, const float *in)
{
    const int64_t N = a.d.plane;
    const int par = (int)(a.sc->iter & 1u);
    const float a4 = (float)a.sc->a4;
    const int64_t step = (int64_t)gridDim.x * VT;
    if (var == GEO_VAR_Y1) {
        for (int64_t g = (int64_t)blockIdx.x * VT + threadIdx.x; g < P / 2 * N; g += step) {
            const int h = g >= N;  // which pair
            const int64_t q = g - (h ? N : 0);
            float2 *y = (h ? a.yb : a.ya)[par];
            if (out) {
                out[2 * h * N + q] = y[q].x;
                out[(2 * h + 1) * N + q] = y[q].y;
            } else {
                y[q] = make_float2(in[2 * h * N + q], in[(2 * h + 1) * N + q]);
            }
        }
        return;
    }
    float *base;
    switch (var) {
    case GEO_VAR_U: base = a.u[par]; break;
    case GEO_VAR_S: base = a.s; break;
    case GEO_VAR_T: base = a.t[par]; break;
    case GEO_VAR_Y3: base = a.y3[par]; break;
    default: base = a.q[par]; break;
    }
    for (int64_t g = (int64_t)blockIdx.x * VT + threadIdx.x; g < N; g += step) {
        if (out)
            out[g] = var == GEO_VAR_Y4 ? a4 * base[g] : base[g];
        else
            base[g] = in[g];  // a loaded y4 is kept as it is, with the factor 1
    }
}

int grid_of(int64_t n)
{
    const int64_t b = (n + VT - 1) / VT;
    return (int)(b < 1 ? 1 : (b > kVarBlocks ? kVarBlocks : b));
}

size_t align256v(size_t x) { return (x + 255) & ~(size_t)255; }

// Sweep blocks that the device holds at once (queried once per form).
template <int P>
int resident_blocks()
{
    static const int cached = [] {
        int dev = 0, cus = 256, per = 1;
        if (hipGetDevice(&dev) == hipSuccess) {
            hipDeviceProp_t prop;
            if (hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
        }
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_var_sweep<P, true, false>, NT, 0) != hipSuccess || per < 1)
            per = 1;
        return cus * per;
    }();
    return cached;
}

// The split of a cube. A tile's points: 8 x 64, or rows x cols fitted to the cube
// where that needs 3/5 of the tiles or less (narrow cubes; the loads of 8 x 64 tiles
// come in full lines and their geometry is known to the compiler, so that between
// 0.65 and 0.75 of the tiles the two take the same time: 300 x 90 x 90 67.9 us an
// iteration of SSTV fitted, 64.9 not, 120 x 70 x 198 52.9 and 55.8, 1024 x 16 x 300 81
// and 189). Where the tiles fill less than 3/10 of their threads, no tiles (rows = 0:
// one thread per voxel, a slot a run of voxels), which takes 35 us per million
// voxels once they fill the device: 1 x 1 x 100000 15 us, 355 in 8 x 64 tiles, 4096 x 2
// x 300 93 us, 106 in fitted ones, 20 x 20 x 1000 36 and 28.
// The band chunk: the depth in 1..32 whose tiles the resident blocks
// finish first, a tile costing its bands and kTileFixedBands more (its first
// loads, the halo bands, the partial sums); ties to the deeper chunk. A search
// slot is one tile, or (bands of more than kMaxTiles tiles) several.
struct VarTiles {
    int rows, cols, ti, tj, tk, kc, slots, per;
};
VarTiles var_tiles(const Dims &d, int blocks)
{
    VarTiles v = {};
    v.rows = kTI;
    v.cols = kTJ;
    auto per_band = [&](int rows, int cols) { return (int64_t)ceil_div(d.n1, rows) * ceil_div(d.n2, cols); };
    const int64_t np = (int64_t)d.n1 * d.n2;
    if (np < kVarPixels) {
        int64_t best = per_band(kTI, kTJ) * 3 / 5;
        for (int s = ceil_div(d.n2, kTJ), e = s + 4; s < e; ++s) {
            const int cols = ceil_div(d.n2, s);
            int rows = NT / cols < kSpan - cols ? NT / cols : kSpan - cols;
            rows = ceil_div(d.n1, ceil_div(d.n1, rows));
            if (per_band(rows, cols) <= best) {
                best = per_band(rows, cols) - 1;
                v.rows = rows;
                v.cols = cols;
            }
        }
    }
    if (10 * np < 3 * NT * per_band(v.rows, v.cols)) {
        v.rows = v.cols = 0;
        v.per = ceil_div(ceil_div(d.plane, kMaxTiles), FT) * FT;
        v.slots = ceil_div(d.plane, v.per);
        return v;
    }
    v.ti = ceil_div(d.n1, v.rows);
    v.tj = ceil_div(d.n2, v.cols);
    const int64_t pb = (int64_t)v.ti * v.tj;
    v.kc = d.n3 < 32 ? d.n3 : 32;
    double best = 0.0;
    for (int kc = v.kc; kc >= 1; --kc) {
        const int64_t T = pb * ceil_div(d.n3, kc);
        if (T > kMaxTiles && best > 0.0) break;
        const double cost = (double)ceil_div(T, blocks) * (kc + kTileFixedBands);
        if (best == 0.0 || cost < best - 1e-9) {
            best = cost;
            v.kc = kc;
        }
    }
    // (very deep cubes: the chunk grows until the tiles fit the search)
    while (v.kc < d.n3 && pb * ceil_div(d.n3, v.kc) > kMaxTiles) v.kc = 2 * v.kc < d.n3 ? 2 * v.kc : d.n3;
    v.tk = ceil_div(d.n3, v.kc);
    const int64_t T = pb * v.tk;
    v.per = ceil_div(T, kMaxTiles);
    v.slots = ceil_div(T, v.per);
    return v;
}

// Workspace: the scalars, the search's regions (sized for kMaxTiles slots: the
// tiling follows the device), the launch table, then the arrays.
struct VarLayout {
    size_t sc, part, winpart, hist, rec, cand, ccount, table, u[2], t[2], s, ya[2], yb[2], y3[2], q[2], total;
    int64_t cap;  // candidates per field
};

VarLayout var_layout(int64_t N, int P)
{
    VarLayout L;
    memset(&L, 0, sizeof L);
    L.cap = N / 16 > 65536 ? N / 16 : 65536;
    size_t o = 0;
    auto take = [&](size_t b) { const size_t at = o; o = align256v(o + b); return at; };
    const size_t f = sizeof(float) * (size_t)N;
    L.sc = take(sizeof(DevScalars));
    L.part = take(sizeof(double) * 3 * kMaxTiles);
    L.winpart = take(sizeof(double) * 2 * 4 * kMaxTiles);
    L.hist = take(6 * sizeof(Hist));  // 3 radix levels x 2 fields
    L.rec = take(6 * sizeof(FbRec));
    L.cand = take(sizeof(float4) * 2 * (size_t)L.cap);
    L.ccount = take(sizeof(uint32_t) * 2 * kMaxTiles);
    L.table = take(table_bytes(1));
    for (int p = 0; p < 2; ++p) {
        L.u[p] = take(f);
        L.t[p] = take(f);
        L.y3[p] = take(f);
        L.q[p] = take(f);
        L.ya[p] = take(2 * f);
        if (P == 4) L.yb[p] = take(2 * f);
    }
    L.s = take(f);
    L.total = o;
    return L;
}

VarArgs var_args(const Dims &d, const geo_params *p, const float *v, void *ws, VarLayout *Lout = nullptr)
{
    VarArgs a;
    memset(&a, 0, sizeof a);
    a.d = d;
    a.variant = p->regularizer;
    const int P = var_planes(p->regularizer);
    const VarLayout L = var_layout(d.plane, P);
    if (Lout) *Lout = L;
    char *b = (char *)ws;
    const double na2 = p->regularizer == GEO_REG_SSTV ? 32.0 : 32.0 + 8.0 * p->omega * p->omega;
    a.gu = (float)(1.0 / (na2 + 1.0));
    a.gt = (float)(1.0 / 5.0);
    a.gy = (float)(1.0 / 3.0);
    a.omega = (float)p->omega;
    a.mu_lo = (float)p->mu_lo;
    a.mu_hi = (float)p->mu_hi;
    a.v = v;
    a.sc = (DevScalars *)(b + L.sc);
    a.part = (double *)(b + L.part);
    a.winpart = (double *)(b + L.winpart);
    a.cand = (float4 *)(b + L.cand);
    a.ccount = (uint32_t *)(b + L.ccount);
    a.flags = slot_flags(b + L.table, 1);
    for (int q = 0; q < 2; ++q) {
        a.u[q] = (float *)(b + L.u[q]);
        a.t[q] = (float *)(b + L.t[q]);
        a.y3[q] = (float *)(b + L.y3[q]);
        a.q[q] = (float *)(b + L.q[q]);
        a.ya[q] = (float2 *)(b + L.ya[q]);
        a.yb[q] = P == 4 ? (float2 *)(b + L.yb[q]) : nullptr;
    }
    a.s = (float *)(b + L.s);
    // (one tiling for all of them, so that HSSTV1 with omega = 0 sums as SSTV does)
    const VarTiles t = var_tiles(d, resident_blocks<4>());
    a.rows = t.rows;
    a.cols = t.cols;
    a.ti = t.ti;
    a.tj = t.tj;
    a.tk = t.tk;
    a.kc = t.kc;
    a.slots = t.slots;
    a.per = t.per;
    a.capt = (int)(L.cap / a.slots);
    return a;
}

// Host image of the launch table entry: the fields the histogram passes, the
// search and the start of a call read.
void var_table_entry(CubeEntry *e, const VarArgs &a, const VarLayout &L, void *ws, const geo_params *p, int n_iter)
{
    memset(e, 0, sizeof *e);
    CubeArgs<float> *x = reinterpret_cast<CubeArgs<float> *>(e->bytes);
    char *b = (char *)ws;
    for (int q = 0; q < 2; ++q) {
        x->side[q].s = a.s;
        x->side[q].t = a.t[q];
        x->side[q].y3 = a.y3[q];
        x->side[q].y4 = a.q[q];
    }
    CubeCommon &c = x->c;
    c.zt_step = a.gt;
    c.d = a.d;
    c.v = a.v;
    c.sc = a.sc;
    c.part = a.part;
    c.winpart = a.winpart;
    c.hist = (Hist *)(b + L.hist);
    c.rec = (FbRec *)(b + L.rec);
    c.cand = a.cand;
    c.ccount = a.ccount;
    c.capt = a.capt;
    c.ntiles = a.slots;
    c.tol = p->tol;
    c.alpha = p->alpha;
    c.beta = p->beta;
    c.eps = p->eps;
    c.set_eps = 1u;
    c.limit = (uint32_t)n_iter;
    c.ahead = 1u;
}

template <int P>
void launch_var_sweep(const VarArgs &a, hipStream_t st)
{
    if (a.rows == 0)
        hipLaunchKernelGGL(k_var_flat<P>, dim3(a.slots), dim3(FT), 0, st, a);
    else if ((uint64_t)a.d.n1 * (uint64_t)a.d.n2 >= kVarPixels)
        hipLaunchKernelGGL((k_var_sweep<P, false, false>), dim3(a.slots), dim3(NT), 0, st, a);
    else if (a.rows == kTI && a.cols == kTJ)
        hipLaunchKernelGGL((k_var_sweep<P, true, false>), dim3(a.slots), dim3(NT), 0, st, a);
    else
        hipLaunchKernelGGL((k_var_sweep<P, true, true>), dim3(a.slots), dim3(NT), 0, st, a);
}

}  // namespace

int var_planes(int regularizer) { return regularizer == GEO_REG_SSTV ? 2 : 4; }

size_t var_workspace_bytes(int n1, int n2, int n3, int regularizer)
{
    return var_layout((int64_t)n1 * n2 * n3, var_planes(regularizer)).total;
}

hipError_t var_state_init(const Dims &d, const geo_params *p, const float *v, void *ws, hipStream_t st)
{
    const VarArgs a = var_args(d, p, v, ws);
    // y4 = gy4 c4 q after an iteration, gy4 the FP32 step the kernels use
    hipLaunchKernelGGL(k_var_init, dim3(grid_of(d.plane)), dim3(VT), 0, st, a, var_planes(p->regularizer), p->eps,
                       p->tol, p->alpha, p->beta, (double)a.gy);
    return hipGetLastError();
}

hipError_t var_step(const Dims &d, const geo_params *p, const float *v, void *ws, int n_iter,
                    hipStream_t st, HostBox &box, int *slots, double *sweep_ms)
{
    DevScalars *const out = box.as<DevScalars>();
    VarLayout L;
    const VarArgs a = var_args(d, p, v, ws, &L);
    void *table = (char *)ws + L.table;
    const int stride = (int)sizeof(CubeEntry);
    LaunchShape sh;
    memset(&sh, 0, sizeof sh);
    sh.ncubes = 1;
    sh.fb_grid = fallback_grid();
    // the table image, with its launch-wide flags zeroed
    std::vector<unsigned char> img(table_image_bytes(1), 0);
    var_table_entry(reinterpret_cast<CubeEntry *>(img.data()), a, L, ws, p, n_iter);
    hipError_t e = hipMemcpyAsync(table, img.data(), img.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = launch_begin(table, stride, 1, st);
    // sweep_ms: events around the sweep of the kTimedEvery-th, 2 kTimedEvery-th,
    // ... slot of the call (every slot in calls of fewer), the mean scaled to
    // the iterations done
    const bool all = n_iter < kTimedEvery;
    std::vector<hipEvent_t> ev;
    if (sweep_ms && e == hipSuccess) {
        ev.resize(2 * (size_t)(all ? n_iter : n_iter / kTimedEvery));
        for (size_t k = 0; k < ev.size() && e == hipSuccess; ++k) e = hipEventCreate(&ev[k]);
    }
    // with a tolerance the host reads the stop flag every check_every slots
    const int every = p->tol > 0.0 ? (p->check_every > 0 ? p->check_every : 32) : (n_iter > 0 ? n_iter : 1);
    size_t ne = 0;
    int issued = 0;
    bool synced = false;
    while (issued < n_iter && e == hipSuccess) {
        const int batch = n_iter - issued < every ? n_iter - issued : every;
        for (int it = issued; it < issued + batch && e == hipSuccess; ++it) {
            e = launch_fallback(table, 4, sh, st);
            if (e != hipSuccess) break;
            const bool timed = sweep_ms && (all || it % kTimedEvery == kTimedEvery - 1) &&
                               ne + 2 <= ev.size();
            if (timed) e = hipEventRecord(ev[ne], st);
            if (a.variant == GEO_REG_SSTV)
                launch_var_sweep<2>(a, st);
            else
                launch_var_sweep<4>(a, st);
            if (timed && e == hipSuccess) e = hipEventRecord(ev[ne + 1], st);
            ne += timed ? 2 : 0;
            if (e == hipSuccess) e = launch_search(table, stride, 1, st);
        }
        issued += batch;
        if (e == hipSuccess) {
            box.use();
            e = launch_report(table, stride, 1, out, st);
        }
        if (e == hipSuccess) e = box.wait();
        synced = e == hipSuccess;
        if (synced && (out->stop || (int)out->calls_iter >= n_iter)) break;
    }
    if (!synced && e == hipSuccess) {  // n_iter = 0
        box.use();
        e = launch_report(table, stride, 1, out, st);
        if (e == hipSuccess) e = box.wait();
    }
    *slots = issued;
    if (e == hipSuccess && sweep_ms) {
        double sum = 0.0;
        for (size_t k = 0; k + 1 < ne && e == hipSuccess; k += 2) {
            float ms = 0.f;
            e = hipEventElapsedTime(&ms, ev[k], ev[k + 1]);
            sum += ms;
        }
        const size_t ns = ne / 2;
        *sweep_ms = ns ? sum / (double)ns * (double)out->calls_iter : 0.0;
    }
    for (hipEvent_t x : ev) (void)hipEventDestroy(x);
    return e;
}

hipError_t var_state_io(const Dims &d, const geo_params *p, void *ws, int var, float *out,
                        const float *in, hipStream_t st)
{
    VarLayout L;
    const VarArgs a = var_args(d, p, nullptr, ws, &L);
    const int P = var_planes(p->regularizer);
    hipLaunchKernelGGL(k_var_io, dim3(grid_of(var == GEO_VAR_Y1 ? P / 2 * d.plane : d.plane)), dim3(VT), 0, st, a, P,
                       var, out, in);
    hipError_t e = hipGetLastError();
    // a loaded state does not continue the previous run
    if (e == hipSuccess && in) e = launch_loaded(a.sc, (Hist *)((char *)ws + L.hist), var, st);
    return e;
}

}  // namespace geo
