// The second sweep of the two-sweep form of the iteration (BF16 duals, see
// sweep.hip), pointwise: steps 2, 3, 7, 8, 13, the rest of step 14 and the
// FP64 partial sums of the l2-ball distance of step 15, at the thresholds that
// the search between the sweeps found; then the finalize (one block per cube):
// the l2-ball factor of step 15 (applied lazily when y4 is next read), the stopping test and the
// iteration counter.
#include "radix.hpp"

namespace geo {

namespace {

constexpr int NPT = 256;  // threads of the pointwise kernels

template <typename DT>
using Table = const CubeArgs<DT> *__restrict__;

constexpr int RB = kSweepBRows;  // rows per sweep B strip
// CPT consecutive values of one row: one 4- or 8-byte access for a pair.
__device__ __forceinline__ void ldv(const float *p, float (&o)[1]) { o[0] = *p; }
__device__ __forceinline__ void ldv(const bf16 *p, float (&o)[1]) { o[0] = ld(p); }
__device__ __forceinline__ void ldv(const float *p, float (&o)[2])
{
    const float2 x = *reinterpret_cast<const float2 *>(p);
    o[0] = x.x;
    o[1] = x.y;
}
__device__ __forceinline__ void ldv(const bf16 *p, float (&o)[2])
{
    const float2 x = ld2(reinterpret_cast<const bf16x2 *>(p));
    o[0] = x.x;
    o[1] = x.y;
}
__device__ __forceinline__ void ldv_nt(const float *p, float (&o)[1]) { o[0] = ld_nt(p); }
__device__ __forceinline__ void ldv_nt(const bf16 *p, float (&o)[1]) { o[0] = ld_nt(p); }
__device__ __forceinline__ void ldv_nt(const float *p, float (&o)[2])
{
    const f32x2 x = __builtin_nontemporal_load(reinterpret_cast<const f32x2 *>(p));
    o[0] = x.x;
    o[1] = x.y;
}
__device__ __forceinline__ void ldv_nt(const bf16 *p, float (&o)[2])
{
    const uint32_t b = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p));
    o[0] = __uint_as_float(b << 16);
    o[1] = __uint_as_float(b & 0xffff0000u);
}
// four columns: one 16-byte FP32 or 8-byte BF16 access
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void ldv(const float *p, float (&o)[4])
{
    const float4 x = *reinterpret_cast<const float4 *>(p);
    o[0] = x.x;
    o[1] = x.y;
    o[2] = x.z;
    o[3] = x.w;
}
__device__ __forceinline__ void ldv(const bf16 *p, float (&o)[4])
{
    const uint2 b = *reinterpret_cast<const uint2 *>(p);
    o[0] = __uint_as_float(b.x << 16);
    o[1] = __uint_as_float(b.x & 0xffff0000u);
    o[2] = __uint_as_float(b.y << 16);
    o[3] = __uint_as_float(b.y & 0xffff0000u);
}
__device__ __forceinline__ void ldv_nt(const float *p, float (&o)[4])
{
    const f32x4 x = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    o[0] = x.x;
    o[1] = x.y;
    o[2] = x.z;
    o[3] = x.w;
}
__device__ __forceinline__ void ldv_nt(const bf16 *p, float (&o)[4])
{
    float a[2], b[2];
    ldv_nt(p, a);
    ldv_nt(p + 2, b);
    o[0] = a[0];
    o[1] = a[1];
    o[2] = b[0];
    o[3] = b[1];
}
template <typename T>
__device__ __forceinline__ void stv_nt(T *p, const float (&x)[1]) { st_nt(p, x[0]); }
__device__ __forceinline__ void stv_nt(float *p, const float (&x)[4])
{
    f32x4 v;
    v.x = x[0];
    v.y = x[1];
    v.z = x[2];
    v.w = x[3];
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(p));
}
__device__ __forceinline__ void stv_nt(bf16 *p, const float (&x)[4])
{
    st2_nt(reinterpret_cast<bf16x2 *>(p), make_float2(x[0], x[1]));
    st2_nt(reinterpret_cast<bf16x2 *>(p + 2), make_float2(x[2], x[3]));
}
__device__ __forceinline__ void stv_nt(float *p, const float (&x)[2])
{
    st_nt(reinterpret_cast<float2 *>(p), make_float2(x[0], x[1]));
}
__device__ __forceinline__ void stv_nt(bf16 *p, const float (&x)[2])
{
    st2_nt(reinterpret_cast<bf16x2 *>(p), make_float2(x[0], x[1]));
}

// Steps 2, 3 (soft thresholds at the selected levels), 7, 8, 13 and 14; the
// z inputs are evaluated again exactly as sweep A did. A thread takes a strip
// of RB rows and CPT adjacent columns of one band and issues all of its loads
// at once; only the rows just above and below the strip (D_v coupling of t'
// and y3) are read twice. CPT = 2 (one access per pair) when the row length
// is even, else 1.
template <typename DT, int CPT>
__device__ __forceinline__ double sweep_b_strips(const CubeArgs<DT> &a, const DevScalars *sc, int lb,
                                                 double ts, double tt)
{
    const Dims d = a.c.d;
    const int n1 = d.n1, n2 = d.n2, n3 = d.n3;
    const int par = (int)(sc->iter & 1u);
    const Side<DT> src = a.side[par], dst = a.side[par ^ 1];
    const float a4 = (float)sc->a4;
    double r2 = 0.0;
    const uint32_t nstrip = (uint32_t)((n1 + RB - 1) / RB);
    const uint32_t ncol = (uint32_t)(n2 / CPT);
    const uint32_t items = (uint32_t)n3 * nstrip * ncol;
    const uint32_t stride = (uint32_t)a.c.nb * NPT;
    for (uint32_t w = (uint32_t)lb * NPT + threadIdx.x; w < items; w += stride) {
        const uint32_t j = CPT * (w % ncol), rr = w / ncol;
        const int ia = (int)(rr % nstrip) * RB, k = (int)(rr / nstrip);
        const uint32_t q0 = ((uint32_t)k * (uint32_t)n1 + (uint32_t)ia) * (uint32_t)n2 + j;
        // rows ia .. ia+RB-1 of the strip, and row ia+RB for the D_v coupling
        float y3r[RB + 1][CPT], y4[RB + 1][CPT], to[RB + 1][CPT], so[RB][CPT], yp[RB][CPT];
        float y3m0[CPT];
        if (ia >= 1) ldv(src.y3 + q0 - n2, y3m0);
        else
#pragma unroll
            for (int c = 0; c < CPT; ++c) y3m0[c] = 0.f;
#pragma unroll
        for (int r = 0; r <= RB; ++r) {
            const bool in = ia + r < n1;
            const uint32_t q = q0 + (uint32_t)(r * n2);
            float q4[CPT];
            if (in) {
                ldv(src.y3 + q, y3r[r]);
                ldv(src.y4 + q, q4);
                ldv(src.t + q, to[r]);
                if (r < RB) {
                    ldv_nt(src.s + q, so[r]);
                    ldv_nt(a.y4p + q, yp[r]);
                }
            } else {
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    y3r[r][c] = q4[c] = to[r][c] = 0.f;
                    if (r < RB) so[r][c] = yp[r][c] = 0.f;
                }
            }
#pragma unroll
            for (int c = 0; c < CPT; ++c) y4[r][c] = in ? y4_of(q4[c], a4) : 0.f;
        }
        float tp[RB + 1][CPT];
#pragma unroll
        for (int r = 0; r <= RB; ++r) {
            const int i = ia + r;
            float tn[CPT];
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const float y3m = r == 0 ? y3m0[c] : y3r[r - 1][c];
                tn[c] = soft(zt_of(to[r][c], y3m, i <= n1 - 2 ? y3r[r][c] : 0.f, y4[r][c], kStepT), tt);
                tp[r][c] = 2.f * tn[c] - to[r][c];
            }
            if (r < RB && i < n1) stv_nt(dst.t + q0 + (uint32_t)(r * n2), tn);
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = ia + r;
            if (i < n1) {
                const uint32_t q = q0 + (uint32_t)(r * n2);
                float sn[CPT], y3n[CPT], qn[CPT];
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    sn[c] = soft(zs_of(so[r][c], y4[r][c]), ts);
                    const float sp = 2.f * sn[c] - so[r][c];
                    const float tp1 = i <= n1 - 2 ? tp[r + 1][c] : 0.f;
                    y3n[c] = y3r[r][c] + kStepY * mask_le(i, n1) * (tp1 - tp[r][c]);
                    // q+ = 5 y4' - v (step 14); r = ||q+|| (step 15)
                    qn[c] = as_stored(dst.y4, yp[r][c] + (sp + tp[r][c]));
                    r2 += (double)qn[c] * (double)qn[c];
                }
                stv_nt(dst.s + q, sn);
                stv_nt(dst.y3 + q, y3n);
                stv_nt(dst.y4 + q, qn);
            }
        }
    }
    return r2;
}

// WIDE: the cubes whose sweep B takes four columns per thread (a kernel of
// their own: that form needs 104 registers, the others 73, and a kernel runs
// at the occupancy of its largest form); otherwise the others.
template <typename DT, bool WIDE>
__global__ __launch_bounds__(NPT) void k_sweep_b(Table<DT> cubes, LaunchShape sh)
{
    __shared__ double red[NPT / 64];
    __shared__ int cube_of_block;
    // blocks [b0, b0 + nb) belong to one cube: the last cube whose b0 is at
    // most this block's index, found by one wavefront (one load per lane;
    // a scan by one thread took a memory round trip per cube of a batch)
    static_assert(kMaxBatch <= 64, "one wavefront covers the cubes");
    if (threadIdx.x < 64) {
        const int c = threadIdx.x;
        const bool le = c < sh.ncubes && cubes[c].c.b0 <= (int)blockIdx.x;
        const unsigned long long m = __ballot(le);
        if (c == 0) cube_of_block = 63 - __clzll((long long)m);  // cube 0 starts at block 0
    }
    __syncthreads();
    const CubeArgs<DT> &a = cubes[__builtin_amdgcn_readfirstlane(cube_of_block)];
    const DevScalars *sc = a.c.sc;
    const int cpt = sweep_b_cpt(a.c.d.n2);
    if (idle(sc) || (cpt == 4) != WIDE) return;
    // a missed window's threshold comes from this slot's histogram passes
    const double ts = sc->sel[0].done ? sc->sel[0].tau : fb_final(a.c.rec, 0).tau;
    const double tt = sc->sel[1].done ? sc->sel[1].tau : fb_final(a.c.rec, 1).tau;
    const int lb = (int)blockIdx.x - a.c.b0;  // block within the cube
    double r2;
    if constexpr (WIDE)
        r2 = sweep_b_strips<DT, 4>(a, sc, lb, ts, tt);
    else
        r2 = cpt == 2 ? sweep_b_strips<DT, 2>(a, sc, lb, ts, tt) : sweep_b_strips<DT, 1>(a, sc, lb, ts, tt);
    const double tot = block_sum<NPT>(r2, red);
    if (threadIdx.x == 0) a.c.part[2 * a.c.ntiles + lb] = tot;
}

// Fixed-order sums of the block partials of both sweeps: relative change of u
// (stopping rule), r = ||y4'/gamma4 - v|| for the lazy scale of y4 (step 15),
// iteration counter. A separate one-block launch: a last-block-done pattern
// inside sweep B needs a device-scope release per block, which writes back
// the XCD's L2 each time.
// One block per cube of the table (entries of `stride` bytes).
__global__ __launch_bounds__(NPT) void k_finalize(const char *table, int stride)
{
    // the launch table through the constant address space (scalar loads)
    const4<CubeCommon> &cc = *(const4<CubeCommon> *)(table + (size_t)blockIdx.x * stride);
    DevScalars *sc = cc.sc;
    const double *part = cc.part;
    const int grid_a = cc.ntiles, blocks_b = cc.nb;
    __shared__ double red[3 * (NPT / 64)];
    // the partials are read together with the flag that may make them moot
    const bool skip = idle(sc);
    // each thread adds its partials b = tid, tid + NPT, ... in that order,
    // kFinUnroll of them loaded at a time
    constexpr int kFinUnroll = 8;
    double du2 = 0.0, u2 = 0.0, r2 = 0.0;
    for (int b0 = threadIdx.x; b0 < grid_a; b0 += kFinUnroll * NPT) {
        double x0[kFinUnroll], x1[kFinUnroll];
#pragma unroll
        for (int k = 0; k < kFinUnroll; ++k) {
            const int b = b0 + k * NPT;
            x0[k] = b < grid_a ? part[2 * b] : 0.0;
            x1[k] = b < grid_a ? part[2 * b + 1] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kFinUnroll; ++k)
            if (b0 + k * NPT < grid_a) {
                du2 += x0[k];
                u2 += x1[k];
            }
    }
    for (int b0 = threadIdx.x; b0 < blocks_b; b0 += kFinUnroll * NPT) {
        double x2[kFinUnroll];
#pragma unroll
        for (int k = 0; k < kFinUnroll; ++k) {
            const int b = b0 + k * NPT;
            x2[k] = b < blocks_b ? part[2 * grid_a + b] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kFinUnroll; ++k)
            if (b0 + k * NPT < blocks_b) r2 += x2[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) passes_over(slot_flags(table, (int)gridDim.x));
    if (skip) return;
    // a threshold found by this slot's histogram passes becomes the field's
    // search state, with the window of the next iteration sized by the
    // density of |z| around it (only this block writes the cube's state)
    if (threadIdx.x == 0) {
        bool missed = false;
        for (int f = 0; f < 2; ++f)
            if (!sc->sel[f].done) {
                missed = true;
                const FbRec &r = fb_final(cc.rec, f);
                SelState o = sc->sel[f];
                o.tau = r.tau;
                o.done = 1u;
                o.full = 0u;
                o.dens = cc.rec[f].dens;
                set_window(o, true, window_budget(cc.d.plane));
                sc->sel[f] = o;
            }
        // whether the next iteration's sweep A stores z (iter counts this one)
        const uint32_t calm = missed ? 0u : sc->calm + 1u;
        sc->calm = calm;
        sc->zstore = (sc->iter + 1u < kZStoreIters || calm < kZStoreCalm) ? 1u : 0u;
    }
    // the three block sums at once, in the order of block_sum: a butterfly
    // within each wavefront, then the wavefronts in order (thread 0)
    du2 = wave_sum(du2);
    u2 = wave_sum(u2);
    r2 = wave_sum(r2);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) {
        red[wid] = du2;
        red[NPT / 64 + wid] = u2;
        red[2 * (NPT / 64) + wid] = r2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        du2 = u2 = r2 = 0.0;
        for (int w = 0; w < NPT / 64; ++w) {
            du2 += red[w];
            u2 += red[NPT / 64 + w];
            r2 += red[2 * (NPT / 64) + w];
        }
        const double r = sqrt(r2);
        const double rel = u2 > 0.0 ? sqrt(du2) / sqrt(u2) : __longlong_as_double(0x7ff0000000000000ll);
        const bool bad = !isfinite(du2) || !isfinite(u2) || !isfinite(r2);
        sc->r = r;
        sc->rel = rel;
        sc->c4 = r > sc->eps ? 1.0 - sc->eps / r : 0.0;
        sc->a4 = sc->gy4 * sc->c4;
        sc->iter = sc->iter + 1u;
        sc->calls_iter = sc->calls_iter + 1u;
        if (bad) sc->nonfinite = 1u;
        // eq. (28), from the second iteration after the initial point on: the
        // first one (zero duals) changes u only by the box projection
        if (bad || (sc->tol > 0.0 && sc->iter >= 2u && rel < sc->tol)) sc->stop = 1u;
    }
}

}  // namespace

hipError_t launch_sweep_b(const void *table, const LaunchShape &sh, hipStream_t st)
{
    const CubeArgs<bf16> *cubes = (const CubeArgs<bf16> *)table;
    if (sh.b_kinds & 1)
        hipLaunchKernelGGL((k_sweep_b<bf16, false>), dim3(sh.total_b), dim3(NPT), 0, st, cubes, sh);
    if (sh.b_kinds & 2)
        hipLaunchKernelGGL((k_sweep_b<bf16, true>), dim3(sh.total_b), dim3(NPT), 0, st, cubes, sh);
    return hipGetLastError();
}

hipError_t launch_finalize(const void *table, int stride, int ncubes, hipStream_t st)
{
    hipLaunchKernelGGL(k_finalize, dim3(ncubes), dim3(NPT), 0, st, (const char *)table, stride);
    return hipGetLastError();
}

}  // namespace geo
