// Standalone operators and proximal tools behind geo_apply_op and the
// geo_project_* / geo_prox_l12 entry points. Neighbours come through the
// caches. The solver itself does not use these kernels: its fused sweeps
// (sweep.hip) stage the same stencils in LDS.
#include "solver.hpp"

namespace geo {

namespace {

constexpr int NT = kPointThreads;
struct Cube {
    Dims d;
    __device__ __forceinline__ bool in(int k, int i, int j) const
    {
        return k >= 0 && k < d.n3 && i >= 0 && i < d.n1 && j >= 0 && j < d.n2;
    }
    __device__ __forceinline__ float at(const float *x, int k, int i, int j) const
    {
        return in(k, i, j) ? x[vox(d, k, i, j)] : 0.0f;
    }
};

// ---- differences (Sec. II-A, Neumann boundary) ----
__device__ __forceinline__ float dv(const Cube &c, const float *x, int k, int i, int j)
{
    return i <= c.d.n1 - 2 ? c.at(x, k, i + 1, j) - c.at(x, k, i, j) : 0.0f;
}
__device__ __forceinline__ float dh(const Cube &c, const float *x, int k, int i, int j)
{
    return j <= c.d.n2 - 2 ? c.at(x, k, i, j + 1) - c.at(x, k, i, j) : 0.0f;
}
__device__ __forceinline__ float ds(const Cube &c, const float *x, int k, int i, int j)
{
    return k <= c.d.n3 - 2 ? c.at(x, k + 1, i, j) - c.at(x, k, i, j) : 0.0f;
}
__device__ __forceinline__ float dv_t(const Cube &c, const float *p, int k, int i, int j)
{
    return (i >= 1 ? c.at(p, k, i - 1, j) : 0.0f) - (i <= c.d.n1 - 2 ? c.at(p, k, i, j) : 0.0f);
}
__device__ __forceinline__ float dh_t(const Cube &c, const float *p, int k, int i, int j)
{
    return (j >= 1 ? c.at(p, k, i, j - 1) : 0.0f) - (j <= c.d.n2 - 2 ? c.at(p, k, i, j) : 0.0f);
}
__device__ __forceinline__ float ds_t(const Cube &c, const float *p, int k, int i, int j)
{
    return (k >= 1 ? c.at(p, k - 1, i, j) : 0.0f) - (k <= c.d.n3 - 2 ? c.at(p, k, i, j) : 0.0f);
}
// D D_s (vertical / horizontal) and its adjoint D_s^T D^T
__device__ __forceinline__ float dds_v(const Cube &c, const float *x, int k, int i, int j)
{
    if (k > c.d.n3 - 2 || i > c.d.n1 - 2) return 0.0f;
    return (c.at(x, k + 1, i + 1, j) - c.at(x, k + 1, i, j)) - (c.at(x, k, i + 1, j) - c.at(x, k, i, j));
}
__device__ __forceinline__ float dds_h(const Cube &c, const float *x, int k, int i, int j)
{
    if (k > c.d.n3 - 2 || j > c.d.n2 - 2) return 0.0f;
    return (c.at(x, k + 1, i, j + 1) - c.at(x, k + 1, i, j)) - (c.at(x, k, i, j + 1) - c.at(x, k, i, j));
}
__device__ __forceinline__ float d_t(const Cube &c, const float *pv, const float *ph, int k, int i, int j)
{
    return dv_t(c, pv, k, i, j) + dh_t(c, ph, k, i, j);
}
__device__ __forceinline__ float dds_t(const Cube &c, const float *pv, const float *ph, int k, int i, int j)
{
    float lo = (k >= 1) ? d_t(c, pv, ph, k - 1, i, j) : 0.0f;
    float hi = (k <= c.d.n3 - 2) ? d_t(c, pv, ph, k, i, j) : 0.0f;
    return lo - hi;
}

// ---- Condat's interpolation operators (Sec. II-D) ----
// dual edge fields: vertical on rows 0..N1-2, horizontal on columns 0..N2-2
__device__ __forceinline__ float yvm(const Cube &c, const float *yv, int k, int i, int j)
{
    return (i <= c.d.n1 - 2) ? c.at(yv, k, i, j) : 0.0f;
}
__device__ __forceinline__ float yhm(const Cube &c, const float *yh, int k, int i, int j)
{
    return (j <= c.d.n2 - 2) ? c.at(yh, k, i, j) : 0.0f;
}
// component cmp (0..5 = ud_v, ud_h, lr_v, lr_h, c_v, c_h) of L y
__device__ float l_comp(const Cube &c, const float *yv, const float *yh, int cmp, int k, int i, int j)
{
    const float mv = mask_le(i, c.d.n1), mh = mask_le(j, c.d.n2);
    switch (cmp) {
    case 0: return mv * yvm(c, yv, k, i, j);
    case 1: return mv * 0.25f * (yhm(c, yh, k, i, j) + yhm(c, yh, k, i, j - 1) + yhm(c, yh, k, i + 1, j) + yhm(c, yh, k, i + 1, j - 1));
    case 2: return mh * 0.25f * (yvm(c, yv, k, i, j) + yvm(c, yv, k, i - 1, j) + yvm(c, yv, k, i, j + 1) + yvm(c, yv, k, i - 1, j + 1));
    case 3: return mh * yhm(c, yh, k, i, j);
    case 4: return 0.5f * (yvm(c, yv, k, i, j) + yvm(c, yv, k, i - 1, j));
    default: return 0.5f * (yhm(c, yh, k, i, j) + yhm(c, yh, k, i, j - 1));
    }
}
// w on the ud grid (rows 0..N1-2) and lr grid (cols 0..N2-2)
__device__ __forceinline__ float wud(const Cube &c, const float *w, int k, int i, int j)
{
    return (i <= c.d.n1 - 2) ? c.at(w, k, i, j) : 0.0f;
}
__device__ __forceinline__ float wlr(const Cube &c, const float *w, int k, int i, int j)
{
    return (j <= c.d.n2 - 2) ? c.at(w, k, i, j) : 0.0f;
}
// part (0: vertical, 1: horizontal) of L_g^T w_g for the grids selected by mask
// (bit 0 ud, bit 1 lr, bit 2 c); w points at the 6 planes
__device__ float lt_comp(const Cube &c, const float *w, int64_t N, int gmask, int part, int k, int i, int j)
{
    float acc = 0.0f;
    if (part == 0) {
        if (gmask & 1) acc += wud(c, w + 0 * N, k, i, j);
        if (gmask & 2)
            acc += 0.25f * (wlr(c, w + 2 * N, k, i, j) + wlr(c, w + 2 * N, k, i + 1, j) + wlr(c, w + 2 * N, k, i, j - 1) + wlr(c, w + 2 * N, k, i + 1, j - 1));
        if (gmask & 4) acc += 0.5f * (c.at(w + 4 * N, k, i, j) + c.at(w + 4 * N, k, i + 1, j));
        return mask_le(i, c.d.n1) * acc;
    }
    if (gmask & 2) acc += wlr(c, w + 3 * N, k, i, j);
    if (gmask & 1)
        acc += 0.25f * (wud(c, w + 1 * N, k, i, j) + wud(c, w + 1 * N, k, i, j + 1) + wud(c, w + 1 * N, k, i - 1, j) + wud(c, w + 1 * N, k, i - 1, j + 1));
    if (gmask & 4) acc += 0.5f * (c.at(w + 5 * N, k, i, j) + c.at(w + 5 * N, k, i, j + 1));
    return mask_le(j, c.d.n2) * acc;
}

__global__ __launch_bounds__(NT) void k_apply(int op, int adj, Dims d, const float *in, float *out,
                                              int out_planes, int64_t g0)
{
    const Cube c{d};
    const int64_t N = d.plane;
    const int64_t g = g0 + (int64_t)blockIdx.x * NT + threadIdx.x;
    if (g >= N * out_planes) return;
    const int pl = (int)(g / N);
    const int64_t q = g - (int64_t)pl * N;
    const int j = (int)(q % d.n2);
    const int64_t r = q / d.n2;
    const int i = (int)(r % d.n1), k = (int)(r / d.n1);
    float o = 0.0f;
    if (!adj) {
        switch (op) {
        case GEO_OP_DV: o = dv(c, in, k, i, j); break;
        case GEO_OP_DH: o = dh(c, in, k, i, j); break;
        case GEO_OP_DS: o = ds(c, in, k, i, j); break;
        case GEO_OP_D: o = pl == 0 ? dv(c, in, k, i, j) : dh(c, in, k, i, j); break;
        case GEO_OP_DDS: o = pl == 0 ? dds_v(c, in, k, i, j) : dds_h(c, in, k, i, j); break;
        case GEO_OP_L_UD: o = l_comp(c, in, in + N, 0 + pl, k, i, j); break;
        case GEO_OP_L_LR: o = l_comp(c, in, in + N, 2 + pl, k, i, j); break;
        case GEO_OP_L_C: o = l_comp(c, in, in + N, 4 + pl, k, i, j); break;
        case GEO_OP_L: o = l_comp(c, in, in + N, pl, k, i, j); break;
        case GEO_OP_K: {
            // in: u, s, t, w1 (6), w2 (6); out: y1 (2), y2 (2), y3, y4
            const float *u = in, *s = in + N, *t = in + 2 * N, *w1 = in + 3 * N, *w2 = in + 9 * N;
            if (pl < 2) o = (pl == 0 ? dv(c, u, k, i, j) : dh(c, u, k, i, j)) - lt_comp(c, w1, N, 7, pl, k, i, j);
            else if (pl < 4) o = (pl == 2 ? dds_v(c, u, k, i, j) : dds_h(c, u, k, i, j)) - lt_comp(c, w2, N, 7, pl - 2, k, i, j);
            else if (pl == 4) o = dv(c, t, k, i, j);
            else o = u[q] + s[q] + t[q];
        } break;
        }
    } else {
        switch (op) {
        case GEO_OP_DV: o = dv_t(c, in, k, i, j); break;
        case GEO_OP_DH: o = dh_t(c, in, k, i, j); break;
        case GEO_OP_DS: o = ds_t(c, in, k, i, j); break;
        case GEO_OP_D: o = d_t(c, in, in + N, k, i, j); break;
        case GEO_OP_DDS: o = dds_t(c, in, in + N, k, i, j); break;
        case GEO_OP_L_UD: {
            // in: the 2 planes of the ud grid, placed as planes 0, 1 of a 6-plane view
            o = pl == 0 ? mask_le(i, d.n1) * wud(c, in, k, i, j)
                        : mask_le(j, d.n2) * 0.25f * (wud(c, in + N, k, i, j) + wud(c, in + N, k, i, j + 1) + wud(c, in + N, k, i - 1, j) + wud(c, in + N, k, i - 1, j + 1));
        } break;
        case GEO_OP_L_LR: {
            o = pl == 0 ? mask_le(i, d.n1) * 0.25f * (wlr(c, in, k, i, j) + wlr(c, in, k, i + 1, j) + wlr(c, in, k, i, j - 1) + wlr(c, in, k, i + 1, j - 1))
                        : mask_le(j, d.n2) * wlr(c, in + N, k, i, j);
        } break;
        case GEO_OP_L_C: {
            o = pl == 0 ? mask_le(i, d.n1) * 0.5f * (c.at(in, k, i, j) + c.at(in, k, i + 1, j))
                        : mask_le(j, d.n2) * 0.5f * (c.at(in + N, k, i, j) + c.at(in + N, k, i, j + 1));
        } break;
        case GEO_OP_L: o = lt_comp(c, in, N, 7, pl, k, i, j); break;
        case GEO_OP_K: {
            // in: y1 (2), y2 (2), y3, y4; out: u, s, t, w1 (6), w2 (6)
            const float *y1 = in, *y2 = in + 2 * N, *y3 = in + 4 * N, *y4 = in + 5 * N;
            if (pl == 0) o = d_t(c, y1, y1 + N, k, i, j) + dds_t(c, y2, y2 + N, k, i, j) + y4[q];
            else if (pl == 1) o = y4[q];
            else if (pl == 2) o = dv_t(c, y3, k, i, j) + y4[q];
            else if (pl < 9) o = -l_comp(c, y1, y1 + N, pl - 3, k, i, j);
            else o = -l_comp(c, y2, y2 + N, pl - 9, k, i, j);
        } break;
        }
    }
    out[g] = o;
}

// One thread per voxel and all of its output planes, for bands that the buffer
// path takes (common.hpp: band_of; below kOpsPixels pixels) and that fill enough
// of their blocks (fills_lanes below). What bounds an
// operator is HBM (K: 21 planes, 84 bytes per voxel): every plane is read from
// HBM once, the neighbours come from the caches, and a thread's loads (37 for K)
// are in flight together. k_apply above, one thread per output element, decodes
// its index with 64-bit divisions and reads a plane once per output plane that
// needs it: K and its adjoint at 256 x 256 x 128 took 324 and 543 us.
constexpr uint32_t kOpsPixels = 1u << 26;
static_assert(kOpsPixels <= kNoPix - kOpsPixels, "a missing pixel and its neighbours lie past a band");

struct OpView {
    const float *in;
    float *out;
    int64_t N;
    uint32_t np, n2, rows;  // pixels of a band, of a row, of the rows that hold a vertical edge
    int n3, k;
    uint32_t c0, cm, cp;    // this pixel, its left and right neighbours (kNoPix: none)
    uint32_t h0;            // this pixel where it holds a horizontal edge
    float mv, mh;           // 1 where the edge to the row below, the next column exists
    bool next;              // there is a next band

    __device__ __forceinline__ BandRsrc band(const float *p, int kk, uint32_t count) const
    {
        return band_of(p, (int64_t)kk * np, kk >= 0 && kk < n3 ? count : 0u);
    }
    // plane pl of the input, whole or its vertical edges only, band k + dk
    __device__ __forceinline__ BandRsrc full(int pl, int dk = 0) const { return band(in + (int64_t)pl * N, k + dk, np); }
    __device__ __forceinline__ BandRsrc vert(int pl, int dk = 0) const { return band(in + (int64_t)pl * N, k + dk, rows); }
    __device__ __forceinline__ float at(BandRsrc r, uint32_t pix) const { return bld((const float *)nullptr, r, pix); }
    __device__ __forceinline__ void put(int pl, float x) const
    {
        bst_nt((const float *)nullptr, band(out + (int64_t)pl * N, k, np), c0, x);
    }
    // x where there is a next band, else 0
    __device__ __forceinline__ float in_band(float x) const { return next ? x : 0.f; }
    // differences of one plane
    __device__ __forceinline__ float dv(int pl, int dk = 0) const
    {
        const BandRsrc r = full(pl, dk);
        const float x = at(r, c0 + n2) - at(r, c0);
        return mv != 0.f ? x : 0.f;  // (a select: an infinite value stays in its own edges)
    }
    __device__ __forceinline__ float dh(int pl, int dk = 0) const
    {
        const BandRsrc r = full(pl, dk);
        const float x = at(r, cp) - at(r, c0);
        return mh != 0.f ? x : 0.f;
    }
    __device__ __forceinline__ float dvt(int pl, int dk = 0) const
    {
        const BandRsrc r = vert(pl, dk);
        return at(r, c0 - n2) - at(r, c0);
    }
    __device__ __forceinline__ float dht(int pl, int dk = 0) const
    {
        const BandRsrc r = full(pl, dk);
        return at(r, cm) - at(r, h0);
    }
    // D^T of the edge field in planes pl, pl + 1; D_s^T D^T of it
    __device__ __forceinline__ float dt(int pl, int dk = 0) const { return dvt(pl, dk) + dht(pl + 1, dk); }
    __device__ __forceinline__ float ddst(int pl) const { return dt(pl, -1) - in_band(dt(pl)); }
    // the six components of L y, y in planes pl, pl + 1
    __device__ __forceinline__ void interp(int pl, float (&o)[6]) const
    {
        const BandRsrc v = vert(pl), h = full(pl + 1);
        const float v00 = at(v, c0), vu = at(v, c0 - n2), vr = at(v, cp), vur = at(v, cp - n2);
        const float h00 = at(h, h0), hl = at(h, cm), hd = at(h, h0 + n2), hld = at(h, cm + n2);
        o[0] = v00;
        o[1] = mv * 0.25f * (h00 + hl + hd + hld);
        o[2] = mh * 0.25f * (v00 + vu + vr + vur);
        o[3] = h00;
        o[4] = 0.5f * (v00 + vu);
        o[5] = 0.5f * (h00 + hl);
    }
    // vertical and horizontal part of L^T w over the grids in G (bit 0 ud, 1 lr,
    // 2 c); ud, lr, c: first plane of each grid's pair
    template <int G>
    __device__ __forceinline__ void interp_t(int ud, int lr, int c, float &pv, float &ph) const
    {
        float a = 0.f, b = 0.f;
        if constexpr (G & 1) a += at(vert(ud), c0);
        if constexpr (G & 2) {
            const BandRsrc r = full(lr);
            a += 0.25f * (at(r, h0) + at(r, h0 + n2) + at(r, cm) + at(r, cm + n2));
            b += at(full(lr + 1), h0);
        }
        if constexpr (G & 1) {
            const BandRsrc r = vert(ud + 1);
            b += 0.25f * (at(r, c0) + at(r, cp) + at(r, c0 - n2) + at(r, cp - n2));
        }
        if constexpr (G & 4) {
            const BandRsrc r = full(c), q = full(c + 1);
            a += 0.5f * (at(r, c0) + at(r, c0 + n2));
            b += 0.5f * (at(q, c0) + at(q, cp));
        }
        pv = mv * a;
        ph = mh * b;
    }
};

// Blocks in an order that gives each of the 8 XCDs a contiguous run of them, so
// that the rows which neighbouring blocks share meet in one L2.
__device__ __forceinline__ uint32_t xcd_order(uint32_t b, uint32_t n)
{
    const uint32_t per = n >> 3;
    return b < 8u * per ? (b & 7u) * per + (b >> 3) : b;
}

template <int OP, bool ADJ>
__global__ __launch_bounds__(NT) void k_op(Dims d, const float *in, float *out, uint32_t bx, uint32_t blocks)
{
    for (uint32_t b0 = blockIdx.x; b0 < blocks; b0 += gridDim.x) {
        const uint32_t b = xcd_order(b0, blocks), np = (uint32_t)d.n1 * (uint32_t)d.n2, n2 = (uint32_t)d.n2;
        OpView v;
        v.k = (int)(b / bx);
        const uint32_t p = (b % bx) * NT + threadIdx.x, i = p / n2, j = p - i * n2;
        const bool ok = p < np;
        v.in = in;
        v.out = out;
        v.N = d.plane;
        v.np = np;
        v.n2 = n2;
        v.rows = np - n2;
        v.n3 = d.n3;
        v.c0 = ok ? p : kNoPix;
        v.cm = ok && j >= 1 ? p - 1 : kNoPix;
        v.cp = ok && j + 1 < n2 ? p + 1 : kNoPix;
        v.h0 = ok && j + 1 < n2 ? p : kNoPix;
        v.mv = mask_le((int)i, d.n1);
        v.mh = mask_le((int)j, d.n2);
        v.next = v.k <= d.n3 - 2;
        if constexpr (!ADJ) {
            if constexpr (OP == GEO_OP_DV) v.put(0, v.dv(0));
            if constexpr (OP == GEO_OP_DH) v.put(0, v.dh(0));
            if constexpr (OP == GEO_OP_DS) v.put(0, v.in_band(v.at(v.full(0, 1), v.c0) - v.at(v.full(0), v.c0)));
            if constexpr (OP == GEO_OP_D) {
                v.put(0, v.dv(0));
                v.put(1, v.dh(0));
            }
            if constexpr (OP == GEO_OP_DDS) {
                v.put(0, v.in_band(v.dv(0, 1) - v.dv(0)));
                v.put(1, v.in_band(v.dh(0, 1) - v.dh(0)));
            }
            if constexpr (OP == GEO_OP_L_UD || OP == GEO_OP_L_LR || OP == GEO_OP_L_C || OP == GEO_OP_L) {
                float o[6];
                v.interp(0, o);
                if constexpr (OP == GEO_OP_L) {
#pragma unroll
                    for (int q = 0; q < 6; ++q) v.put(q, o[q]);
                } else {
                    constexpr int q = 2 * (OP - GEO_OP_L_UD);
                    v.put(0, o[q]);
                    v.put(1, o[q + 1]);
                }
            }
            if constexpr (OP == GEO_OP_K) {
                // in: u, s, t, w1 (6), w2 (6); out: y1 (2), y2 (2), y3, y4
                float av, ah, bv, bh;
                v.interp_t<7>(3, 5, 7, av, ah);
                v.interp_t<7>(9, 11, 13, bv, bh);
                const float gv = v.dv(0), gh = v.dh(0);
                v.put(0, gv - av);
                v.put(1, gh - ah);
                v.put(2, v.in_band(v.dv(0, 1) - gv) - bv);
                v.put(3, v.in_band(v.dh(0, 1) - gh) - bh);
                v.put(4, v.dv(2));
                v.put(5, v.at(v.full(0), v.c0) + v.at(v.full(1), v.c0) + v.at(v.full(2), v.c0));
            }
        } else {
            if constexpr (OP == GEO_OP_DV) v.put(0, v.dvt(0));
            if constexpr (OP == GEO_OP_DH) v.put(0, v.dht(0));
            if constexpr (OP == GEO_OP_DS) v.put(0, v.at(v.full(0, -1), v.c0) - v.in_band(v.at(v.full(0), v.c0)));
            if constexpr (OP == GEO_OP_D) v.put(0, v.dt(0));
            if constexpr (OP == GEO_OP_DDS) v.put(0, v.ddst(0));
            if constexpr (OP == GEO_OP_L_UD || OP == GEO_OP_L_LR || OP == GEO_OP_L_C || OP == GEO_OP_L) {
                float pv, ph;
                if constexpr (OP == GEO_OP_L) v.interp_t<7>(0, 2, 4, pv, ph);
                if constexpr (OP == GEO_OP_L_UD) v.interp_t<1>(0, 0, 0, pv, ph);
                if constexpr (OP == GEO_OP_L_LR) v.interp_t<2>(0, 0, 0, pv, ph);
                if constexpr (OP == GEO_OP_L_C) v.interp_t<4>(0, 0, 0, pv, ph);
                v.put(0, pv);
                v.put(1, ph);
            }
            if constexpr (OP == GEO_OP_K) {
                // in: y1 (2), y2 (2), y3, y4; out: u, s, t, w1 (6), w2 (6)
                const float y4 = v.at(v.full(5), v.c0);
                v.put(0, v.dt(0) + v.ddst(2) + y4);
                v.put(1, y4);
                v.put(2, v.dvt(4) + y4);
                float o[6];
                v.interp(0, o);
#pragma unroll
                for (int q = 0; q < 6; ++q) v.put(3 + q, -o[q]);
                v.interp(2, o);
#pragma unroll
                for (int q = 0; q < 6; ++q) v.put(9 + q, -o[q]);
            }
        }
    }
}

// Whether one thread per voxel is the faster form for bands of np pixels. A band
// takes whole blocks of it, so bands of few pixels leave lanes idle, and k_apply
// has none: it took K on 100000 bands of one pixel from 141 us to 10. The line is
// the share of lanes filled where the two meet, over bands of 16 to 400 pixels of
// 4M and 30M voxels; the more planes an operator writes, the more often k_apply
// decodes an index and reads its inputs again. Time of a thread per voxel over
// that of k_apply:
//   one plane out: share 0.56 D_s 1.08 to 1.20, D^T 0.93 to 0.98; 0.77 0.87, 0.72
//   two: 0.32 D 1.09 to 1.28, L_ud 0.97 to 1.08; 0.39 D 0.90 to 1.04, L_ud 0.79 to 0.89
//   six: 0.14 K 1.30 to 1.80, L 0.83 to 0.96; 0.25 K 0.77 to 1.08, L 0.48 to 0.57
//   fifteen: 0.06 K^T 1.5 to 1.9; 0.14 0.80 to 1.05
bool fills_lanes(int64_t np, int pout)
{
    const int64_t lanes = (np + NT - 1) / NT * NT;
    return 16 * np >= lanes * (pout == 1 ? 10 : pout == 2 ? 6 : pout == 6 ? 4 : 2);
}

template <int OP>
void launch_op(int adjoint, const Dims &d, const float *in, float *out, hipStream_t st)
{
    const int64_t np = (int64_t)d.n1 * d.n2;
    const uint32_t bx = (uint32_t)((np + NT - 1) / NT);
    const uint32_t blocks = bx * (uint32_t)d.n3;  // at most N / NT + n3 < 2^32
    const dim3 grid(blocks < kGridMost ? blocks : kGridMost);
    if (adjoint)
        hipLaunchKernelGGL((k_op<OP, true>), grid, dim3(NT), 0, st, d, in, out, bx, blocks);
    else
        hipLaunchKernelGGL((k_op<OP, false>), grid, dim3(NT), 0, st, d, in, out, bx, blocks);
}

// The pointwise operators below stream their arrays: kPointUnroll groups of four
// consecutive values per thread, nontemporal stores (lines of results would
// otherwise push inputs out of the L2). 256 x 256 x 128, one value per thread and
// step before: l2 sum 14.2 -> 12.4 us, l2 apply 18.2 and a launch of 3.8 for the
// norm -> 18.7, l12 22.4 -> 20.0 (6.7 TB/s), box 12.4 -> 10.8 (6.2 TB/s).
constexpr int kPointUnroll = 2;
__device__ __forceinline__ int64_t point_at() { return ((int64_t)blockIdx.x * kPointUnroll * NT + threadIdx.x) * 4; }

// ---- l2 ball, eq. (23): FP64 partial sums of the squared norm, then the scaling,
// each block of which adds the partials in the same order ----
__global__ __launch_bounds__(NT) void k_l2_partial(const float *x, const float *cc, int64_t n, double *part)
{
    __shared__ double red[NT / 64];
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * NT * 4;
    for (int64_t q = ((int64_t)blockIdx.x * NT + threadIdx.x) * 4; q < n; q += kPointUnroll * stride) {
        Quad a[kPointUnroll], c[kPointUnroll];
#pragma unroll
        for (int u = 0; u < kPointUnroll; ++u) {
            a[u] = ld_quad(x, q + u * stride, n);
            c[u] = ld_quad(cc, q + u * stride, n);
        }
#pragma unroll
        for (int u = 0; u < kPointUnroll; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double d = (double)a[u].x[e] - (double)c[u].x[e];
                acc += d * d;
            }
    }
    acc = block_sum<NT>(acc, red);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

__global__ __launch_bounds__(NT) void k_l2_apply(const float *x, const float *cc, int64_t n, double eps,
                                                 const double *part, int nb, double *r_out, float *out)
{
    __shared__ double red[NT / 64], norm;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nb; b += NT) acc += part[b];
    acc = block_sum<NT>(acc, red);
    if (threadIdx.x == 0) {
        norm = sqrt(acc);
        if (blockIdx.x == 0) *r_out = norm;
    }
    __syncthreads();
    const double rr = norm;
    const bool inside = rr <= eps;
    const double f = inside ? 1.0 : eps / rr;
    const int64_t stride = (int64_t)gridDim.x * NT * 4;
    for (int64_t q = ((int64_t)blockIdx.x * NT + threadIdx.x) * 4; q < n; q += kPointUnroll * stride) {
        Quad a[kPointUnroll], c[kPointUnroll];
#pragma unroll
        for (int u = 0; u < kPointUnroll; ++u) {
            a[u] = ld_quad(x, q + u * stride, n);
            c[u] = ld_quad(cc, q + u * stride, n);
        }
#pragma unroll
        for (int u = 0; u < kPointUnroll; ++u) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                a[u].x[e] = inside ? a[u].x[e]
                                   : (float)((double)c[u].x[e] + f * ((double)a[u].x[e] - (double)c[u].x[e]));
            st_quad_nt(out, q + u * stride, n, a[u]);
        }
    }
}

__global__ __launch_bounds__(NT) void k_prox_l12(const float *xa, const float *xb, int64_t n, float g,
                                                 float *oa, float *ob)
{
    const int64_t q = point_at();
    Quad a[kPointUnroll], b[kPointUnroll];
#pragma unroll
    for (int u = 0; u < kPointUnroll; ++u) {
        a[u] = ld_quad(xa, q + 4 * u * NT, n);
        b[u] = ld_quad(xb, q + 4 * u * NT, n);
    }
#pragma unroll
    for (int u = 0; u < kPointUnroll; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e) shrink2(a[u].x[e], b[u].x[e], g);
        st_quad_nt(oa, q + 4 * u * NT, n, a[u]);
        st_quad_nt(ob, q + 4 * u * NT, n, b[u]);
    }
}

__global__ __launch_bounds__(NT) void k_box(const float *x, int64_t n, float lo, float hi, float *out)
{
    const int64_t q = point_at();
    Quad v[kPointUnroll];
#pragma unroll
    for (int u = 0; u < kPointUnroll; ++u) v[u] = ld_quad(x, q + 4 * u * NT, n);
#pragma unroll
    for (int u = 0; u < kPointUnroll; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = v[u].x[e];
            v[u].x[e] = a < lo ? lo : (a > hi ? hi : a);
        }
        st_quad_nt(out, q + 4 * u * NT, n, v[u]);
    }
}

// One launch takes kPointMost values (kGridMost blocks' worth); more go in several.
constexpr int64_t kPointMost = (int64_t)kGridMost * 4 * kPointUnroll * NT;
unsigned point_grid(int64_t n) { return (unsigned)((n + 4 * kPointUnroll * NT - 1) / (4 * kPointUnroll * NT)); }

int grid_for(int64_t n)
{
    int64_t b = (n + NT - 1) / NT;
    return (int)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

}  // namespace

int op_planes(int op, int adj, int *pin, int *pout)
{
    static const int tin[] = {1, 1, 1, 1, 1, 2, 2, 2, 2, 15};
    static const int tout[] = {1, 1, 1, 2, 2, 2, 2, 2, 6, 6};
    if (op < 0 || op > GEO_OP_K) return -1;
    *pin = adj ? tout[op] : tin[op];
    *pout = adj ? tin[op] : tout[op];
    return 0;
}

hipError_t launch_apply_op(int op, int adjoint, const Dims &d, const float *in, float *out, hipStream_t st)
{
    int pin, pout;
    if (op_planes(op, adjoint, &pin, &pout)) return hipErrorInvalidValue;
    const int64_t np = (int64_t)d.n1 * d.n2;
    if (np < kOpsPixels && fills_lanes(np, pout)) {
        switch (op) {
        case GEO_OP_DV: launch_op<GEO_OP_DV>(adjoint, d, in, out, st); break;
        case GEO_OP_DH: launch_op<GEO_OP_DH>(adjoint, d, in, out, st); break;
        case GEO_OP_DS: launch_op<GEO_OP_DS>(adjoint, d, in, out, st); break;
        case GEO_OP_D: launch_op<GEO_OP_D>(adjoint, d, in, out, st); break;
        case GEO_OP_DDS: launch_op<GEO_OP_DDS>(adjoint, d, in, out, st); break;
        case GEO_OP_L_UD: launch_op<GEO_OP_L_UD>(adjoint, d, in, out, st); break;
        case GEO_OP_L_LR: launch_op<GEO_OP_L_LR>(adjoint, d, in, out, st); break;
        case GEO_OP_L_C: launch_op<GEO_OP_L_C>(adjoint, d, in, out, st); break;
        case GEO_OP_L: launch_op<GEO_OP_L>(adjoint, d, in, out, st); break;
        default: launch_op<GEO_OP_K>(adjoint, d, in, out, st); break;
        }
        return hipGetLastError();
    }
    // (in launches of kGridMost blocks: a loop in the kernel made it 1.4 times slower)
    const int64_t total = d.plane * pout, most = (int64_t)kGridMost * NT;
    for (int64_t g0 = 0; g0 < total; g0 += most) {
        const int64_t n = total - g0 < most ? total - g0 : most;
        hipLaunchKernelGGL(k_apply, dim3((unsigned)((n + NT - 1) / NT)), dim3(NT), 0, st, op, adjoint, d, in, out, pout,
                           g0);
    }
    return hipGetLastError();
}

int l2_blocks(int64_t n) { return grid_for(n) > 1024 ? 1024 : grid_for(n); }

hipError_t launch_l2(const float *x, const float *c, int64_t n, double eps, float *out, double *partials,
                     double *r_out, hipStream_t st)
{
    const int nb = l2_blocks(n);
    hipLaunchKernelGGL(k_l2_partial, dim3(nb), dim3(NT), 0, st, x, c, n, partials);
    hipLaunchKernelGGL(k_l2_apply, dim3(nb), dim3(NT), 0, st, x, c, n, eps, partials, nb, r_out, out);
    return hipGetLastError();
}

hipError_t launch_prox_l12(const float *xa, const float *xb, int64_t n, float gamma, float *oa, float *ob,
                           hipStream_t st)
{
    for (int64_t q = 0; q < n; q += kPointMost) {
        const int64_t m = n - q < kPointMost ? n - q : kPointMost;
        hipLaunchKernelGGL(k_prox_l12, dim3(point_grid(m)), dim3(NT), 0, st, xa + q, xb + q, m, gamma, oa + q, ob + q);
    }
    return hipGetLastError();
}

hipError_t launch_box(const float *x, int64_t n, float lo, float hi, float *out, hipStream_t st)
{
    for (int64_t q = 0; q < n; q += kPointMost) {
        const int64_t m = n - q < kPointMost ? n - q : kPointMost;
        hipLaunchKernelGGL(k_box, dim3(point_grid(m)), dim3(NT), 0, st, x + q, m, lo, hi, out + q);
    }
    return hipGetLastError();
}

}  // namespace geo
