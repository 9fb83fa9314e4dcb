// Device-side helpers shared by the gfx950 kernels of the GeoSSTV solver.
//
// Cube layout is band-sequential: element (i, j, k) of an N1 x N2 x N3 cube at
// (k*N1 + i)*N2 + j, so a wavefront of 64 lanes along j reads 256 contiguous
// bytes of one band row.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace geo {

constexpr float kStepU = 1.0f / 13.0f;  // step sizes printed after eq. (24)
constexpr float kStepW = 0.25f;         // w1 and w2
constexpr float kStepT = 1.0f / 3.0f;
constexpr float kStepY = 0.2f;          // y1..y4 (and s has step 1)

// Storage of the dual variables: FP32, or BF16 with FP32 arithmetic.
struct bf16 {
    uint16_t bits;
};

__device__ __forceinline__ float ld(const float *p) { return *p; }
__device__ __forceinline__ float ld(const bf16 *p)
{
    return __uint_as_float(((uint32_t)p->bits) << 16);
}
__device__ __forceinline__ void st(float *p, float x) { *p = x; }
__device__ __forceinline__ void st(bf16 *p, float x)
{
    // round to nearest even; NaN stays NaN
    uint32_t u = __float_as_uint(x);
    uint32_t r = ((u & 0x7fffffffu) > 0x7f800000u) ? (u | 0x00400000u)
                                                   : u + 0x7fffu + ((u >> 16) & 1u);
    bf16 b;
    b.bits = (uint16_t)(r >> 16);
    *p = b;
}

// Pairs stored together: the (vertical, horizontal) components of a dual
// edge field, or the two components of one l_{1,2} group of w.
struct bf16x2 {
    uint32_t bits;  // low half: first component, high half: second
};
template <typename DT> struct PairOf;
template <> struct PairOf<float> { using type = float2; };
template <> struct PairOf<bf16> { using type = bf16x2; };

__device__ __forceinline__ float2 ld2(const float2 *p) { return *p; }
__device__ __forceinline__ float2 ld2(const bf16x2 *p)
{
    const uint32_t b = p->bits;
    return make_float2(__uint_as_float(b << 16), __uint_as_float(b & 0xffff0000u));
}
__device__ __forceinline__ void st2(float2 *p, float2 x) { *p = x; }
__device__ __forceinline__ void st2(bf16x2 *p, float2 x)
{
    bf16 a, b;
    st(&a, x.x);
    st(&b, x.y);
    bf16x2 o;
    o.bits = (uint32_t)a.bits | ((uint32_t)b.bits << 16);
    *p = o;
}

// Stores of results this launch does not read again: with the nontemporal
// hint their lines leave the L2 early and do not push out the halo lines
// that neighbouring tiles still read.
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void st_nt(float *p, float x)
{
    __builtin_nontemporal_store(x, p);
}
__device__ __forceinline__ void st_nt(float2 *p, float2 x)
{
    f32x2 v;
    v.x = x.x;
    v.y = x.y;
    __builtin_nontemporal_store(v, reinterpret_cast<f32x2 *>(p));
}
__device__ __forceinline__ void st_nt(bf16 *p, float x)
{
    bf16 b;
    st(&b, x);
    __builtin_nontemporal_store(b.bits, &p->bits);
}
typedef float f32x4n __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st_nt(float4 *p, float4 x)
{
    f32x4n v;
    v.x = x.x;
    v.y = x.y;
    v.z = x.z;
    v.w = x.w;
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4n *>(p));
}
__device__ __forceinline__ void st2_nt(float2 *p, float2 x) { st_nt(p, x); }
__device__ __forceinline__ void st2_nt(bf16x2 *p, float2 x)
{
    bf16 a, b;
    st(&a, x.x);
    st(&b, x.y);
    const uint32_t bits = (uint32_t)a.bits | ((uint32_t)b.bits << 16);
    __builtin_nontemporal_store(bits, &p->bits);
}

// Loads of values no other thread or tile reads (no halo reuse).
__device__ __forceinline__ float ld_nt(const float *p)
{
    return __builtin_nontemporal_load(p);
}
__device__ __forceinline__ float ld_nt(const bf16 *p)
{
    return __uint_as_float(((uint32_t)__builtin_nontemporal_load(&p->bits)) << 16);
}

// Four consecutive floats at any 4-byte alignment (global memory takes it), and
// a group of U of them per thread: element e of group u of thread t of a block of
// NT threads at base + 4 (u NT + t) + e, of n.
struct __attribute__((aligned(4))) Quad {
    float x[4];
};
__device__ __forceinline__ Quad ld_quad(const float *p, int64_t q, int64_t n)
{
    Quad o;
    if (q + 4 <= n) {
        __builtin_memcpy(&o, p + q, sizeof o);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) o.x[e] = q + e < n ? p[q + e] : 0.f;
    }
    return o;
}
__device__ __forceinline__ void st_quad_nt(float *p, int64_t q, int64_t n, const Quad &v)
{
    typedef float unaligned4 __attribute__((ext_vector_type(4), aligned(4)));
    if (q + 4 <= n) {
        unaligned4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = v.x[e];
        __builtin_nontemporal_store(w, reinterpret_cast<unaligned4 *>(p + q));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (q + e < n) p[q + e] = v.x[e];
    }
}

// Value as stored (FP32 or rounded to BF16).
__device__ __forceinline__ float as_stored(const float *, float x) { return x; }
__device__ __forceinline__ float as_stored(const bf16 *, float x)
{
    bf16 b;
    st(&b, x);
    return ld(&b);
}

// Soft threshold of the l1-ball projections.
__device__ __forceinline__ float soft(float z, double tau)
{
    const double m = fabs((double)z) - tau;
    return m > 0.0 ? copysignf((float)m, z) : 0.0f;
}

// One band of an array through the buffer path: a resource over the band
// (uniform base and size) and a 32-bit byte offset per lane. A lane whose
// offset lies past the band (kNoPix of any element size) loads zeros and
// stores nothing, so code full of edge conditions stays straight-line: no
// branches around the accesses, one 32-bit offset for every array of an
// element size, and the compiler knows exactly how many loads are in flight
// when one of them is needed.
using BandRsrc = __amdgpu_buffer_rsrc_t;
// The index of a missing pixel. Its byte offset, for elements of 2 to 16 bytes, lies
// past every band that goes this way: fewer than 2^22 pixels of up to 16 bytes in
// the solver's sweeps, 2^26 of 4 in the operators, 2^27 of up to 8 in the
// regularizers' sweep. So does, in the first two, that of a missing pixel's
// neighbours a row above or below, and everywhere that of a pixel above the first
// row (negative, so near 2^32). (In a regularizer's band of one row of more than
// 100M pixels a missing pixel's neighbour above may be a pixel: what it loads is
// not used.)
constexpr uint32_t kNoPix = 0x0c000000u;
static_assert(kNoPix <= 0xffffffffu / 16, "offsets of missing pixels do not wrap");
template <typename T>
__device__ __forceinline__ BandRsrc band_of(const T *p, int64_t first, uint32_t count)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)(p + first), 0, (int)(count * (uint32_t)sizeof(T)), 0x00020000);
}
constexpr int kNT = 2;  // the nontemporal hint of a buffer access
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <int AUX = 0>
__device__ __forceinline__ float bld(const float *, BandRsrc r, uint32_t pix)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, pix * 4u, 0, AUX));
}
template <int AUX = 0>
__device__ __forceinline__ float bld(const bf16 *, BandRsrc r, uint32_t pix)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, pix * 2u, 0, AUX) << 16);
}
__device__ __forceinline__ u32x2 bld_raw(const float2 *, BandRsrc r, uint32_t pix)
{
    return __builtin_amdgcn_raw_buffer_load_b64(r, pix * 8u, 0, 0);
}
__device__ __forceinline__ uint32_t bld_raw(const bf16x2 *, BandRsrc r, uint32_t pix)
{
    return __builtin_amdgcn_raw_buffer_load_b32(r, pix * 4u, 0, 0);
}
__device__ __forceinline__ u32x4 bld_raw(const float4 *, BandRsrc r, uint32_t pix)
{
    return __builtin_amdgcn_raw_buffer_load_b128(r, pix * 16u, 0, 0);
}
// the pair in a raw word or two
__device__ __forceinline__ float2 pair_of(u32x2 x) { return make_float2(__uint_as_float(x.x), __uint_as_float(x.y)); }
__device__ __forceinline__ float2 pair_of(uint32_t b)
{
    return make_float2(__uint_as_float(b << 16), __uint_as_float(b & 0xffff0000u));
}
__device__ __forceinline__ void bst(const float *, BandRsrc r, uint32_t pix, float x)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, pix * 4u, 0, 0);
}
__device__ __forceinline__ void bst_nt(const float *, BandRsrc r, uint32_t pix, float x)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, pix * 4u, 0, kNT);
}
__device__ __forceinline__ void bst_nt(const bf16 *, BandRsrc r, uint32_t pix, float x)
{
    bf16 b;
    st(&b, x);
    __builtin_amdgcn_raw_buffer_store_b16(b.bits, r, pix * 2u, 0, kNT);
}
__device__ __forceinline__ void bst_nt(const float2 *, BandRsrc r, uint32_t pix, float2 x)
{
    u32x2 v;
    v.x = __float_as_uint(x.x);
    v.y = __float_as_uint(x.y);
    __builtin_amdgcn_raw_buffer_store_b64(v, r, pix * 8u, 0, kNT);
}
__device__ __forceinline__ void bst_nt(const bf16x2 *, BandRsrc r, uint32_t pix, float2 x)
{
    bf16 a, b;
    st(&a, x.x);
    st(&b, x.y);
    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)a.bits | ((uint32_t)b.bits << 16), r, pix * 4u, 0, kNT);
}
__device__ __forceinline__ void bst_nt(const float4 *, BandRsrc r, uint32_t pix, float4 x)
{
    u32x4 v;
    v.x = __float_as_uint(x.x);
    v.y = __float_as_uint(x.y);
    v.z = __float_as_uint(x.z);
    v.w = __float_as_uint(x.w);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, pix * 16u, 0, kNT);
}
// one component (c = 0 first, 1 second) of a stored pair
__device__ __forceinline__ void bst_comp_nt(const float2 *, BandRsrc r, uint32_t pix, int c, float x)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, pix * 8u + 4u * (uint32_t)c, 0, kNT);
}
__device__ __forceinline__ void bst_comp_nt(const bf16x2 *, BandRsrc r, uint32_t pix, int c, float x)
{
    bf16 b;
    st(&b, x);
    __builtin_amdgcn_raw_buffer_store_b16(b.bits, r, pix * 4u + 2u * (uint32_t)c, 0, kNT);
}

struct Dims {
    int n1, n2, n3;
    int64_t plane;  // N = n1*n2*n3 (distance between planes of a field)
};

__device__ __forceinline__ int64_t vox(const Dims &d, int k, int i, int j)
{
    return ((int64_t)k * d.n1 + i) * d.n2 + j;
}

// Masks of the forward differences (Neumann boundary): an edge exists between
// index x and x+1 only for x <= n-2.
__device__ __forceinline__ float mask_le(int x, int n) { return (x >= 0 && x <= n - 2) ? 1.0f : 0.0f; }

// Group shrink of eq. (24) on one pair: scale by max(1 - thr/||(a, b)||, 0),
// with the reciprocal square root instruction (about 1 ulp); a zero pair
// gives rsq = +inf and a zero scale.
__device__ __forceinline__ void shrink2(float &a, float &b, float thr)
{
    const float r = __builtin_amdgcn_rsqf(a * a + b * b);
    const float f = fmaxf(1.0f - thr * r, 0.0f);
    a *= f;
    b *= f;
}

// x moved between lanes by a DPP control (lanes without a source get 0).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_double(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Wavefront-wide sum of a double (64 lanes), the same in every lane: within
// rows of 16 lanes by shifts of 1, 2, 4, 8, then across the rows, by DPP moves
// of the vector unit. As cross-lane LDS moves (six dependent round trips, two
// moves each, queueing on one unit per CU) the sums of eleven values by the 16
// wavefronts of a sweep tile took about 4 us.
__device__ __forceinline__ double wave_sum(double x)
{
    x += dpp_double<0x111, 0xf>(x);  // row_shr:1
    x += dpp_double<0x112, 0xf>(x);  // row_shr:2
    x += dpp_double<0x114, 0xf>(x);  // row_shr:4
    x += dpp_double<0x118, 0xf>(x);  // row_shr:8: lane 15 of a row holds its sum
    x += dpp_double<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
    x += dpp_double<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3: lane 63
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Two values in, their sums over pairs of lanes out: the lower half of the lanes
// (SWAP 32: lanes 0..31; 16: the even rows of 16) the sums of a, the upper half
// those of b.
template <int SWAP>
__device__ __forceinline__ double sum_halves(double a, double b)
{
    const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
    auto swap = [](uint32_t p, uint32_t q) {
        if constexpr (SWAP == 32) return __builtin_amdgcn_permlane32_swap(p, q, false, false);
        else return __builtin_amdgcn_permlane16_swap(p, q, false, false);
    };
    const auto lo = swap((uint32_t)x, (uint32_t)y), hi = swap((uint32_t)(x >> 32), (uint32_t)(y >> 32));
    return __longlong_as_double((long long)((uint64_t)hi[0] << 32 | lo[0])) +
           __longlong_as_double((long long)((uint64_t)hi[1] << 32 | lo[1]));
}
// Sum over each half row of 8 lanes, in all of them.
__device__ __forceinline__ double sum_half_row(double x)
{
    x += dpp_double<0x141, 0xf>(x);  // row_half_mirror
    x += dpp_double<0xb1, 0xf>(x);   // quad_perm 1 0 3 2
    x += dpp_double<0x4e, 0xf>(x);   // quad_perm 2 3 0 1
    return x;
}
// Wavefront-wide sums of eight values at once: the lanes halve with each step,
// so it takes 10 additions where eight sums by themselves take 48. Lane 8 h + 16 r
// and the 7 after it get the sum of value 4 h + (r & 1) * 2 + (r >> 1).
__device__ __forceinline__ double wave_sums8(const double (&x)[8])
{
    const double a = sum_halves<16>(sum_halves<32>(x[0], x[1]), sum_halves<32>(x[2], x[3]));
    const double b = sum_halves<16>(sum_halves<32>(x[4], x[5]), sum_halves<32>(x[6], x[7]));
    const bool h = (__lane_id() & 8) != 0;
    return sum_half_row((h ? b : a) + dpp_double<0x128, 0xf>(h ? a : b));  // row_ror:8
}

// Wavefront-wide sums of two values: a's in lanes 0..31, b's in the others.
__device__ __forceinline__ double wave_pair(double a, double b)
{
    const double x = sum_halves<32>(a, b), y = sum_halves<16>(x, x);
    return sum_half_row(y + dpp_double<0x128, 0xf>(y));  // row_ror:8
}
// Wavefront-wide minimum (no NaN among the lanes), in every lane.
__device__ __forceinline__ float wave_min(float x)
{
    auto dpp = [](float v, auto ctrl) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), decltype(ctrl)::value,
                                                                     0xf, 0xf, true));
    };
    x = fminf(x, dpp(x, std::integral_constant<int, 0x128>()));  // row_ror:8
    x = fminf(x, dpp(x, std::integral_constant<int, 0x141>()));  // row_half_mirror
    x = fminf(x, dpp(x, std::integral_constant<int, 0xb1>()));   // quad_perm 1 0 3 2
    x = fminf(x, dpp(x, std::integral_constant<int, 0x4e>()));   // quad_perm 2 3 0 1
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fminf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// The value of one lane, uniform.
__device__ __forceinline__ double lane_double(double x, int lane)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Block-wide sum for blocks of up to 1024 threads; result valid in thread 0.
template <int NT>
__device__ __forceinline__ double block_sum(double x, double *lds /* NT/64 */)
{
    x = wave_sum(x);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) lds[wid] = x;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < NT / 64; ++w) s += lds[w];
    return s;
}

}  // namespace geo

namespace geo {

// Radix levels of the exact l1-ball threshold search over FP32 bit patterns
// of |z|: level 0 = bits 30..20 (2048 bins), 1 = bits 19..10, 2 = bits 9..0.
__device__ __forceinline__ uint32_t abs_bits(float x) { return __float_as_uint(x) & 0x7fffffffu; }
__device__ __forceinline__ uint64_t significand(uint32_t p)
{
    const uint32_t e = p >> 23, m = p & 0x7fffffu;
    return e ? (uint64_t)(m | 0x800000u) : (uint64_t)m;
}
__device__ __forceinline__ int lvl_shift(int level) { return level == 0 ? 20 : (level == 1 ? 10 : 0); }
__device__ __forceinline__ int lvl_bins(int level) { return level == 0 ? 2048 : 1024; }
// exponent shared by the values of a bin of the given level
__device__ __forceinline__ uint32_t lvl_exponent(int level, uint32_t prefix, int b)
{
    return level == 0 ? (uint32_t)(b >> 3) : (level == 1 ? (prefix >> 3) : (prefix >> 13));
}

// The inputs of the two l1-ball projections (steps 2 and 3 of Alg. 1) and
// y4, with every rounding fixed (contraction off, the one fused operation
// written as such), so that every kernel that evaluates them (the sweeps, the
// search and the histogram passes) gets bit-identical values: the rounding
// intrinsics alone do not keep the compiler from fusing them with what
// follows. y4 is stored as q = 5 y4' - v, the residual of the fidelity ball
// before step 15 rescales it, and read as y4 = a q with a device factor a
// (max(0, 1 - eps/||q||) / 5 after an iteration).
__device__ __forceinline__ float y4_of(float q, float a)
{
#pragma clang fp contract(off)
    return a * q;
}
__device__ __forceinline__ float zs_of(float s, float y4)
{
#pragma clang fp contract(off)
    return s - y4;
}
// e = y3 at (i-1) (0 on the first row) minus y3 at i masked by m_v(i), step
// the step size of t (1/3 here; 1/5 for the comparison regularizers)
__device__ __forceinline__ float zt_of(float t, float e, float y4, float step)
{
#pragma clang fp contract(off)
    const float x = e + y4;
    return __builtin_fmaf(-step, x, t);
}
__device__ __forceinline__ float zt_of(float t, float y3m, float y3c, float y4, float step)
{
#pragma clang fp contract(off)
    const float e = y3m - y3c;
    return zt_of(t, e, y4, step);
}

}  // namespace geo
