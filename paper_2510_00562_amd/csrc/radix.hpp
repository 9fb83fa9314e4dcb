// The radix levels of the exact l1-ball threshold search, read back from the
// per-level histograms of one field by a single wavefront.
//
// tau solves f(tau) = radius with f(x) = sum max(|z| - x, 0) (the threshold
// of the l1-ball projection of constraint sets (16), (17)). Over the FP32
// bit patterns P of |z| (monotone in the value), three histograms narrow the
// range that holds tau: level 0 bins bits 30..20 (2048 bins), level 1 bits
// 19..10 and level 2 bits 9..0 (1024 bins each) of the values whose higher
// bits equal the bins chosen before. At a bin edge e, f(e) = S(e) - e C(e)
// is exact from the counts and sums of the values at or above e; the level
// picks the highest bin whose lower edge has f >= radius. A level finishes
// the search when that bin is empty or holds one value (f is linear across
// the rest), when its edge gives f = radius exactly, or at level 2, where
// each bin is a single pattern.
//
// Every kernel that needs the outcome (the next level's histogram pass, the
// final pick) evaluates it from the same histograms with the same code: one
// wavefront in a fixed order, independent of the block size, so the FP64
// sums and every decision are bit-identical everywhere.
#pragma once

#include "solver.hpp"

namespace geo {

// Outcome of the radix levels so far for one field.
struct RadixPick {
    double tau;        // final level (done)
    double s_above;    // sum of the values above the current range
    double c_above;    // and their count (exact in FP64)
    double dens;       // values per unit of |z| in the bin chosen last (levels 0, 1)
    uint32_t prefix;   // bits fixed by the levels so far
    int level;         // next level to histogram (3: none)
    int done;
};

__device__ __forceinline__ double bin_scale(uint32_t e) { return ldexp(1.0, (int)(e ? e : 1u) - 150); }

// Where bin b is staged: a lane reads 32 (or 16) bins in a row, and with one word
// left out after every 32 the lanes' reads fall into different banks. (All in
// one bank, the pick took 3 us longer.)
constexpr int kHistStage = kHistBins + kHistBins / 32;
__device__ __forceinline__ int bin_at(int b) { return b + (b >> 5); }

// One level for one field from its histogram staged in LDS (bin sums as
// doubles in bs, counts in bc, bin b at bin_at(b)), by wavefront lanes 0..63 of
// the caller (every lane must call; all lanes return the same result). nb/64
// bins per lane, lane 0 the top ones.
__device__ __forceinline__ void radix_level_wave(const double *bs, const uint32_t *bc, double radius,
                                                 RadixPick &pk)
{
    const int level = pk.level;
    const int nb = level == 0 ? 2048 : 1024, shift = level == 0 ? 20 : (level == 1 ? 10 : 0);
    const int per = nb / 64;
    const int lane = __lane_id();
    const uint32_t base = level == 0 ? 0u : (pk.prefix << (level == 1 ? 20 : 10));
    const int btop = nb - 1 - per * lane;
    // this lane's bins, top down
    double ls = 0.0, lc = 0.0;
#pragma unroll 16
    for (int q = 0; q < per; ++q) {
        ls += bs[bin_at(btop - q)];
        lc += (double)bc[bin_at(btop - q)];
    }
    // inclusive scan over the lanes, lane 0 first
    double xs = ls, xc = lc;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double ys = __shfl_up(xs, o, 64), yc = __shfl_up(xc, o, 64);
        if (lane >= o) {
            xs += ys;
            xc += yc;
        }
    }
    // exclusive: the inclusive value of the lane before
    double es = __shfl_up(xs, 1, 64), ec = __shfl_up(xc, 1, 64);
    if (lane == 0) es = ec = 0.0;
    double S = pk.s_above + es, C = pk.c_above + ec;
    const double allS = pk.s_above + lane_double(xs, 63), allC = pk.c_above + lane_double(xc, 63);
    // down to the highest bin whose lower edge has f >= radius: S and C stay at the
    // sums strictly above it. (Without a way out of the loop, which left each
    // bin's reads to wait for the bin before.)
    int mine = btop;
    bool found = false;
#pragma unroll 16
    for (int q = 0; q < per; ++q) {
        const int b = btop - q;
        const double vs = bs[bin_at(b)], vc = (double)bc[bin_at(b)];
        const float eb = __uint_as_float(base | ((uint32_t)b << shift));
        found = found || (S + vs) - (double)eb * (C + vc) >= radius;
        mine = found ? mine : b - 1;
        S = found ? S : S + vs;
        C = found ? C : C + vc;
    }
    // the highest qualifying bin sits in the lowest lane that has one
    const unsigned long long hit = __ballot(found);
    double mS, mC, mbs, mbc, mfb;
    int b;
    if (hit) {
        const int src = __builtin_amdgcn_readfirstlane(__ffsll((long long)hit) - 1);
        b = __builtin_amdgcn_readlane(mine, src);
        mS = lane_double(S, src);
        mC = lane_double(C, src);
        mbs = bs[bin_at(b)];
        mbc = (double)bc[bin_at(b)];
        mfb = (mS + mbs) - (double)__uint_as_float(base | ((uint32_t)b << shift)) * (mC + mbc);
    } else {
        if (level == 0) {
            // f(0) = sum |z| < radius: inside the ball
            pk.tau = 0.0;
            pk.done = 1;
            pk.level = 3;
            return;
        }
        // FP64 rounding at the lower edge of a deeper range (f there is >=
        // radius by the choice of the range): take bin 0
        b = 0;
        mbs = bs[0];
        mbc = (double)bc[0];
        mS = allS - mbs;
        mC = allC - mbc;
        mfb = allS - (double)__uint_as_float(base) * allC;
    }
    const float eb = __uint_as_float(base | ((uint32_t)b << shift));
    if (level == 0) {
        // density of values around tau (sizes the next window); the top bin
        // (patterns of Inf/NaN) never holds tau for finite data
        const double e1 = b + 1 < nb ? (double)__uint_as_float((uint32_t)(b + 1) << shift) : (double)eb;
        pk.dens = e1 > (double)eb ? mbc / (e1 - (double)eb) : 0.0;
    } else if (level == 1) {
        // and closer to it, where the bin (1.2e-4 tau wide or less) holds enough
        // of them
        const double e1 = (double)__uint_as_float(base + ((uint32_t)(b + 1) << shift));
        pk.dens = mbc >= 64.0 ? mbc / (e1 - (double)eb) : 0.0;
    }
    if (mfb == radius) {
        pk.tau = (double)eb;
        pk.done = 1;
    } else if (mbc == 0.0 || level == 2) {
        pk.tau = (mS - radius) / mC;
        pk.done = 1;
    } else if (mbc == 1.0) {
        const double t1 = mC > 0.0 ? (mS - radius) / mC : -1.0;
        pk.tau = (mC > 0.0 && t1 >= mbs) ? t1 : (mS + mbs - radius) / (mC + 1.0);
        pk.done = 1;
    } else {
        pk.prefix = (level == 0 ? 0u : (pk.prefix << 10)) | (uint32_t)b;
        pk.s_above = mS;
        pk.c_above = mC;
    }
    pk.level = pk.done ? 3 : level + 1;
}

// Empty histograms (the three radix levels) of field f, by a block of NT threads.
template <int NT>
__device__ __forceinline__ void clear_hist(Hist *hist, int f)
{
    for (int q = threadIdx.x; q < 3 * kHistBins; q += NT) {
        Hist &h = hist[(q / kHistBins) * 2 + f];
        h.count[q % kHistBins] = 0u;
        h.msum[q % kHistBins] = 0ull;
    }
}

// Sums of K FP64 values over a block of NT threads; result valid in thread 0.
template <int K, int NT>
__device__ __forceinline__ void block_sums(double (&x)[K], double *red /* K * NT/64 */)
{
#pragma unroll
    for (int q = 0; q < K; ++q) x[q] = wave_sum(x[q]);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < K; ++q) red[q * (NT / 64) + wid] = x[q];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int q = 0; q < K; ++q) {
            double t = 0.0;
            for (int w = 0; w < NT / 64; ++w) t += red[q * (NT / 64) + w];
            x[q] = t;
        }
}

// What a sweep sums for the search of the next thresholds (search.hip), by
// field: |z| above the window at the interval's centre, its slope in a4, how
// many, and how many values are inside it; without a window, |z| at the two ends
// of the interval. The sums are FP64 (a tile has up to thousands of bands: in FP32
// a sum of 4096 equal values was low by 3.4e-5, more than the search's margin
// between inside the ball and outside), counts are per wavefront, in scalar
// registers.
struct Gathered {
    double sum[2] = {0.0, 0.0};
    uint32_t cnt[2] = {0u, 0u}, inside[2] = {0u, 0u};
};
// The slope's sums of a thread: in registers, or (SSTV's sweep, whose 80
// registers are all taken) in LDS words of its own.
struct SlopeRegs {
    double x[2] = {0.0, 0.0};
    __device__ __forceinline__ void add(int f, double v) { x[f] += v; }
    __device__ __forceinline__ double get(int f) const { return x[f]; }
};
template <int NT>
struct SlopeLds {
    __attribute__((address_space(3))) double *x;  // [2][NT], this thread's first
    __device__ __forceinline__ void add(int f, double v) const { __builtin_amdgcn_ds_atomic_fadd_f64(x + f * NT, v); }
    __device__ __forceinline__ double get(int f) const { return x[f * NT]; }
};

// The end of a sweep tile: the sums over the block of NT threads of x (the
// stopping rule's du2, u2, r2) and of what the next search needs, to the tile's
// partials. red: 10 NT / 64 words of 8 bytes. Every thread calls; the caller
// needs no barrier after it if several stand before it writes red again. (Eleven
// wavefront sums one after another and one thread that added them over the
// wavefronts took 9 us of a tile's 16 beside its bands.)
template <int NT, typename Slope>
__device__ __forceinline__ void tile_sums(double du2, double u2, double r2, const Gathered &ga, const Slope &sl, double *red,
                                          double *part, double *win0, double *win1)
{
    constexpr int NW = NT / 64;
    static_assert(NW <= 16, "a row of lanes adds over the wavefronts");
    uint32_t *cnt = reinterpret_cast<uint32_t *>(red + 8 * NW);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // (nothing below is worth a register before)
    const int lane = tid & 63, wid = tid >> 6, row = lane >> 4, col = lane & 15;
    const double x[8] = {du2, u2, r2, ga.sum[0], sl.get(0), ga.sum[1], sl.get(1), 0.0};
    const double s = wave_sums8(x);
    if ((lane & 7) == 0) red[((col >> 1) + (row & 1) * 2 + (row >> 1)) * NW + wid] = s;  // col >> 1: 0 or 4
    if (lane == 0) {
        cnt[wid] = ga.cnt[0];
        cnt[NW + wid] = ga.inside[0];
        cnt[2 * NW + wid] = ga.cnt[1];
        cnt[3 * NW + wid] = ga.inside[1];
    }
    __syncthreads();
    if (tid >= 64) return;
    // over the wavefronts: row r takes values r and 4 + r and count r
    const bool in = col < NW;
    double a = in ? red[row * NW + col] : 0.0, b = in ? red[(4 + row) * NW + col] : 0.0;
    double c = in ? (double)cnt[row * NW + col] : 0.0;
    a = sum_half_row(a + dpp_double<0x128, 0xf>(a));
    b = sum_half_row(b + dpp_double<0x128, 0xf>(b));
    c = sum_half_row(c + dpp_double<0x128, 0xf>(c));
    // count above, sum above, its slope in a4, count inside
    if (col == 0) *(row < 3 ? part + row : win0 + 1) = a;
    if (col == 1 && row < 3) *(row == 0 ? win0 + 2 : win1 + row) = b;
    if (col == 2) *((row < 2 ? win0 : win1) + 3 * (row & 1)) = c;
}

// The scalars of a state at the initial point.
__device__ inline void init_scalars(DevScalars *sc, double eps, double tol, double alpha, double beta, double gy4)
{
    DevScalars z = {};
    z.c4 = 1.0;
    z.a4 = 1.0;
    z.eps = eps;
    z.tol = tol;
    z.sel[0].radius = alpha;
    z.sel[1].radius = beta;
    // z_s = z_t = 0: inside the balls, tau = 0 (radius 0: +inf)
    for (int f = 0; f < 2; ++f) {
        z.sel[f].done = 1u;
        if (!(z.sel[f].radius > 0.0)) z.sel[f].tau = __longlong_as_double(0x7ff0000000000000ll);
        z.in.set(f, z.sel[f]);
    }
    z.gy4 = gy4;
    z.zstore = 1u;
    z.in.a4 = 1.f;
    z.in.a_hi = __double2float_ru(gy4);
    z.in.a_c = 0.5f * (float)gy4;
    *sc = z;
}

// Append val to this block's slice of a field's candidate list. The slot
// comes from an LDS counter (wavefront-aggregated), so a sweep never waits on
// a global atomic; entries past the slice's capacity are counted but
// dropped, which the search detects as an overflow. Every lane of the
// wavefront must call it.
template <typename T>
__device__ __forceinline__ void wave_append(bool want, const T &val, T *slice, uint32_t *lds_count, int capb)
{
    const unsigned long long m = __ballot(want);
    if (m == 0ull) return;
    const int lane = __lane_id();
    const int leader = __ffsll((long long)m) - 1;
    uint32_t base = 0u;
    if (lane == leader) base = atomicAdd(lds_count, (uint32_t)__popcll(m));
    base = __shfl(base, leader, 64);
    const uint32_t off = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    if (want && base + off < (uint32_t)capb) slice[base + off] = val;
}

// One value of the next search, z = x - g (e + a4 q), over the interval of a4.
// in: the lane has a value. Every lane of the wavefront takes part.
template <typename Slope>
__device__ __forceinline__ void gather_ahead(Gathered &o, Slope &sl, const4<DevScalars::SweepIn> &w, int f, bool in, float x,
                                             float e, float g, float q, float4 *slice, uint32_t *lds_count, int capt)
{
    const float zl = zt_of(x, e, y4_of(q, w.a_lo), g), zh = zt_of(x, e, y4_of(q, w.a_hi), g);
    if (!w.on[f]) {
        // inside the ball so far: sum |z| at both ends
        o.sum[f] += in ? (double)fabsf(zl) : 0.0;
        sl.add(f, in ? (double)fabsf(zh) : 0.0);
        return;
    }
    const float lo = w.lo[f], hi = w.hi[f];
    const float zmin = fminf(zl, zh), zmax = fmaxf(zl, zh);
    const float zc = zt_of(x, e, y4_of(q, w.a_c), g);
    const bool above = in && (zmin > hi || zmax < -hi);
    const bool below = zmin > -lo && zmax < lo;
    o.cnt[f] += (uint32_t)__popcll(__ballot(above));
    o.inside[f] += (uint32_t)__popcll(__ballot(in && fabsf(zc) >= lo && fabsf(zc) <= hi));
    o.sum[f] += above ? (double)fabsf(zc) : 0.0;
    sl.add(f, above ? (double)(copysignf(1.f, zc) * q) : 0.0);
    wave_append(in && !above && !below, make_float4(x, e, q, 0.f), slice, lds_count, capt);
}

// Candidates a window is widened to when the density of |z| near tau is
// known: the search handles that many in LDS at almost the same cost as a
// few, and a wider window misses less. Once the windows have held for
// kCalmNarrow iterations in a row (tau moves smoothly, and the half-width that
// the prediction errors ask for is a small part of this) the narrower fill
// saves the sweep's appends and the search's loads: one batch of 16 per
// thread instead of two (256 x 256 x 128, search 19 us at 4096 candidates,
// 13 us at 2048; before that 0.362 ms per iteration at 16384 and 0.3555 at
// 4096); from the start it would miss more.
constexpr double kWindowFill = 16384.0;
constexpr double kWindowFillCalm = 2048.0;
constexpr uint32_t kCalmNarrow = 8;
// FP32 duals (the search of search.hip, whose time follows the candidates): 8192,
// narrow after 6. From the initial point, 16384 and 8 before: 30 iterations of
// 64 x 64 x 16 1145 -> 1074 us, 60 of 128 x 128 x 64 4350 -> 4236, of 120 x 120 x
// 198 8370 -> 8347 with one miss more, of 256 x 256 x 128 19520 -> 19635 with two.
constexpr double kAheadFill = 8192.0;
constexpr uint32_t kAheadCalm = 6;

// Window of |z| that the sweep collects for the next iteration. tau is
// extrapolated from the last levels: quadratically once four are known (the
// levels follow a smooth path after the first iterations, and the quadratic
// error is a fraction of the linear one there), linearly from two or three.
// The half-width is twice the error the same extrapolation made for this
// iteration (plus 5e-5 tau, and never less than the last step plus 2e-4 tau
// when the history is short or the prediction failed). Three times the
// error plus 2e-4 tau held as well in steady state, with windows a third
// wider: the 512 x 512 x 224 search took 89 instead of 51 us. budget > 0
// and the density of |z| near tau known from this iteration: the window is
// widened to hold about `fill` values (the search's cost is flat up to
// there, and a wider window misses less) and narrowed to hold at most about
// `budget` (a window of hundreds of thousands of candidates costs the search
// more than the histogram passes that a miss costs).
// ahead (FP32 duals): the 5e-5 tau give way to 5% of the last step plus 1e-6
// tau where those are less, and the error is no less than half of the one
// before it. Towards convergence the values crowd around the thresholds while
// the steps shrink: HSSTV2 on 256 x 256 x 128 after 950 iterations had 260K
// values of t in a window that 5e-5 tau had set, and missed in every iteration
// (278 us each, 167 now).
__device__ inline void set_window(SelState &o, bool missed, double budget, double fill = kWindowFill,
                                  bool ahead = false)
{
    const double tau = o.tau;
    if (!(tau > 0.0) || !isfinite(tau)) {
        o.win_on = 0u;
        o.tau_prev3 = 0.0;
        o.tau_prev2 = 0.0;
        o.tau_prev = tau;
        return;
    }
    const double t1 = o.tau_prev, t2 = o.tau_prev2, t3 = o.tau_prev3;
    const bool h1 = t1 > 0.0 && isfinite(t1), h2 = h1 && t2 > 0.0 && isfinite(t2);
    const bool h3 = h2 && t3 > 0.0 && isfinite(t3);
    const double step = h1 ? tau - t1 : 0.05 * tau;
    double c = tau + (h1 ? step : 0.0);
    double err = h2 ? fabs(tau - (2.0 * t1 - t2)) : fabs(step);
    if (h3) {
        const double cq = 3.0 * (tau - t1) + t2;
        if (cq > 0.0) {
            c = cq;
            err = fabs(tau - (3.0 * (t1 - t2) + t3));
        }
    }
    double least = 5e-5 * tau;
    if (ahead) {
        if (h3) least = fmin(least, 0.05 * fabs(step) + 1e-6 * tau);
        const double e = err;
        err = fmax(err, 0.5 * o.err);
        o.err = e;
    }
    double h = 2.0 * err + least;
    if (!h2 || missed) h = fmax(h, fabs(step) + 2e-4 * tau);
    if (budget > 0.0 && o.dens > 0.0) {
        // as wide as the search's flat cost allows, narrower than the budget;
        // ahead: within [0, 2 tau], or a cube of fewer than `fill` values would
        // widen its window from iteration to iteration without end, and the
        // search sums in units of the window's upper end
        const double wide = fill / (2.0 * o.dens);
        h = fmax(h, ahead ? fmin(wide, tau) : wide);
        h = fmin(h, budget / (2.0 * o.dens));
    }
    double lo = c - h, hi = c + h;
    if (lo < 0.0) lo = 0.0;
    o.win_lo = __double2float_rd(lo);
    o.win_hi = __double2float_ru(hi);
    o.win_on = 1u;
    o.tau_prev3 = h2 ? t2 : 0.0;
    o.tau_prev2 = h1 ? t1 : 0.0;
    o.tau_prev = tau;
}

// Candidate budget of a cube's window: what LDS holds with room for the
// error of the density estimate (20K of the 28K), or for large cubes N/256,
// a streamed search that costs well under the three histogram passes over
// the field that a miss costs.
__host__ __device__ inline double window_budget(int64_t n)
{
    const double b = (double)n / 256.0;
    return b > 20480.0 ? b : 20480.0;
}

// FP32 duals: less where N/256 would overflow the 32768 that search.hip holds in
// LDS: 24576, room for the error of the estimate, or N/1024. A wide window pays while
// its search costs less than the miss that a narrow one risks. Of one field, in us:
//   a search   9 and 2 for each thousand candidates held in LDS (256 x 256 x 128: 22 with
//              8.1K, 57 to 67 with 24.5K); streamed, on one CU, 1 to 3 for each thousand
//              (512 x 512 x 224: 75 to 120 with 56K, 160 to 230 in the first ones); with
//              4096 tiles 30 more (2048 x 2048 x 4)
//   a miss     50 and 5 for each million voxels, over all CUs (64 x 64 x 16 55, 256 x 256
//              x 128 90, 2048 x 2048 x 4 124, 512 x 512 x 224 330; the other field of the
//              same slot adds a third to two thirds)
// so that a search at the budget takes two thirds of a miss at 8M voxels, half at 17M
// and a quarter to a third at 59M: more values than that would have to save almost
// every miss they cover, and windows grow by less than half from one iteration to
// the next while they miss. Whole solves move by 0.5 to 4% over the range (with
// N/256 the first 24 iterations of 512 x 512 x 224 took 55.5 ms, now 53.4, with N/2048
// 54.4; with 32768 or N/512 the first 30 of 2048 x 2048 x 4 26.7 ms, now 24.9; 25 of
// 256 x 256 x 128 9280 and 9207 us), a miss more or less among it. Less than 20480 for
// small cubes (12288, 8192): 64 x 64 x 16 1100 and 1133 instead of 1090 us, 120 x 120 x
// 198 8345 instead of 8297.
__host__ __device__ inline double ahead_budget(int64_t n)
{
    const double most = (double)n / 1024.0 > 24576.0 ? (double)n / 1024.0 : 24576.0;
    const double b = window_budget(n);
    return b < most ? b : most;
}

// The search state of field f as this slot's sweep and search use it: a
// field whose window missed takes its threshold from the slot's histogram
// passes, and the window of the iteration after it follows from that.
// r0, r1: the field's records of levels 0 and 1; last: of the level that ended it.
__device__ inline SelState resolved(const SelState &s, const FbRec &r0, const FbRec &r1, const FbRec &last, int64_t n)
{
    SelState o = s;
    o.tau = last.tau;
    o.dens = !r0.done && r1.dens > 0.0 ? r1.dens : r0.dens;
    o.done = 1u;
    o.full = 0u;
    set_window(o, true, ahead_budget(n), kAheadFill, true);
    return o;
}
__device__ inline SelState resolved(const SelState &s, const FbRec *rec, int f, int64_t n)
{
    return s.done ? s : resolved(s, rec[f], rec[2 + f], fb_final(rec, f), n);
}

// The interval in which the next a4 (y4 = a4 q) is expected, after a4 of this
// iteration: extrapolated like the thresholds, with a half-width of 2.5 times
// the larger of the last prediction's error and half of the one before it
// (an error that happens to cross zero says nothing) plus 5e-5 a4 or, once
// extrapolated quadratically, 5% of the last step and 1e-6 a4 if that is less:
// every value that some a4 of the interval moves across the window is recorded,
// and towards convergence those are many. Without a
// history, every value a4 can take: gy4 max(0, 1 - eps/r) lies in [0, gy4].
struct A4History {
    double p1, p2, p3;  // a4 of the iterations before
    double err;         // error of the last prediction
    uint32_t n;         // how many of them there are
};
__device__ inline A4History a4_history(const DevScalars *sc)
{
    return {sc->a_prev[0], sc->a_prev[1], sc->a_prev[2], sc->a_err, sc->a_n};
}
__device__ inline void predict_a4(DevScalars *sc, const A4History &h, double gy4, double a)
{
    double lo = 0.0, hi = gy4, c = 0.5 * gy4;
    if (h.n >= 2u) {
        const bool quad = h.n >= 3u;
        c = quad ? 3.0 * (a - h.p1) + h.p2 : 2.0 * a - h.p1;
        const double err = quad ? fabs(a - (3.0 * (h.p1 - h.p2) + h.p3))
                                : fabs(a - (2.0 * h.p1 - h.p2)) + fabs(a - h.p1);
        const double least = quad ? fmin(5e-5 * a, 0.05 * fabs(a - h.p1) + 1e-6 * a) : 5e-5 * a;
        const double w = 2.5 * fmax(err, 0.5 * h.err) + least;
        sc->a_err = err;
        lo = fmax(0.0, c - w);
        hi = fmin(gy4, c + w);
        if (!(lo <= hi)) lo = 0.0, hi = gy4;
        c = fmin(fmax(c, lo), hi);
    }
    sc->in.a_lo = __double2float_rd(lo);
    sc->in.a_hi = __double2float_ru(hi);
    sc->in.a_c = (float)c;
    sc->a_prev[2] = h.p2;
    sc->a_prev[1] = h.p1;
    sc->a_prev[0] = a;
    sc->a_n = h.n < 3u ? h.n + 1u : 3u;
}

}  // namespace geo
