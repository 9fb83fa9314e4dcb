// The end of an iteration of Alg. 1 and the thresholds of the next one.
//
// The sweep (sweep.hip) does steps 1-14 in one pass, so the thresholds
// tau_s, tau_t of the l1-ball projections (steps 2, 3) must be known before
// it starts, and they depend on y4 = a4 q, whose factor a4 comes out of the
// norm of the residual q over the whole cube (step 15) at the end of the
// sweep before. The sweep therefore gathers the inputs of the next search
// for a whole interval of a4 (predicted from its last values, which follow a
// smooth path): a value z of the next iteration is linear in a4, and
// monotone also as evaluated in FP32, so its values at the ends of the
// interval bound it.
//   above:     |z| > window at both ends, same sign: counted, |z| at the
//              interval's centre and its slope in a4 summed;
//   below:     |z| < window at both ends: ignored;
//   candidate: anything else: (x, e, q) recorded, z evaluated here.
// This kernel closes the iteration (r, a4, the stopping rule, the counter),
// then searches each field's threshold: f(x) = sum max(|z| - x, 0) = radius
// within the window. A window or an interval that missed leaves the field
// pending for the histogram passes of the next launch slot (fallback.hip).
#include <type_traits>

#include "radix.hpp"

namespace geo {

namespace {

// What bounds this kernel is latency: it works on a few hundred tile partials
// and a few thousand candidates in one block per field. 256 x 256 x 128: with
// 1024 threads and cross-lane sums through LDS 22 us (4.6K candidates; the moves
// of 16 wavefronts queue on one LDS unit); with 256 threads, straight-line loads
// (no branch around one, so that a thread's batch is in flight together) and sums
// by vector-unit moves 12 us with 2.5K candidates, 31 us at 512 x 512 x 224
// (8.9K); with 512 threads 13 and 26 us, and 37 instead of 54 us for the widest
// windows of the first iterations. Then the partials' sums eight at a time, over
// the wavefronts by lanes, batches of six candidates when there are few, and no
// pass to see that nothing changed: 10 us (its first loads 2.6, sums and scan 1.1,
// candidates 2.3, passes 2.5, windows 0.8), an iteration of 64 x 64 x 16 28.9 ->
// 26.3 us, of 120 x 120 x 198 126.3 -> 124.1.
constexpr int kSrThreads = 512;
constexpr int kSrWaves = kSrThreads / 64;
constexpr int kSrList = 32768;  // candidates held in LDS
constexpr int kSrFew = 6;       // candidates of a thread that calm windows stay below
constexpr int kSrSplit = 4;     // parts a streamed window is split into per round
constexpr int kBeginThreads = 1024;

// Count and sum of some values; the sums are of multiples of one unit below
// 2^53 units, so they are exact in FP64, in any order.
struct PassSum {
    double cnt, sum;
};

// Count and sum of the listed values above some point, and the least of them.
struct Pass {
    double cnt, sum;
    float least;
};

// Block sums of N pairs. buf: alternates between two calls, so that one barrier
// each is enough.
template <int N>
__device__ __forceinline__ void block_pairs(PassSum (&x)[N], PassSum (*buf)[kSrWaves])
{
#pragma unroll
    for (int k = 0; k < N; ++k) {
        x[k].cnt = wave_sum(x[k].cnt);
        x[k].sum = wave_sum(x[k].sum);
    }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) buf[k][threadIdx.x >> 6] = x[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        x[k] = buf[k][0];
#pragma unroll
        for (int w = 1; w < kSrWaves; ++w) {
            x[k].cnt += buf[k][w].cnt;
            x[k].sum += buf[k][w].sum;
        }
    }
}

// One block per (cube, field): block 2c + f. Field 0's block also closes the
// cube's iteration.
__global__ __launch_bounds__(kSrThreads) void k_search(const char *table, int stride, int ncubes)
{
    const const4<CubeCommon> &cc = *(const4<CubeCommon> *)(table + (size_t)(blockIdx.x >> 1) * stride);
    const int f = blockIdx.x & 1, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    DevScalars *sc = cc.sc;
    __shared__ SelState s;
    __shared__ uint32_t was_pending;
    __shared__ double wsum[8 * kSrWaves];
    __shared__ uint32_t wcnt[kSrWaves], wovf[kSrWaves];
    __shared__ uint32_t pre[kMaxTiles + 1];
    __shared__ float list[kSrList];
    __shared__ uint32_t nlist;
    __shared__ PassSum pbuf[2][kSrSplit + 2][kSrWaves];
    __shared__ Pass pass_buf[2][kSrWaves];

    // every first read goes out together; an idle cube has read a few KB for
    // nothing
    const float view_lo = sc->view.a_lo, view_hi = sc->view.a_hi, view_c = sc->view.a_c;
    const uint32_t view_idle = sc->view.idle;
    const int nt = cc.ntiles;
    const uint32_t capt = (uint32_t)cc.capt;
    const int per = (nt + kSrThreads - 1) / kSrThreads;  // consecutive tiles of a thread
    double acc[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // du2, u2, r2, count, S, Q, inside
    uint32_t mine = 0u, ovf = 0u;
    const double eps = sc->eps, gy4 = sc->gy4, tol = sc->tol;
    // (field 0's block alone writes these; field 1's does not use them)
    const A4History hist_a4 = a4_history(sc);
    const uint32_t iter = sc->iter, calls = sc->calls_iter;
    if (tid == 0) {
        const SelState s0 = sc->sel[f];
        was_pending = s0.done ? 0u : 1u;
        s = resolved(s0, cc.rec, f, cc.d.plane);
        nlist = 0u;
    }
    // four tiles' loads in flight (a tile past the thread's share repeats one
    // of the cube's and counts for nothing)
    for (int k0 = 0; k0 < per; k0 += 4) {
        double p[4][7];
        uint32_t c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = per * tid + k0 + u, bb = k0 + u < per && b < nt ? b : 0;
            const double *q = cc.part + 3 * (int64_t)bb, *w = cc.winpart + ((int64_t)f * nt + bb) * 4;
#pragma unroll
            for (int i = 0; i < 3; ++i) p[u][i] = q[i];
#pragma unroll
            for (int i = 0; i < 4; ++i) p[u][3 + i] = w[i];
            c[u] = cc.ccount[(int64_t)f * nt + bb];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = per * tid + k0 + u;
            if (k0 + u < per && b < nt) {
#pragma unroll
                for (int i = 0; i < 7; ++i) acc[i] += p[u][i];
                pre[b] = c[u] < capt ? c[u] : capt;
                mine += c[u] < capt ? c[u] : capt;
                ovf |= c[u] > capt ? 1u : 0u;
            }
        }
    }
    if (view_idle) return;
    // sums (a butterfly in each wavefront, then the wavefronts in order) and
    // the scan of the tiles' candidate counts
    uint32_t inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)inc, o, 64);
        if (lane >= o) inc += y;
    }
    const double all[8] = {acc[0], acc[1], acc[2], acc[3], acc[4], acc[5], acc[6], 0.0};
    const double s8 = wave_sums8(all);  // lanes 16 r + 8 h: value 4 h + 2 (r & 1) + (r >> 1)
    const int v8 = ((lane >> 3) & 1) * 4 + ((lane >> 4) & 1) * 2 + (lane >> 5);
    const bool any_ovf = __ballot(ovf != 0u) != 0ull;
    if (lane == 63) wcnt[wv] = inc;
    if ((lane & 7) == 0) wsum[v8 * kSrWaves + wv] = s8;
    if (lane == 0) wovf[wv] = any_ovf ? 1u : 0u;
    __syncthreads();
    uint32_t total = 0u, before = 0u, overflow = 0u;
#pragma unroll
    for (int w = 0; w < kSrWaves; ++w) {
        before += w < wv ? wcnt[w] : 0u;
        total += wcnt[w];
        overflow |= wovf[w];
    }
    // (eight wavefronts: value q over them in lanes 8 q .. 8 q + 7)
    static_assert(kSrWaves == 8, "a half row of lanes adds over the wavefronts");
    const double tot = sum_half_row(wsum[lane]);
#pragma unroll
    for (int q = 0; q < 7; ++q) acc[q] = lane_double(tot, 8 * q);
    {
        uint32_t at = before + inc - mine;
        for (int k = 0; k < per; ++k) {
            const int b = per * tid + k;
            if (b < nt) {
                const uint32_t c = pre[b];
                pre[b] = at;
                at += c;
            }
        }
        if (tid == 0) pre[nt] = total;
    }
    const double r = sqrt(acc[2]);
    const double c4 = r > eps ? 1.0 - eps / r : 0.0;
    const double a4d = gy4 * c4;
    const float a4 = (float)a4d;
    const float g = f ? cc.zt_step : 1.f;  // z = x - g (e + a4 q); e = 0 for s
    const bool in_iv = a4 >= view_lo && a4 <= view_hi;
    const double radius = s.radius;
    const bool won = s.win_on != 0u;
    const double lo = (double)s.win_lo, hi = (double)s.win_hi;
    int verdict = 0;  // 0 searching, 1 done, 2 missed
    double tau = 0.0;
    const uint32_t n_in = won ? (uint32_t)acc[6] : 0u;  // values inside the window
    if (radius <= 0.0) {
        verdict = 1;
        tau = __longlong_as_double(0x7ff0000000000000ll);
    } else if (!won) {
        // inside the ball so far: S and Q are sum |z| at the two ends of the
        // interval, and sum |z| is convex in a4, so the chord bounds it
        const double wd = (double)view_hi - (double)view_lo;
        const double x = wd > 0.0 ? ((double)a4 - (double)view_lo) / wd : 0.0;
        const double bound = (1.0 - x) * acc[4] + x * acc[5];
        verdict = in_iv && bound * (1.0 + 1e-5) <= radius ? 1 : 2;
    } else if (!in_iv || overflow || (double)total > fmax((double)kSrList, 2.0 * window_budget(cc.d.plane))) {
        verdict = 2;
    }
    __syncthreads();  // pre complete
    // sum and count of the values above the window, at this a4
    double Sh = acc[4] - ((double)a4 - (double)view_c) * (double)g * acc[5], Ch = acc[3];
    if (verdict == 0) {
        // the values, below zmax = 64 hi, rounded to multiples of a unit of which
        // total * zmax is less than 2^52: with few candidates finer than the
        // last bit of values near the window
        const int eh = ilogbf(fmaxf(s.win_hi, 1e-30f)) + 7;
        const float zmax = ldexpf(1.f, eh);
        const double rnd = ldexp(1.5, eh + (32 - __clz((int)total | 1)) + 1);  // 1.5 * 2^52 units
        bool wild = false;  // a value far above the window, or NaN
        auto fixed = [&](float z) { return ((double)z + rnd) - rnd; };
        auto eval = [&](const float4 &c) {
            const float z = fabsf(zt_of(c.x, c.y, y4_of(c.z, a4), g));
            if (!(z < zmax)) wild = true;
            return z;
        };
        const float4 *cand = cc.cand + (int64_t)f * nt * capt;
        int buf = 0;
        double wlo = lo, whi = hi;  // the range searched in LDS
        if (total <= (uint32_t)kSrList) {
            // positions tid, tid + kSrThreads, ... of the tiles' slices one after
            // another, a batch of loads in flight; a thread reads back only what
            // it staged
            // (a batch no larger than what there is: 2K candidates in batches of
            // 16 a thread took 1 us longer)
            auto stage = [&](auto batch) {
                constexpr int U = decltype(batch)::value;
                for (uint32_t p0 = (uint32_t)tid; p0 < total; p0 += U * kSrThreads) {
                    // (straight-line: positions past the end repeat the last one)
                    float4 c[U];
                    uint32_t p[U];
                    int a[U];
#pragma unroll
                    for (int e = 0; e < U; ++e) {
                        p[e] = p0 + e * kSrThreads < total ? p0 + e * kSrThreads : total - 1u;
                        a[e] = 0;
                    }
                    // the last tile whose slice starts at or before p
                    for (int step = 1 << (31 - __clz(nt)); step > 0; step >>= 1)
#pragma unroll
                        for (int e = 0; e < U; ++e) {
                            const int m = a[e] + step < nt ? a[e] + step : nt;  // pre[nt] = total
                            a[e] = pre[m] <= p[e] ? m : a[e];
                        }
#pragma unroll
                    for (int e = 0; e < U; ++e) c[e] = cand[(uint32_t)a[e] * capt + (p[e] - pre[a[e]])];
#pragma unroll
                    for (int e = 0; e < U; ++e) {
                        const float z = eval(c[e]);
                        if (p0 + e * kSrThreads < total) list[p0 + e * kSrThreads] = z;
                    }
                }
            };
            if (total <= kSrFew * kSrThreads)
                stage(std::integral_constant<int, kSrFew>());
            else
                stage(std::integral_constant<int, 16>());
        } else {
            // every candidate once: L lanes a tile's entries, U x 64 / L tiles of a
            // wavefront at a time. Many tiles of few entries (4096 of 15 in 4 bands of
            // 2048 x 2048) take 8 lanes each: with a wavefront to a tile, four at a
            // time, an SSTV iteration of 610 x 340 x 103 with 60K candidates took
            // 675 us, now 503 to 530 (445 with few).
            auto tiles = [&](auto lanes, auto loads, auto fn) {
                constexpr int L = decltype(lanes)::value, U = decltype(loads)::value, G = 64 / L;
                const int grp = lane / L;
                for (int b0 = G * U * wv; b0 < nt; b0 += G * U * kSrWaves) {
                    uint32_t n[U], nm = 0u;
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        const int b = b0 + q * G + grp;
                        n[q] = b < nt ? pre[b + 1] - pre[b] : 0u;
                        nm = n[q] > nm ? n[q] : nm;
                    }
                    for (uint32_t i = (uint32_t)(lane & (L - 1)); i < nm; i += L) {
                        float4 c[U];
#pragma unroll
                        for (int q = 0; q < U; ++q)
                            c[q] = cand[i < n[q] ? (uint32_t)(b0 + q * G + grp) * capt + i : 0u];
#pragma unroll
                        for (int q = 0; q < U; ++q)
                            if (i < n[q]) fn(eval(c[q]));
                    }
                }
            };
            auto each = [&](auto fn) {
                if (total > 64u * (uint32_t)nt)
                    tiles(std::integral_constant<int, 64>(), std::integral_constant<int, 4>(), fn);
                else
                    tiles(std::integral_constant<int, 8>(), std::integral_constant<int, 8>(), fn);
            };
            // Streamed: each round sums the values above kSrSplit points of the
            // range and keeps the part that holds tau, until what lies in it
            // fits LDS.
            for (int round = 0; round < 20 && verdict == 0; ++round) {
                PassSum x[kSrSplit + 1];
                double th[kSrSplit + 1];
                float tf[kSrSplit + 1];  // z > th as FP32: z above the last float at or below it
                uint32_t above[kSrSplit + 1];
#pragma unroll
                for (int k = 0; k <= kSrSplit; ++k) {
                    x[k] = {0.0, 0.0};
                    above[k] = 0u;
                    th[k] = k == kSrSplit ? whi : wlo + (whi - wlo) * ((double)k / kSrSplit);
                    tf[k] = __double2float_rd(th[k]);
                }
                each([&](float z) {
                    const double v = fixed(z);
#pragma unroll
                    for (int k = 0; k <= kSrSplit; ++k) {
                        above[k] += z > tf[k] ? 1u : 0u;
                        x[k].sum += z > tf[k] ? v : 0.0;
                    }
                });
                if (__syncthreads_or(wild ? 1 : 0)) {
                    verdict = 2;
                    break;
                }
#pragma unroll
                for (int k = 0; k <= kSrSplit; ++k) x[k].cnt = (double)above[k];
                block_pairs(x, pbuf[buf]);
                buf ^= 1;
                int best = -1;
#pragma unroll
                for (int k = 0; k <= kSrSplit; ++k)
                    if ((Sh + x[k].sum) - th[k] * (Ch + x[k].cnt) >= radius) best = k;
                if (best < 0 || best == kSrSplit) {
                    verdict = 2;  // below or above the window
                    break;
                }
                float flo = 0.f, fhi = 0.f;
                double cin = 0.0, nS = 0.0, nC = 0.0, nlo = 0.0, nhi = 0.0;
#pragma unroll
                for (int k = 0; k < kSrSplit; ++k)
                    if (k == best) {
                        cin = x[k].cnt - x[k + 1].cnt;
                        nS = x[k + 1].sum;
                        nC = x[k + 1].cnt;
                        nlo = th[k];
                        nhi = th[k + 1];
                        flo = tf[k];
                        fhi = tf[k + 1];
                    }
                wlo = nlo;
                whi = nhi;
                if (cin <= (double)kSrList) {
                    // the values above the part join the sums, those in it the list
                    Sh += nS;
                    Ch += nC;
                    each([&](float z) {
                        if (z > flo && !(z > fhi)) {
                            const uint32_t q = atomicAdd(&nlist, 1u);
                            if (q < (uint32_t)kSrList) list[q] = z;
                        }
                    });
                    __syncthreads();
                    total = nlist < (uint32_t)kSrList ? nlist : (uint32_t)kSrList;
                    verdict = -1;  // found its part
                } else if (round == 19) {
                    verdict = 2;
                }
            }
            if (verdict == -1) verdict = 0;
        }
        if (verdict == 0) {
            // count and sum of the listed values above t, and the least of them
            auto pass = [&](double t) {
                const float tf = __double2float_rd(t);
                double sum = 0.0;
                float n = 0.f, least = __int_as_float(0x7f800000);
                for (uint32_t p0 = (uint32_t)tid; p0 < total; p0 += kSrFew * kSrThreads) {
                    float z[kSrFew];
#pragma unroll
                    for (int e = 0; e < kSrFew; ++e) {
                        const uint32_t p = p0 + e * kSrThreads;
                        z[e] = list[p < total ? p : total - 1u];
                        z[e] = p < total ? z[e] : -1.f;
                    }
#pragma unroll
                    for (int e = 0; e < kSrFew; ++e) {
                        n += z[e] > tf ? 1.f : 0.f;
                        sum += z[e] > tf ? fixed(z[e]) : 0.0;
                        least = fminf(least, z[e] > tf ? z[e] : least);
                    }
                }
                if (wild) sum = __longlong_as_double(0x7ff8000000000000ll);  // NaN: no verdict below
                // over the wavefront, then over the eight of them; the two buffers
                // alternate, so that one barrier each is enough
                const double s2 = wave_pair(sum, (double)n);
                least = wave_min(least);
                Pass *o = &pass_buf[buf][wv];
                if (lane == 0) {
                    o->sum = s2;
                    o->least = least;
                }
                if (lane == 32) o->cnt = s2;
                __syncthreads();
                const Pass w = pass_buf[buf][lane & 7];
                buf ^= 1;
                Pass y;
                y.sum = lane_double(sum_half_row(w.sum), 0);
                y.cnt = lane_double(sum_half_row(w.cnt), 0);
                y.least = wave_min(w.least);  // (the lanes repeat the eight)
                return y;
            };
            // Newton's iteration on the convex decreasing f from the centre of
            // the range (the predicted threshold when the whole window is
            // searched): a tangent's root never exceeds the root of f, so from
            // the first one on the iterates rise to it, and the one whose set of
            // values above it no longer changes is exact: tau = (S - radius) / C.
            // The first one may fall short of the range, below which the values
            // are not known: the iteration then goes on from the lower end, if f
            // there is at least the radius.
            double C = -1.0;  // values above the point before
            bool first = true, at_lo = false;
            tau = 0.5 * (wlo + whi);
            verdict = 2;
            for (int it = 0; it < 64 && tau <= whi; ++it) {
                const Pass y = pass(tau);
                const double Cn = Ch + y.cnt, Sn = Sh + y.sum;
                if (Cn == C) {
                    verdict = 1;
                    break;
                }
                const double tn = Cn > 0.0 ? (Sn - radius) / Cn : -1.0;
                if (first) {
                    first = false;
                    if (!(tn >= wlo)) {
                        if (!(tn < wlo)) break;  // NaN
                        tau = wlo;
                        at_lo = true;
                        continue;
                    }
                } else if (!(tn > tau)) {
                    // f(tau) = radius up to rounding, or the range lies above tau
                    if (!at_lo || Sn - tau * Cn >= radius) verdict = 1;
                    break;
                }
                at_lo = false;
                C = Cn;
                // no value between here and there: the set above does not change
                const bool same = tn >= tau && tn <= whi && !((double)y.least <= tn);
                tau = tn;
                if (same) {
                    verdict = 1;
                    break;
                }
            }
            if (!(tau >= lo && tau <= hi)) verdict = 2;
        }
    }
    if (tid == 0) {
        sc->tau_used[f] = s.tau;
        sc->cand_used[f] = s.cand_count;
        if (was_pending) sc->missed[f] = sc->missed[f] + 1u;
        SelState o = s;
        o.cand_count = n_in;
        if (verdict == 1) {
            o.done = 1u;
            o.tau = tau;
            const double wdt = hi - lo;
            o.dens = won && wdt > 0.0 ? (double)n_in / wdt : 0.0;
            set_window(o, false, ahead_budget(cc.d.plane), s.calm >= kAheadCalm ? kWindowFillCalm : kAheadFill,
                       true);
            o.calm = s.calm + 1u;
        } else {
            o.done = 0u;
            o.full = 1u;
            o.win_on = 0u;
            o.calm = 0u;
            *slot_flags(table, ncubes) = 1u;  // the next slot's histogram passes run
        }
        sc->sel[f] = o;
        sc->in.set(f, o);
    }
    if (f == 0 && tid == 64) {  // another wavefront, beside the one above
        const double du2 = acc[0], u2 = acc[1];
        const double rel = u2 > 0.0 ? sqrt(du2) / sqrt(u2) : __longlong_as_double(0x7ff0000000000000ll);
        const bool bad = !isfinite(du2) || !isfinite(u2) || !isfinite(acc[2]);
        const uint32_t it = iter + 1u;
        sc->r = r;
        sc->rel = rel;
        sc->c4 = c4;
        sc->a4 = a4d;
        predict_a4(sc, hist_a4, gy4, a4d);
        sc->in.a4 = a4;
        sc->iter = it;
        sc->calls_iter = calls + 1u;
        if (bad) sc->nonfinite = 1u;
        // eq. (28), from the second iteration after the initial point on: the
        // first one (zero duals) changes u only by the box projection
        if (bad || (tol > 0.0 && it >= 2u && rel < tol)) sc->stop = 1u;
    }
    if (verdict != 1) clear_hist<kSrThreads>(cc.hist, f);
}

// Start of a call, one block per cube: its limits, and the fields whose
// threshold has to be found anew (a radius that changed since the search, or
// a search left pending).
__global__ __launch_bounds__(kBeginThreads) void k_begin(const char *table, int stride, int ncubes)
{
    const const4<CubeCommon> &cc = *(const4<CubeCommon> *)(table + (size_t)blockIdx.x * stride);
    DevScalars *sc = cc.sc;
    const double rad[2] = {cc.alpha, cc.beta};
    if (blockIdx.x == 0)
        for (int q = threadIdx.x; q < 3 * kFbMost; q += kBeginThreads) slot_flags(table, ncubes)[kFbClaimWord + q] = 0u;
    if (!cc.ahead) {  // the thresholds are searched within each iteration
        if (threadIdx.x == 0) {
            sc->tol = cc.tol;
            sc->calls_iter = 0u;
            sc->call_limit = cc.limit;
            sc->fallback = 0u;
            sc->sel[0].radius = rad[0];
            sc->sel[1].radius = rad[1];
            if (!sc->nonfinite) sc->stop = 0u;
        }
        return;
    }
    bool changed[2];
    for (int f = 0; f < 2; ++f) changed[f] = rad[f] != sc->sel[f].radius;
    __syncthreads();  // every thread has read the old radii
    for (int f = 0; f < 2; ++f)
        if (changed[f] && rad[f] > 0.0) clear_hist<kBeginThreads>(cc.hist, f);
    if (threadIdx.x == 0) {
        sc->tol = cc.tol;
        if (cc.set_eps) sc->eps = cc.eps;
        sc->calls_iter = 0u;
        sc->call_limit = cc.limit;
        bool pending = false;
        for (int f = 0; f < 2; ++f) {
            sc->missed[f] = 0u;
            if (changed[f]) {
                sc->sel[f].radius = rad[f];
                sc->sel[f].win_on = 0u;
                sc->sel[f].done = rad[f] > 0.0 ? 0u : 1u;
                if (!(rad[f] > 0.0)) sc->sel[f].tau = __longlong_as_double(0x7ff0000000000000ll);
                sc->in.set(f, sc->sel[f]);
            }
            pending = pending || !sc->sel[f].done;
        }
        if (!sc->nonfinite) sc->stop = 0u;
        if (pending) *slot_flags(table, ncubes) = 1u;
    }
}

// After a state load: y4 loaded as-is is read back with the factor 1, the
// predictions are dropped (the loaded state does not continue the previous
// run) and both thresholds are pending.
__global__ __launch_bounds__(kBeginThreads) void k_loaded(DevScalars *sc, Hist *hist, int y4)
{
    for (int f = 0; f < 2; ++f) clear_hist<kBeginThreads>(hist, f);
    if (threadIdx.x == 0) {
        if (y4) sc->a4 = 1.0;
        sc->a_n = 0u;
        sc->a_err = 0.0;
        sc->in.a4 = (float)sc->a4;
        sc->in.a_lo = 0.f;
        sc->in.a_hi = __double2float_ru(sc->gy4);
        sc->in.a_c = 0.5f * (float)sc->gy4;
        for (int f = 0; f < 2; ++f) {
            SelState &s = sc->sel[f];
            s.win_on = 0u;
            s.tau_prev = s.tau_prev2 = s.tau_prev3 = 0.0;
            s.err = 0.0;
            s.calm = 0u;
            s.done = s.radius > 0.0 ? 0u : 1u;
            if (!(s.radius > 0.0)) s.tau = __longlong_as_double(0x7ff0000000000000ll);
            sc->in.set(f, s);
        }
    }
}

constexpr int kReportThreads = 64;
static_assert(sizeof(DevScalars) % 8 == 0, "copied by words of 8 bytes");
__global__ __launch_bounds__(kReportThreads) void k_report(const char *table, int stride, uint64_t *out)
{
    const CubeCommon &cc = *(const CubeCommon *)(table + (size_t)blockIdx.x * stride);
    constexpr int words = sizeof(DevScalars) / 8;
    for (int q = threadIdx.x; q < words; q += kReportThreads)
        out[blockIdx.x * words + q] = reinterpret_cast<const uint64_t *>(cc.sc)[q];
}

}  // namespace

hipError_t launch_search(const void *table, int stride, int ncubes, hipStream_t st)
{
    hipLaunchKernelGGL(k_search, dim3(2 * ncubes), dim3(kSrThreads), 0, st, (const char *)table, stride, ncubes);
    return hipGetLastError();
}

hipError_t launch_begin(const void *table, int stride, int ncubes, hipStream_t st)
{
    hipLaunchKernelGGL(k_begin, dim3(ncubes), dim3(kBeginThreads), 0, st, (const char *)table, stride, ncubes);
    return hipGetLastError();
}

hipError_t launch_report(const void *table, int stride, int ncubes, DevScalars *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_report, dim3(ncubes), dim3(kReportThreads), 0, st, (const char *)table, stride, (uint64_t *)out);
    return hipGetLastError();
}

hipError_t launch_loaded(DevScalars *sc, Hist *hist, int var, hipStream_t st)
{
    hipLaunchKernelGGL(k_loaded, dim3(1), dim3(kBeginThreads), 0, st, sc, hist, var == GEO_VAR_Y4 ? 1 : 0);
    return hipGetLastError();
}

}  // namespace geo
