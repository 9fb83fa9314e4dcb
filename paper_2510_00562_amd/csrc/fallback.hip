// Exact l1-ball thresholds whose predicted window missed, found inside one
// launch slot: three histogram passes over the field (the radix levels of
// radix.hpp) in one launch, before the sweep that needs the thresholds (FP32
// duals: the search at the end of the slot before left them pending) or between
// the window search and sweep B (BF16 duals).
// The launch is a no-op (its blocks read one flag and leave) unless a search left
// a field of some working cube pending. That takes 1.5 us, and with a launch for
// each level there were three of them: an iteration of 64 x 64 x 16 took 31.8 us,
// now 28.9, of 120 x 120 x 198 128.0, now 126.3.
// What bounds a level that works (256 x 256 x 128, one field, 88 us for the three):
// the state once, at level 0 (23 us; the values found there are kept for the next
// levels, which take 8 and 6 us over them), then a chain of round trips beyond the
// L2: the work and the claims 3 us, the atomics on the global bins 1 to 6, the
// bins read back 3, the pick 3 to 5. From the state at each level and with the
// claims in front of the work, 512 x 512 x 224 took 1.25 ms more over its first 16
// misses, and 60 iterations of 100 x 100 x 360 10512 instead of 10422 us.
// The voxels of the cubes with a pending field are split evenly into chunks, one
// per block of the launch. A block takes its own chunk and then those whose block
// has not come yet, reads z_s and z_t where sweep A stored them in this
// iteration (BF16), or else evaluates them from the state exactly as the sweep
// does (the same rounding operations, so the values are bit-identical), takes the
// values whose higher bits match the bins the earlier levels chose, and adds
// them to LDS histograms that are flushed into the cube's global histogram
// of the level with integer atomics (order-free, exact). The last block to
// finish a cube (a counter) reads the level back. Then the blocks wait for the
// level's cubes to be read back. They may: whatever is not done by then is in the
// hands of a block that has claimed it, so one that runs, and that does not wait
// before it is done; blocks that have not come yet hold nothing.
#include "radix.hpp"

namespace geo {

namespace {

// One 1024-thread block per CU: the blocks' atomics on a common bin of the
// global histogram are performed one after another, so fewer, larger blocks
// shorten that chain.
constexpr int kFbThreads = 1024;
constexpr int kFbUnroll = 4;    // voxels per thread in flight at once (from the state)
constexpr int kFbUnrollZ = 16;  // and from stored z (one load per field and voxel)

// Blocks of a pass whose voxel range [W b / G, W (b + 1) / G) meets the
// work range [c0, c1) of a cube (empty ranges inside it count too): the
// first is the smallest b with W (b + 1) / G > c0, the last the largest b
// with W b / G < c1 (integer divisions).
__device__ __forceinline__ int blocks_meeting(int64_t W, int G, int64_t c0, int64_t c1)
{
    const int64_t first = (G * (c0 + 1) + W - 1) / W - 1;
    const int64_t last = (G * c1 + W - 1) / W - 1;
    return (int)(last - first + 1);
}

// Words that pass between blocks while the launch runs: atomics and loads of
// system scope, performed beyond the XCD's L2.
__device__ __forceinline__ uint32_t word_load(const uint32_t *p)
{
    return __hip_atomic_load(const_cast<uint32_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
static_assert(sizeof(FbRec) % 8 == 0, "a record moves by words of 8 bytes");
__device__ __forceinline__ FbRec rec_load(const FbRec *p)
{
    FbRec o;
    uint64_t w[sizeof o / 8];
#pragma unroll
    for (unsigned k = 0; k < sizeof o / 8; ++k)
        w[k] = __hip_atomic_load((uint64_t *)p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __builtin_memcpy(&o, w, sizeof o);
    return o;
}
__device__ __forceinline__ void rec_store(FbRec *p, const FbRec &o)
{
    uint64_t w[sizeof o / 8];
    __builtin_memcpy(w, &o, sizeof o);
#pragma unroll
    for (unsigned k = 0; k < sizeof o / 8; ++k)
        __hip_atomic_store((uint64_t *)p + k, w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Per level: the histogram of every field whose window missed and whose search
// reached this level. The last block to finish a cube's share reads that cube's
// histograms back (the level's bin, or the threshold when the level ends the
// search) into the field's record of the level, which the next level, sweep B and
// the finalize read. Nothing that decides the work of a level changes once it has
// begun, so every block sees the same work whenever it comes.
template <typename DT>
__global__ __launch_bounds__(kFbThreads) void k_fb_hist(const CubeArgs<DT> *__restrict__ cubes, LaunchShape sh,
                                                        uint32_t *flags)
{
    if (flags[0] == 0u) return;  // no window missed in this slot
    const uint32_t run = flags[1] + 1u;  // of this launch (a later launch counts it)
    __shared__ uint32_t hc[2][kHistStage];
    __shared__ unsigned long long hm[2][kHistStage];
    __shared__ int64_t seg0[kMaxBatch + 1];  // first work index of each cube
    __shared__ uint32_t fmask[kMaxBatch];    // fields of each cube at this level
    __shared__ uint32_t prefix[2][kMaxBatch];  // and the bits their earlier levels fixed
    __shared__ int last, active, mine, next;
    __shared__ uint32_t mine0[kFbMost / 32];  // chunks of level 0 whose z this block stored
    static_assert(kMaxBatch <= 64, "one wavefront scans the cubes");
    const int tid = threadIdx.x;
    const int G = (int)gridDim.x;  // chunks
    int64_t W0 = 0;                // voxels at level 0: as many later means the same cubes
    if (tid < kFbMost / 32) mine0[tid] = 0u;
    for (int level = 0; level < 3; ++level) {
        uint32_t *claims = flags + kFbClaimWord + level * kFbMost;
        __syncthreads();
        if (tid == 64) {
            // this block's own chunk
            mine = __hip_atomic_exchange(&claims[blockIdx.x], run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != run ? 1 : 0;
            next = G;
            if (level == 0 && mine) mine0[blockIdx.x >> 5] |= 1u << (blockIdx.x & 31);
        }
        if (tid < 64) {
            const int c = tid;
            uint32_t m = 0u;
            int64_t n = 0;
            if (c < sh.ncubes) {
                const DevScalars *sc = cubes[c].c.sc;
                // fields still searching at this level: the window search and the
                // earlier levels decided it (a record is of this launch only if
                // no level before it ended the search)
                const FbRec *rec = cubes[c].c.rec;
                uint32_t over[2] = {sc->sel[0].done, sc->sel[1].done};
                if (level > 0)
                    for (int f = 0; f < 2; ++f) {
                        over[f] |= word_load(&rec[f].done);
                        if (level > 1) over[f] |= word_load(&rec[2 + f].done);
                        prefix[f][c] = word_load(&rec[(level - 1) * 2 + f].prefix);
                    }
                if (!idle(sc)) m = (over[0] ? 0u : 1u) | (over[1] ? 0u : 2u);
                if (m) n = cubes[c].c.d.plane;
            }
            const int busy = (int)__popcll(__ballot(n > 0));
            int64_t x = n;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int64_t y = __shfl_up(x, o, 64);
                if (c >= o) x += y;
            }
            if (c < sh.ncubes) {
                seg0[c + 1] = x;
                fmask[c] = m;
            }
            if (c == 0) {
                seg0[0] = 0;
                active = busy;
            }
        }
        __syncthreads();
        const int64_t W = seg0[sh.ncubes];
        if (W == 0) return;
        if (level == 0) W0 = W;
        const int shift = lvl_shift(level), pshift = shift + (level == 0 ? 11 : 10);
        const uint32_t bmask = (uint32_t)lvl_bins(level) - 1u;
        for (int j = (int)blockIdx.x; j < G;) {
            const int64_t lo = W * (int64_t)j / G, hi = W * (int64_t)(j + 1) / G;
            for (int c = 0; mine && c < sh.ncubes; ++c) {
                const int64_t c0 = seg0[c], c1 = seg0[c + 1];
                if (c0 == c1 || !(lo < c1 && hi > c0)) continue;  // the chunk has no part of cube c
                const CubeArgs<DT> &a = cubes[c];
                DevScalars *sc = a.c.sc;
                const uint32_t m = fmask[c];
                const bool act0 = m & 1u, act1 = m & 2u;
                FbRec *rec = a.c.rec;
                const uint32_t pre0 = level ? prefix[0][c] : 0u, pre1 = level ? prefix[1][c] : 0u;
                for (int b = tid; b < 2 * kHistBins; b += kFbThreads) {
                    hc[b / kHistBins][b % kHistBins] = 0u;
                    hm[b / kHistBins][b % kHistBins] = 0ull;
                }
                __syncthreads();
                {
                    const Dims d = a.c.d;
                    const int n1 = d.n1, n2 = d.n2;
                    const int par = (int)(sc->iter & 1u);
                    const Side<DT> src = a.side[par];
                    const float a4 = (float)sc->a4, gt = a.c.zt_step;
                    // z as it was stored, by sweep A (BF16) or by this block at level
                    // 0 (FP32: on the side of the state that the coming sweep writes
                    // whole), or evaluated again. A level over the same cubes has the
                    // same chunks, and each thread reads what it wrote.
                    const uint32_t N = (uint32_t)d.plane;
                    const float *zs = nullptr, *zt = nullptr;
                    float *ws = nullptr, *wt = nullptr;  // to be stored
                    if constexpr (sizeof(DT) == 2) {
                        if (sc->zstore) zs = a.c.zbuf, zt = zs + N;
                    } else if (level == 0) {
                        ws = a.side[par ^ 1].y4, wt = a.side[par ^ 1].t;
                    } else if (W == W0 && (mine0[j >> 5] >> (j & 31) & 1u)) {
                        zs = a.side[par ^ 1].y4, zt = a.side[par ^ 1].t;
                    }
                    const uint32_t q0 = (uint32_t)((lo > c0 ? lo : c0) - c0), q1 = (uint32_t)((hi < c1 ? hi : c1) - c0);
                    auto add = [&](int f, uint32_t pre, float z) {
                        const uint32_t p = abs_bits(z);
                        if (level > 0 && (p >> pshift) != pre) return;
                        const uint32_t b = (p >> shift) & bmask;
                        atomicAdd(&hc[f][b], 1u);
                        atomicAdd(&hm[f][b], (unsigned long long)significand(p));
                    };
                    if (zs) {
                        for (uint32_t q = q0 + (uint32_t)tid; q < q1; q += kFbUnrollZ * kFbThreads) {
                            float z0[kFbUnrollZ], z1[kFbUnrollZ];
#pragma unroll
                            for (int u = 0; u < kFbUnrollZ; ++u) {
                                const uint32_t x = q + (uint32_t)(u * kFbThreads);
                                z0[u] = z1[u] = 0.f;
                                if (x < q1) {
                                    if (act0) z0[u] = zs[x];
                                    if (act1) z1[u] = zt[x];
                                }
                            }
#pragma unroll
                            for (int u = 0; u < kFbUnrollZ; ++u) {
                                if (q + (uint32_t)(u * kFbThreads) >= q1) break;
                                if (act0) add(0, pre0, z0[u]);
                                if (act1) add(1, pre1, z1[u]);
                            }
                        }
                    } else
                    for (uint32_t q = q0 + (uint32_t)tid; q < q1; q += kFbUnroll * kFbThreads) {
                        // every load of kFbUnroll voxels first, then their bins
                        float y4s[kFbUnroll], sv[kFbUnroll], tv[kFbUnroll], y3c[kFbUnroll], y3m[kFbUnroll];
#pragma unroll
                        for (int u = 0; u < kFbUnroll; ++u) {
                            const uint32_t x = q + (uint32_t)(u * kFbThreads);
                            y4s[u] = sv[u] = tv[u] = y3c[u] = y3m[u] = 0.f;
                            if (x < q1) {
                                y4s[u] = ld(src.y4 + x);
                                if (act0) sv[u] = src.s[x];
                                if (act1) {
                                    const int i = (int)((x / (uint32_t)n2) % (uint32_t)n1);
                                    tv[u] = src.t[x];
                                    if (i <= n1 - 2) y3c[u] = ld(src.y3 + x);
                                    if (i >= 1) y3m[u] = ld(src.y3 + x - n2);
                                }
                            }
                        }
#pragma unroll
                        for (int u = 0; u < kFbUnroll; ++u) {
                            const uint32_t x = q + (uint32_t)(u * kFbThreads);
                            if (x >= q1) break;
                            const float y4 = y4_of(y4s[u], a4);
                            if (act0) {
                                const float z = zs_of(sv[u], y4);
                                if (ws) ws[x] = z;
                                add(0, pre0, z);
                            }
                            if (act1) {
                                const float z = zt_of(tv[u], y3m[u], y3c[u], y4, gt);
                                if (wt) wt[x] = z;
                                add(1, pre1, z);
                            }
                        }
                    }
                }
                __syncthreads();
                // The block's histograms go to the global ones with atomics of system
                // scope, performed beyond the XCD's L2 (visible to every XCD without
                // writing back any cache), and returning, so that the wait below
                // covers their completion; all of a thread's atomics go out before
                // their results are used. Then the block counts itself done with
                // the cube; the last one reads the histograms back.
                Hist *hist = a.c.hist;
                uint32_t seen = 0u;
                {
                    constexpr int per = 2 * kHistBins / kFbThreads;
                    uint32_t rc[per];
                    unsigned long long rm[per];
#pragma unroll
                    for (int k = 0; k < per; ++k) {
                        const int b = tid + k * kFbThreads;
                        const int f = b / kHistBins, bb = b % kHistBins;
                        rc[k] = 0u;
                        rm[k] = 0ull;
                        if (hc[f][bb]) {
                            rc[k] = __hip_atomic_fetch_add(&hist[level * 2 + f].count[bb], hc[f][bb], __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_SYSTEM);
                            rm[k] = __hip_atomic_fetch_add((unsigned long long *)&hist[level * 2 + f].msum[bb], hm[f][bb],
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < per; ++k) seen |= rc[k] | (uint32_t)rm[k];
                }
                __builtin_amdgcn_s_waitcnt(0);  // this thread's atomics are done
                __syncthreads();
                uint32_t *counter = slot_flags(cubes, sh.ncubes) + kFbCounterWord + c;
                if (tid == 0) {
                    const int nbk = blocks_meeting(W, G, c0, c1);
                    const uint32_t done = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    last = done == (uint32_t)(nbk - 1) ? 1 : 0;
                }
                __syncthreads();
                // (the returned values are kept alive by a store no launch reaches:
                // a table holds at most kMaxBatch cubes)
                if (sh.ncubes > kMaxBatch && tid == 0) hc[0][0] = seen;
                if (last) {
                    // acquire: drop cached copies so that the reads see every block's atomics
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    const int nb = lvl_bins(level);
                    // both fields' bins, then one wavefront each
                    for (int k = tid; k < 2 * nb; k += kFbThreads) {
                        const int f = k >= nb ? 1 : 0, b = k - f * nb;
                        if (!(m >> f & 1u)) continue;
                        Hist &h = hist[level * 2 + f];
                        // read where the atomics were performed
                        const uint32_t e = lvl_exponent(level, f ? pre1 : pre0, b);
                        const unsigned long long ms = __hip_atomic_load((unsigned long long *)&h.msum[b], __ATOMIC_RELAXED,
                                                                        __HIP_MEMORY_SCOPE_SYSTEM);
                        reinterpret_cast<double *>(hm[f])[bin_at(b)] = (double)ms * bin_scale(e);
                        hc[f][bin_at(b)] = __hip_atomic_load((uint32_t *)&h.count[b], __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_SYSTEM);
                    }
                    __syncthreads();
                    const int f = __builtin_amdgcn_readfirstlane(tid >> 6);
                    if (f < 2 && (m >> f & 1u)) {
                        RadixPick pk = {0.0, 0.0, 0.0, 0.0, 0u, level, 0};
                        FbRec r0 = {}, r1 = {};
                        if (level > 0) {
                            r0 = rec_load(&rec[f]);
                            if (level > 1) r1 = rec_load(&rec[2 + f]);
                            const FbRec &pr = level > 1 ? r1 : r0;
                            pk.s_above = pr.s_above;
                            pk.c_above = pr.c_above;
                            pk.prefix = pr.prefix;
                        }
                        radix_level_wave(reinterpret_cast<double *>(hm[f]), hc[f], sc->sel[f].radius, pk);
                        if ((tid & 63) == 0) {
                            FbRec o;
                            o.tau = pk.tau;
                            o.s_above = pk.s_above;
                            o.c_above = pk.c_above;
                            o.dens = pk.dens;
                            o.prefix = pk.prefix;
                            o.done = pk.done ? 1u : 0u;
                            rec_store(&rec[level * 2 + f], o);
                            // what the sweep of this slot reads of the threshold (no
                            // pass reads it)
                            if (o.done)
                                sc->in.set(f, resolved(sc->sel[f], level ? r0 : o, level > 1 ? r1 : o, o, a.c.d.plane));
                        }
                    }
                    __builtin_amdgcn_s_waitcnt(0);  // the records are out
                    __syncthreads();
                    if (tid == 0) {
                        __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                        __builtin_amdgcn_s_waitcnt(0);
                        (void)__hip_atomic_fetch_add(&flags[kFbReadyWord + level], 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_SYSTEM);
                    }
                }
                __syncthreads();  // the LDS histograms are reused by the next cube
            }
            // the first chunk that nobody has taken
            __syncthreads();
            for (int q = tid; q < G; q += kFbThreads)
                if (word_load(&claims[q]) != run) atomicMin(&next, q);
            __syncthreads();
            j = next;
            __syncthreads();
            if (tid == 0 && j < G) {
                mine = __hip_atomic_exchange(&claims[j], run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != run ? 1 : 0;
                next = G;
                if (level == 0 && mine) mine0[j >> 5] |= 1u << (j & 31);
            }
            __syncthreads();
        }
        // every chunk is taken: wait for the level
        if (tid == 0)
            while (word_load(&flags[kFbReadyWord + level]) < (uint32_t)active) __builtin_amdgcn_s_sleep(1);
    }
}

}  // namespace

// Persistent blocks of a fallback pass: one per compute unit.
int fallback_grid()
{
    static const int cached = [] {
        int dev = 0, cus = 256;
        if (hipGetDevice(&dev) == hipSuccess) {
            hipDeviceProp_t prop;
            if (hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
        }
        return cus < kFbMost ? cus : kFbMost;
    }();
    return cached;
}

hipError_t launch_fallback(const void *table, int dual_bytes, const LaunchShape &sh, hipStream_t st)
{
    uint32_t *flags = slot_flags(table, sh.ncubes);
    if (dual_bytes == 2)
        hipLaunchKernelGGL(k_fb_hist<bf16>, dim3(sh.fb_grid), dim3(kFbThreads), 0, st,
                           (const CubeArgs<bf16> *)table, sh, flags);
    else
        hipLaunchKernelGGL(k_fb_hist<float>, dim3(sh.fb_grid), dim3(kFbThreads), 0, st,
                           (const CubeArgs<float> *)table, sh, flags);
    return hipGetLastError();
}

}  // namespace geo
