// Dispatch plan: Algorithm 1 of §3.1 with a single source rank, built on the
// device with no host readback.  With one rank the position of route j in
// expert e's region is the number of earlier routes to e, so the plan is a
// stable counting sort of the routes by expert:
//
//   1. plan_hist:    per-chunk expert histograms (LDS integer counters),
//                    stored expert-major ([E][chunks]) so that the scan's
//                    lanes, one chunk each, read and write consecutive words;
//   2. plan_scan:    exclusive scans over chunks (per expert) and experts;
//   3. plan_scatter: each chunk walks its routes in order in 64-lane groups;
//                    lanes with equal expert ids are matched with ballots, so
//                    ranks come from popcounts, never from position atomics.
//
// Up to 2^20 routes the same sort runs in one launch or two (plan_place_kernel).
//
// Every step is integer-exact and independent of scheduling.
#include "common.h"
#include "kernels.h"

namespace {

constexpr int MAXE = 256;
// Routes of the one-launch plan: a wave then walks up to 8 groups of 64 in
// turn.  128 experts, us: 4000 routes 7.8 in one launch against 10.1 in two,
// 8000 the same 9.8 and 10.2, 16000 18 against 10.2.
constexpr int PLAN_ONE_MAX = 8192;
// Routes of the two-launch plan: 256 blocks, whose histograms each block can
// still sum itself.
constexpr int PLAN_MAX = 256 * 4096;

__global__ __launch_bounds__(64) void plan_hist_kernel(const int *__restrict__ idx, int R, int E,
                                                       int *__restrict__ blockcounts,
                                                       int *__restrict__ blockflags) {
    __shared__ int cnt[MAXE];
    const int b = blockIdx.x, l = threadIdx.x;
    for (int e = l; e < E; e += 64) cnt[e] = 0;
    __syncthreads();
    const int j0 = b * PLAN_CHUNK;
    const int j1 = min(R, j0 + PLAN_CHUNK);
    // all of the lane's ids first (their loads overlap), then the counts
    constexpr int PER = PLAN_CHUNK / 64;
    int ev[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = j0 + l + 64 * q;
        ev[q] = j < j1 ? idx[j] : 0;
    }
    int bad = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (j0 + l + 64 * q >= j1) break;
        const int e = ev[q];
        if (e >= 0 && e < E) atomicAdd(&cnt[e], 1);
        else bad = 1;
    }
    __syncthreads();
    for (int e = l; e < E; e += 64) blockcounts[(long)e * gridDim.x + b] = cnt[e];
    const unsigned long long anybad = __ballot(bad);
    if (l == 0) blockflags[b] = anybad != 0ull;
}

DEV int wave_incl_scan(int v, int l) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(v, off, 64);
        if (l >= off) v += y;
    }
    return v;
}

__global__ __launch_bounds__(1024) void plan_scan_kernel(int nb, int E,
                                                         const int *__restrict__ blockcounts,
                                                         int *__restrict__ blockbase,
                                                         int *__restrict__ counts,
                                                         int *__restrict__ offsets,
                                                         const int *__restrict__ blockflags,
                                                         int *__restrict__ err) {
    __shared__ int tot[MAXE];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    for (int e = w; e < E; e += 16) {
        int run = 0;
        for (int base = 0; base < nb; base += 64) {
            const int b = base + l;
            const int v = b < nb ? blockcounts[(long)e * nb + b] : 0;
            const int x = wave_incl_scan(v, l);
            if (b < nb) blockbase[(long)e * nb + b] = run + x - v;
            run += __shfl(x, 63, 64);
        }
        if (l == 0) tot[e] = run;
    }
    __syncthreads();
    if (w == 0) {
        int run = 0;
        for (int base = 0; base < E; base += 64) {
            const int e = base + l;
            const int v = e < E ? tot[e] : 0;
            const int x = wave_incl_scan(v, l);
            if (e < E) {
                offsets[e] = run + x - v;
                counts[e] = v;
            }
            run += __shfl(x, 63, 64);
        }
        if (l == 0) offsets[E] = run;
    } else if (w == 1) {
        int f = 0;
        for (int b = l; b < nb; b += 64) f |= blockflags[b];
        const unsigned long long any = __ballot(f != 0);
        if (l == 0) err[0] = any != 0ull;
    }
}

__global__ __launch_bounds__(64) void plan_scatter_kernel(const int *__restrict__ idx, int R, int E,
                                                          int ebits,
                                                          const int *__restrict__ blockbase,
                                                          const int *__restrict__ offsets,
                                                          int *__restrict__ perm,
                                                          int *__restrict__ route_pos) {
    __shared__ int run[MAXE];
    const int b = blockIdx.x, l = threadIdx.x;
    for (int e = l; e < E; e += 64) run[e] = offsets[e] + blockbase[(long)e * gridDim.x + b];
    __syncthreads();
    const int j0 = b * PLAN_CHUNK;
    const int j1 = min(R, j0 + PLAN_CHUNK);
    const unsigned long long lt = (l == 0) ? 0ull : (~0ull >> (64 - l));
    // all of the lane's ids first (their loads overlap), then the ranks
    constexpr int PER = PLAN_CHUNK / 64;
    int ev[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = j0 + l + 64 * q;
        ev[q] = j < j1 ? idx[j] : -1;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int base = j0 + 64 * q;
        if (base >= j1) break;
        const int j = base + l;
        const bool valid = j < j1;
        const int e = valid ? ev[q] : -1;
        const bool ok = valid && e >= 0 && e < E;
        unsigned long long m = __ballot(ok);
        for (int bit = 0; bit < ebits; ++bit) {
            const bool on = ok && ((e >> bit) & 1);
            const unsigned long long bb = __ballot(on);
            m &= on ? bb : ~bb;
        }
        if (!ok) m = 0ull;
        const int rank = __popcll(m & lt);
        const int grp = __popcll(m);
        const int pos = ok ? run[e] + rank : -1;
        __syncthreads();
        if (ok && rank == grp - 1) run[e] += grp;
        __syncthreads();
        if (valid) route_pos[j] = (ok && pos < R) ? pos : -1;
        if (ok && pos >= 0 && pos < R) perm[pos] = j;
    }
}

// Up to PLAN_MAX routes the plan takes one launch (a single block) or two.
// Its work is small next to the latencies of the launches and of a wave
// walking its routes group by group, so a block has 16 waves of up to NG
// groups of 64 consecutive routes each, per-wave expert counters in LDS take
// the place of the chunk histograms, and with several blocks (MULTI) each one
// sums the other blocks' histograms itself instead of waiting for a scan
// launch.  Ranks come from ballots as in plan_scatter_kernel: the plan is the
// same, integer for integer.  Measured (calls back to back, us): 8 routes 15 ->
// 7.6 (the host's time for one launch), 16384 tokens to 32 experts 22 -> 10, 8192
// tokens to 128 experts 30 of kernel time -> 10.
constexpr int PLAN_BLOCK = 4096;          // routes per block of the two-launch form

__global__ __launch_bounds__(1024) void plan_count_kernel(const int *__restrict__ idx, int R, int E,
                                                          int *__restrict__ blockcounts,
                                                          int *__restrict__ blockflags) {
    __shared__ int cnt[MAXE];
    __shared__ int anybad;
    const int b = blockIdx.x, tid = threadIdx.x;
    constexpr int PER = PLAN_BLOCK / 1024;
    int ev[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = b * PLAN_BLOCK + tid + 1024 * q;
        ev[q] = j < R ? idx[j] : 0;
    }
    if (tid < MAXE) cnt[tid] = 0;
    if (tid == 0) anybad = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (b * PLAN_BLOCK + tid + 1024 * q >= R) break;
        if (ev[q] >= 0 && ev[q] < E) atomicAdd(&cnt[ev[q]], 1);
        else anybad = 1;
    }
    __syncthreads();
    if (tid < E) blockcounts[(long)b * E + tid] = cnt[tid];
    if (tid == 0) blockflags[b] = anybad;
}

template <int NG, bool MULTI>
__global__ __launch_bounds__(1024) void plan_place_kernel(const int *__restrict__ idx, int R, int E,
                                                          int ebits,
                                                          const int *__restrict__ blockcounts,
                                                          const int *__restrict__ blockflags,
                                                          int *__restrict__ counts,
                                                          int *__restrict__ offsets,
                                                          int *__restrict__ perm,
                                                          int *__restrict__ route_pos,
                                                          int *__restrict__ err) {
    __shared__ int cnt[16][MAXE];            // routes of wave w to expert e, then its running position
    __shared__ int before[4][MAXE], all[4][MAXE];   // other blocks' routes to e: in earlier blocks, in all
    __shared__ int tot[MAXE], offs[MAXE];
    __shared__ int anybad;
    const int b = blockIdx.x, w = threadIdx.x >> 6, l = threadIdx.x & 63;
    for (int i = threadIdx.x; i < 16 * MAXE; i += 1024) cnt[i / MAXE][i % MAXE] = 0;
    if (threadIdx.x == 0) anybad = 0;
    const int r0 = MULTI ? b * PLAN_BLOCK : 0, r1 = MULTI ? min(R, r0 + PLAN_BLOCK) : R;
    const int per = MULTI ? NG : (R + 1023) / 1024;    // groups per wave, <= NG
    const int j0 = r0 + w * per * 64, j1 = min(r1, j0 + per * 64);
    int ev[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int j = j0 + l + 64 * q;
        ev[q] = (q < per && j < j1) ? idx[j] : 0;
    }
    int flag = 0;
    if constexpr (MULTI) {
        // a quarter of the blocks' histograms per 256 threads
        const int nb = gridDim.x, e = threadIdx.x & 255, h = threadIdx.x >> 8;
        const int b0 = nb * h / 4, b1 = nb * (h + 1) / 4;
        int pre = 0, sum = 0;
        for (int c0 = b0; c0 < b1; c0 += 8) {
            int v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = (e < E && c0 + u < b1) ? blockcounts[(long)(c0 + u) * E + e] : 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                sum += v[u];
                if (c0 + u < b) pre += v[u];
            }
        }
        before[h][e] = pre;
        all[h][e] = sum;
        if (b == 0 && threadIdx.x < nb) flag = blockflags[threadIdx.x];
    }
    __syncthreads();
    int bad = flag;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        if (q >= per || j0 + l + 64 * q >= j1) break;
        if (ev[q] >= 0 && ev[q] < E) atomicAdd(&cnt[w][ev[q]], 1);
        else bad = 1;
    }
    if (bad) anybad = 1;
    __syncthreads();
    // exclusive scan over the waves per expert, then over the experts
    if (threadIdx.x < MAXE) {
        const int e = threadIdx.x;
        int c[16], run = MULTI ? before[0][e] + before[1][e] + before[2][e] + before[3][e] : 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) c[v] = cnt[v][e];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            cnt[v][e] = run;
            run += c[v];
        }
        tot[e] = MULTI ? all[0][e] + all[1][e] + all[2][e] + all[3][e] : run;
    }
    __syncthreads();
    if (w == 0) {
        int run = 0;
        for (int base = 0; base < E; base += 64) {
            const int e = base + l;
            const int v = e < E ? tot[e] : 0;
            const int x = wave_incl_scan(v, l);
            if (e < E) {
                offs[e] = run + x - v;
                if (b == 0) {
                    offsets[e] = run + x - v;
                    counts[e] = v;
                }
            }
            run += __shfl(x, 63, 64);
        }
        if (l == 0 && b == 0) {
            offsets[E] = run;
            err[0] = anybad;
        }
    }
    __syncthreads();
    const unsigned long long lt = (l == 0) ? 0ull : (~0ull >> (64 - l));
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int base = j0 + 64 * q;
        if (q >= per || base >= j1) break;
        const int j = base + l;
        const bool valid = j < j1;
        const int e = valid ? ev[q] : -1;
        const bool ok = valid && e >= 0 && e < E;
        unsigned long long m = __ballot(ok);
        for (int bit = 0; bit < ebits; ++bit) {
            const bool on = ok && ((e >> bit) & 1);
            const unsigned long long bb = __ballot(on);
            m &= on ? bb : ~bb;
        }
        if (!ok) m = 0ull;
        const int rank = __popcll(m & lt);
        const int grp = __popcll(m);
        // cnt[w] is this wave's own, and a wave's LDS accesses run in order
        const int at = ok ? cnt[w][e] : 0;
        const int pos = ok ? offs[e] + at + rank : -1;
        asm volatile("" ::: "memory");
        if (ok && rank == grp - 1) cnt[w][e] = at + grp;
        asm volatile("" ::: "memory");
        if (valid) route_pos[j] = (ok && pos < R) ? pos : -1;
        if (ok && pos >= 0 && pos < R) perm[pos] = j;
    }
}

}  // namespace

int plan_nblocks(long R) { return (int)((R + PLAN_CHUNK - 1) / PLAN_CHUNK); }

hipError_t launch_plan(const int *topk_idx, int R, int E, int *counts, int *offsets, int *perm,
                       int *route_pos, int *blockcounts, int *blockbase, int *blockflags,
                       int *err, hipStream_t st) {
    const int nb = plan_nblocks(R);
    int ebits = 0;
    while ((1 << ebits) < E) ++ebits;
    if (R > 0 && R <= PLAN_MAX) {
#define PLAN_PLACE(NG, MULTI, BLOCKS)                                                              \
    plan_place_kernel<NG, MULTI><<<dim3(BLOCKS), dim3(1024), 0, st>>>(                             \
        topk_idx, R, E, ebits, blockcounts, blockflags, counts, offsets, perm, route_pos, err)
        if (R <= 2048) {
            PLAN_PLACE(2, false, 1);
        } else if (R <= PLAN_ONE_MAX) {
            PLAN_PLACE(PLAN_ONE_MAX / 1024, false, 1);
        } else {
            // at most 256 blocks, a quarter as many as the scratch's chunks
            const unsigned blocks = (unsigned)((R + PLAN_BLOCK - 1) / PLAN_BLOCK);
            plan_count_kernel<<<dim3(blocks), dim3(1024), 0, st>>>(topk_idx, R, E, blockcounts, blockflags);
            PLAN_PLACE(PLAN_BLOCK / 1024, true, blocks);
        }
#undef PLAN_PLACE
        return hipGetLastError();
    }
    if (nb > 0)
        plan_hist_kernel<<<dim3(nb), dim3(64), 0, st>>>(topk_idx, R, E, blockcounts, blockflags);
    plan_scan_kernel<<<dim3(1), dim3(1024), 0, st>>>(nb, E, blockcounts, blockbase, counts, offsets,
                                                      blockflags, err);
    if (nb > 0)
        plan_scatter_kernel<<<dim3(nb), dim3(64), 0, st>>>(topk_idx, R, E, ebits, blockbase, offsets,
                                                            perm, route_pos);
    return hipGetLastError();
}
