// Expert FFN products of small batches (decoding): few rows per expert, so a
// product is a stream of the expert weights from HBM and everything else is
// arranged around keeping that stream in flight.
//
// A workgroup owns 16 TT rows of one expert and 128 weight columns (up/gate:
// 64 gate columns and the 64 up columns of the same f range); its 4 waves take
// every fourth 32-row slice of K, so together they walk K through neighbouring
// memory.  A wave's step is 32 k rows x 128 columns: 8 loads of 16 bytes per
// lane straight into registers (8 consecutive columns of one k row), the next
// step's loads issued before this step's arithmetic.  No two waves need the
// same weights, so LDS would only add a round trip: the 8 x 8 block a lane
// then holds (8 k rows x 8 columns) is transposed in its registers (one
// v_perm_b32 per two elements, under 5 % of the time the bytes take to arrive)
// into the operands of 8 v_mfma_f32_16x16x32_bf16, the weights as the row
// operand: product i takes column 8 r + i in row r.  The activations are the
// column operand, 16 tokens each, from L2.
//
// Where the tiles are too few for the CUs, several workgroups share a tile's K
// (skinny_kslices).
//
// The 4 partial sums are added through LDS in wave order, so results are
// bitwise deterministic; then the SwiGLU, the row scale (dense routing) and
// the stores.  The token of a plan row is perm[p] / k, so no plan-order
// prologue has to run first.  The shared expert's tiles ride in the same launch.
//
// Measured against the 256 x 256 tile GEMMs these calls took before (whole
// step, us): d 4096, 32 experts of 1536, top 8: 16 tokens 370 -> 270 (up/gate
// 243 -> 155, 5.2 TB/s; down 107 -> 70, 5.7 TB/s), 150 tokens 392 -> 304;
// d 7168, 8 experts of 2048 and a shared one, all taken: 61 tokens 996 -> 282;
// d 2048, 128 experts of 768: 1 token 119 -> 57, 512 tokens 380 -> 315.  Tried and
// slower: 64 columns per workgroup (16 tokens, up/gate 155 -> 202: half-line
// segments), 8 waves on contiguous eighths of K (512 tokens, 128 experts: 351).
#include "common.h"
#include "kernels.h"
#include "rules.h"

namespace {

constexpr int SK_NW = 4;              // waves per workgroup, each 1/4 of K
constexpr int SK_COLS = 128;          // weight columns per workgroup, 8 per lane
constexpr int SK_PITCH = SK_COLS + 4; // floats per token row of the reduction buffer

template <int MODE, int TT>
__global__ __launch_bounds__(64 * SK_NW, 2) void skinny_kernel(SkinnyArgs g) {
    constexpr bool UP = MODE == SK_UP || MODE == SK_UP_PART;
    constexpr int NCOL = UP ? SK_COLS / 2 : SK_COLS;   // output columns per workgroup
    __shared__ __attribute__((aligned(16))) float red[SK_NW][16][SK_PITCH];
    constexpr int BM = 16 * TT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g4 = lane >> 4;

    // ---------------- which rows, which columns ----------------
    // with K split over several workgroups, slice `ks` of the tiles' K
    const int ks = MODE == SK_UP_PART ? (int)(blockIdx.x / g.ntiles) : 0;
    const int b = (int)blockIdx.x - ks * g.ntiles;
    const bool sh = b < g.nshared;    // the shared expert's tiles come first
    int e = 0, row0, row_end, ntile;
    if (sh) {
        const int ncol = g.Ns / NCOL;
        row0 = (b / ncol) * BM;
        row_end = g.T;
        ntile = b % ncol;
    } else {
        const int ncol = g.N / NCOL;
        const int slot = (b - g.nshared) / ncol;
        ntile = (b - g.nshared) % ncol;
        // the expert of m-tile slot `slot`: every wave scans the plan's offsets
        int found = -1, within = 0, cum = 0;
        for (int base = 0; base < g.E && found < 0; base += 64) {
            const int ee = base + lane;
            const int cnt = ee < g.E ? g.offsets[ee + 1] - g.offsets[ee] : 0;
            const int tiles = cnt > 0 ? (cnt + BM - 1) / BM : 0;
            int x = tiles;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off, 64);
                if (lane >= off) x += y;
            }
            const int excl = cum + x - tiles;
            const unsigned long long m = __ballot(slot >= excl && slot < excl + tiles);
            if (m) {
                const int src = __builtin_ctzll(m);
                found = base + src;
                within = slot - __shfl(excl, src, 64);
            }
            cum += __shfl(x, 63, 64);
        }
        found = __builtin_amdgcn_readfirstlane(found);
        if (found < 0) return;
        e = found;
        row0 = g.offsets[e] + __builtin_amdgcn_readfirstlane(within) * BM;
        row_end = g.offsets[e + 1];
    }
    const int K = sh ? g.Ks : g.K;
    const long ldb = sh ? g.ldb_s : g.ldb;
    const uint16_t *A = sh ? g.As : g.A;
    const long lda = sh ? g.lda_s : g.lda;
    const int n0 = ntile * NCOL;

    // ---------------- operand pointers of this lane ----------------
    // K in 256-row units over the slices
    const int k0 = MODE == SK_UP_PART ? K / 256 * ks / g.kslices * 256 : 0;
    const int k1 = MODE == SK_UP_PART ? K / 256 * (ks + 1) / g.kslices * 256 : K;
    const int kw = k0 + 32 * wave + 8 * g4;           // its first k
    const uint16_t *wp;
    if constexpr (UP) {
        const uint16_t *m = r < 8 ? (sh ? g.Bs : g.B) : (sh ? g.Bs2 : g.B2);
        wp = m + (long)e * g.b_estride + (long)kw * ldb + n0 + 8 * (r & 7);
    } else {
        wp = (sh ? g.Bs : g.B) + (long)e * g.b_estride + (long)kw * ldb + n0 + 8 * r;
    }
    uint32_t xo[TT];   // element offsets (a small batch's rows span under 2^32)
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        // rows past the region's end load its last row; they are never stored
        const int p = min(row0 + 16 * t + r, row_end - 1);
        int row = p;
        if (UP && !sh) {
            const int j = g.perm[min(max(p, 0), g.R - 1)];
            row = (j >= 0 && j < g.R) ? j / g.k : 0;
        }
        row = min(max(row, 0), (sh ? g.T : g.a_nrows) - 1);
        xo[t] = (uint32_t)row * (uint32_t)lda + (uint32_t)kw;
    }

    f32x4_t acc[TT][8];
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[t][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    int xk = 0;
    // Weights and activations are requested one step ahead, the activations
    // first: loads return in order, so waiting for a step's operands leaves
    // the next step's weights in flight.
    auto load = [&](u32x4_t (&w)[8], u32x4_t (&x)[TT]) {
#pragma unroll
        for (int t = 0; t < TT; ++t) x[t] = ld_u32x4(A + (xo[t] + (uint32_t)xk));
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = ld_u32x4(wp + j * ldb);
        xk += 32 * SK_NW;
        wp += 32 * SK_NW * ldb;
    };
    auto mul = [&](const u32x4_t (&w)[8], const u32x4_t (&x)[TT]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            u32x4_t a;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                a[q] = __builtin_amdgcn_perm(w[2 * q + 1][i >> 1], w[2 * q][i >> 1],
                                             (i & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int t = 0; t < TT; ++t)
                acc[t][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, x[t]), acc[t][i],
                    0, 0, 0);
            if (TT > 2) __builtin_amdgcn_sched_barrier(0);   // one column set's operand at a time
        }
    };

    const int steps = (k1 - k0) / (32 * SK_NW);   // even: a multiple of 256 rows
    u32x4_t w[2][8], x[2][TT];
    load(w[0], x[0]);
    for (int s = 0; s < steps; s += 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (i == 0 || s + 2 < steps) load(w[i ^ 1], x[i ^ 1]);
            __builtin_amdgcn_sched_barrier(0);
            mul(w[i], x[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---------------- sum over the waves, epilogue ----------------
    // accumulator layout: lane (g4, r), register q holds weight column row
    // 4 g4 + q of product i, i.e. column 8 (4 g4 + q) + i, for token r
    const int en = 4 * (tid & 31);        // columns this thread finishes, of two tokens
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        if (t > 0) {
            if (row0 + 16 * t >= row_end) break;      // uniform: no rows left
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<f32x4_t *>(&red[wave][r][8 * (4 * g4 + q) + 4 * h]) =
                    f32x4_t{acc[t][4 * h][q], acc[t][4 * h + 1][q], acc[t][4 * h + 2][q],
                            acc[t][4 * h + 3][q]};
        __syncthreads();
#pragma unroll
        for (int eh = 0; eh < 2; ++eh) {
            const int et = (tid >> 5) + 8 * eh;
            f32x4_t v = *reinterpret_cast<const f32x4_t *>(&red[0][et][en]);
#pragma unroll
            for (int w = 1; w < SK_NW; ++w) {
                const f32x4_t u = *reinterpret_cast<const f32x4_t *>(&red[w][et][en]);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = v[q] + u[q];
            }
            const int p = row0 + 16 * t + et;
            if constexpr (MODE == SK_UP_PART) {
                // gate columns in the first half of a partial row, up in the second
                const long f = sh ? g.ldc_s : g.ldc, rows = sh ? g.T : g.R;
                if (p < row_end)
                    *reinterpret_cast<f32x4_t *>((sh ? g.Cfs : g.Cf) + ((long)ks * rows + p) * 2 * f + n0
                                                 + (en < NCOL ? en : f + en - NCOL)) = v;
            } else if constexpr (UP) {
                // the first half of a token's threads hold the gate, the second
                // the up projection of the same f columns
                f32x4_t u;
#pragma unroll
                for (int q = 0; q < 4; ++q) u[q] = shfl_xor_f(v[q], 16);
                if (p < row_end && en < NCOL) {
                    const long o = (long)p * (sh ? g.ldc_s : g.ldc) + n0 + en;
                    float ws = 1.0f;
                    if (g.row_w && !sh) {
                        const int j = g.perm[p];
                        ws = (j >= 0 && j < g.R) ? g.row_w[j] : 0.f;
                    }
                    float h[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) h[q] = ws * (silu_f(v[q]) * u[q]);
                    *reinterpret_cast<u32x2_t *>((sh ? g.Cs : g.C) + o) =
                        u32x2_t{pack_bf2(h[0], h[1]), pack_bf2(h[2], h[3])};
                }
            } else if (p < row_end) {
                const long o = (long)p * (sh ? g.ldc_s : g.ldc) + n0 + en;
                if constexpr (MODE == SK_DOWN_PART)
                    *reinterpret_cast<f32x4_t *>((sh ? g.Cfs : g.Cf) + o) = v;
                else
                    *reinterpret_cast<u32x2_t *>((sh ? g.Cs : g.C) + o) =
                        u32x2_t{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
            }
        }
    }
}

// The K slices of a split up/gate product added in slice order, then the
// SwiGLU: H for the plan's rows (blocks below `rblocks`) and the shared
// expert's.  Four columns of one row per thread.
__global__ __launch_bounds__(256) void skinny_act_kernel(SkinnyArgs g, long rblocks) {
    const bool sh = blockIdx.x >= rblocks;
    const long f = sh ? g.ldc_s : g.ldc, rows = sh ? g.T : g.R;
    const long i = 4 * (((long)blockIdx.x - (sh ? rblocks : 0)) * 256 + threadIdx.x);
    const long p = i / f, c = i % f;
    if (p >= (sh ? rows : (long)g.offsets[g.E])) return;
    const float *src = (sh ? g.Cfs : g.Cf) + p * 2 * f + c;
    f32x4_t a = f32x4_t{0.f, 0.f, 0.f, 0.f}, b = a;
    for (int s = 0; s < g.kslices; ++s) {
        const f32x4_t u = *reinterpret_cast<const f32x4_t *>(src + s * rows * 2 * f);
        const f32x4_t v = *reinterpret_cast<const f32x4_t *>(src + s * rows * 2 * f + f);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = a[q] + u[q];
            b[q] = b[q] + v[q];
        }
    }
    float ws = 1.0f;
    if (g.row_w && !sh) {
        const int j = g.perm[p];
        ws = (j >= 0 && j < g.R) ? g.row_w[j] : 0.f;
    }
    float h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = ws * (silu_f(a[q]) * b[q]);
    *reinterpret_cast<u32x2_t *>((sh ? g.Cs : g.C) + i) = u32x2_t{pack_bf2(h[0], h[1]), pack_bf2(h[2], h[3])};
}

// Dense routing: Y[t] = sum over the experts' fp32 down products in ascending
// id, then the shared expert's, rounded once.  Four columns per thread.
__global__ __launch_bounds__(256) void dense_sum_kernel(const float *__restrict__ part,
                                                        const float *__restrict__ part_s,
                                                        const int *__restrict__ offsets, int E, int T,
                                                        int R, int d, uint16_t *__restrict__ Y) {
    const int t = blockIdx.y, c = 4 * (blockIdx.x * 256 + threadIdx.x);
    if (c >= d) return;
    f32x4_t v = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int e0 = 0; e0 < E; e0 += 8) {
        f32x4_t u[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // an offset that a malformed plan would push past the buffer is clamped into it
            const int off = min(max(offsets[min(e0 + i, E - 1)], 0), R - T);
            u[i] = *reinterpret_cast<const f32x4_t *>(part + (long)(off + t) * d + c);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (e0 + i < E)
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = v[q] + u[i][q];
    }
    if (part_s) {
        const f32x4_t u = *reinterpret_cast<const f32x4_t *>(part_s + (long)t * d + c);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = v[q] + u[q];
    }
    *reinterpret_cast<u32x2_t *>(Y + (long)t * d + c) = u32x2_t{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
}

template <int MODE>
hipError_t launch_mode(SkinnyArgs g, int tt, hipStream_t st) {
    const int ncols = MODE == SK_UP || MODE == SK_UP_PART ? SK_COLS / 2 : SK_COLS, bm = 16 * tt;
    const long slots = skinny_slots(g.R, g.E, bm);
    g.nshared = g.Ns > 0 ? (g.T + bm - 1) / bm * (g.Ns / ncols) : 0;
    g.ntiles = (int)(g.nshared + slots * (g.N / ncols));
    const long grid = (long)g.ntiles * (MODE == SK_UP_PART ? g.kslices : 1);
    if (grid <= 0) return hipSuccess;
    const dim3 gr((unsigned)grid), bl(64 * SK_NW);
    if (tt == 1) skinny_kernel<MODE, 1><<<gr, bl, 0, st>>>(g);
    else skinny_kernel<MODE, 4><<<gr, bl, 0, st>>>(g);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_skinny_up(const SkinnyArgs &g, int tt, hipStream_t st) {
    if (g.kslices <= 1) return launch_mode<SK_UP>(g, tt, st);
    const hipError_t e = launch_mode<SK_UP_PART>(g, tt, st);
    if (e != hipSuccess) return e;
    const long rb = ((long)g.R * g.ldc / 4 + 255) / 256;
    const long sb = g.Ns > 0 ? ((long)g.T * g.ldc_s / 4 + 255) / 256 : 0;
    skinny_act_kernel<<<dim3((unsigned)(rb + sb)), dim3(256), 0, st>>>(g, rb);
    return hipGetLastError();
}
hipError_t launch_skinny_down(const SkinnyArgs &g, int tt, hipStream_t st) {
    return g.Cf ? launch_mode<SK_DOWN_PART>(g, tt, st) : launch_mode<SK_DOWN>(g, tt, st);
}
hipError_t launch_dense_sum(const float *part, const float *part_s, const int *offsets, int E, int T,
                            int R, int d, uint16_t *Y, hipStream_t st) {
    dense_sum_kernel<<<dim3((d / 4 + 255) / 256, T), dim3(256), 0, st>>>(part, part_s, offsets, E, T, R, d, Y);
    return hipGetLastError();
}
