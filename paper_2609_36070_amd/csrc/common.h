// Shared device helpers for the gfx950 MoE kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

#define DEV __device__ __forceinline__

// bf16 bits -> fp32 (exact)
DEV float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
DEV float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
DEV float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// fp32 -> bf16 bits, round to nearest even (gfx950 converts natively).
DEV uint16_t f2bf(float x) {
    __bf16 b = (__bf16)x;
    return __builtin_bit_cast(uint16_t, b);
}
// Two at once: one v_cvt_pk_bf16_f32 with both sources (the scalar
// conversions above take one each, plus a shift and an OR to combine them).
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
DEV uint32_t pack_bf2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

// The gated activation's logistic function from the hardware base-2
// exponential and reciprocal (v_exp_f32, v_rcp_f32, each within about 1 ulp,
// plus the rounding of -a log2(e)): a handful of instructions where expf and
// an IEEE division take about twenty, which matters in the SwiGLU epilogues,
// whose per-element arithmetic is a large part of their time.  Limits:
// a -> +inf gives 1, a -> -inf gives 0, NaN stays NaN.
DEV float sigmoid_f(float a) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-a * 1.4426950408889634f));
}
DEV float silu_f(float a) { return a * sigmoid_f(a); }

typedef float f32x8 __attribute__((ext_vector_type(8)));

DEV int wave_lane() { return threadIdx.x & 63; }

// 32-bit wave shuffles
DEV float shfl_xor_f(float v, int m) { return __shfl_xor(v, m, 64); }
DEV int shfl_xor_i(int v, int m) { return __shfl_xor(v, m, 64); }

DEV u32x4_t ld_u32x4(const void *p) { return *reinterpret_cast<const u32x4_t *>(p); }
DEV void st_u32x4(void *p, u32x4_t v) { *reinterpret_cast<u32x4_t *>(p) = v; }
DEV u32x2_t ld_u32x2(const void *p) { return *reinterpret_cast<const u32x2_t *>(p); }
// 8 consecutive floats (two 16-byte accesses)
DEV f32x8 ld_f32x8(const float *p) {
    const f32x4_t lo = *reinterpret_cast<const f32x4_t *>(p);
    const f32x4_t hi = *reinterpret_cast<const f32x4_t *>(p + 4);
    return f32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}
DEV void st_f32x8(float *p, const f32x8 &v) {
    *reinterpret_cast<f32x4_t *>(p) = f32x4_t{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4_t *>(p + 4) = f32x4_t{v[4], v[5], v[6], v[7]};
}

// 8 floats -> 8 bf16 (round to nearest even) packed in 16 bytes
DEV u32x4_t pack_bf8(const f32x8 &v) {
    return u32x4_t{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]),
                   pack_bf2(v[6], v[7])};
}

// XCD-aware rasters.  Workgroups are dealt to the 8 XCDs round-robin
// (workgroup b runs on XCD b % 8).  The N tiles of a launch are numbered so
// that neighbours share operand panels, and the numbering is cut into chunks
// of CH tiles, chunk c to XCD c % 8: a chunk shares its panels in that XCD's
// L2, and at any time the 8 XCDs work on 8 neighbouring chunks, which read
// the same expert's weights, so those reads hit in the Infinity Cache (3-7 %
// faster than giving each XCD one contiguous run of tiles).  What is left
// after the whole rounds of 8 chunks is dealt evenly, so no XCD runs more
// tiles than ceil(N / (8 CH)) CH, and with CH = 32 no CU more than
// ceil(N / 256).  -1: workgroup b has no tile.
DEV int deal_tile(int b, int N, int CH) {
    const int x = b % 8, j = b / 8, rounds = N / (8 * CH);
    if (j < rounds * CH) return (j / CH * 8 + x) * CH + j % CH;
    const int rest = N - rounds * 8 * CH, each = (rest + 7) / 8;
    const int i = j - rounds * CH, t = x * each + i;
    return i < each && t < rest ? rounds * 8 * CH + t : -1;
}
inline long deal_grid(long N, int CH) { return (N + 8 * CH - 1) / (8 * CH) * (8 * CH); }

// The same with chunks of 32 and a short last round (at most SPLIT_MAX tiles
// beyond a multiple of 256, one per CU) dealt as quarters of its tiles, 0..3 in
// `quarter` (else -1), neighbours to one XCD: a quarter takes about 0.4 of a
// tile's time, so the round ends that much earlier.  Whole calls without ->
// with (us): 1000 tokens, 32 experts 451 -> 434; 4099 tokens, dense + shared
// 2947 -> 2828; 4001-token training step 4167 -> 4099.  Up to 128 tiles (two
// quarters per CU) measured the same.
constexpr int SPLIT_MAX = 64;
DEV int deal_tile_split(int b, int N, int &quarter) {
    const int rest = N % 256, full = N - rest;
    quarter = -1;
    if (rest == 0 || rest > SPLIT_MAX) return deal_tile(b, N, 32);
    if (b < full) return deal_tile(b, full, 32);
    const int s = b - full, each = (4 * rest + 7) / 8, u = (s % 8) * each + s / 8;
    if (s / 8 >= each || u >= 4 * rest) return -1;
    quarter = u & 3;
    return full + u / 4;
}

// Row products: groups of RASTER_GM m-tiles x all n-tiles, walked m-tile
// fastest, in chunks of 32 tiles, what an XCD runs at once: 4 A panels and
// ~8 B panels in its L2.  Dealing whole groups instead left the XCDs uneven
// when there are few: 41 m-tiles x 12 n-tiles are 11 groups, so two XCDs ran
// three rounds while five ran one and a half and the CUs were busy 58 % of
// the launch.  Whole forward, groups -> chunks (us): 4099 tokens to 8 experts
// and a shared one 4027 -> 3062 (the shared and the folded down product are
// 17 m-tiles: 5 groups on 8 XCDs).
constexpr int RASTER_GM = 4, RASTER_CHUNK = 32;

// Place of tile `within` of group `group`.
DEV bool map_group_tile(int group, int within, int tiles_m, int ntn, int &mt, int &nt) {
    const int first = group * RASTER_GM;
    if (first >= tiles_m) return false;
    const int gm = min(RASTER_GM, tiles_m - first);
    if (within >= gm * ntn) return false;
    mt = first + within % gm;
    nt = within / gm;
    return true;
}

DEV bool map_tile(int b, int tiles_m, int ntn, int &mt, int &nt) {
    const int t = deal_tile(b, tiles_m * ntn, RASTER_CHUNK);
    const int tpg = RASTER_GM * ntn;
    return t >= 0 && map_group_tile(t / tpg, t % tpg, tiles_m, ntn, mt, nt);
}

// Workgroups of a launch whose tiles map_tile places (tiles_m or fewer
// m-tiles), whole or with the last round split.
inline long raster_grid(long tiles_m, int ntn) { return deal_grid(tiles_m * ntn, RASTER_CHUNK); }
static_assert(4 * SPLIT_MAX <= 256 && 8 * RASTER_CHUNK == 256, "the quarters fit the round's own slots");

// The fused forward's raster: whole groups dealt to the XCDs, group g to XCD
// g % 8, so that a tile and the tiles that wait for it can share an XCD.
DEV bool map_tile_groups(int b, int tiles_m, int ntn, int &mt, int &nt) {
    const int x = b % 8, j = b / 8;
    const int tpg = RASTER_GM * ntn;
    return map_group_tile((j / tpg) * 8 + x, j % tpg, tiles_m, ntn, mt, nt);
}
inline long raster_grid_groups(long tiles_m, int ntn) {
    const long groups = (tiles_m + RASTER_GM - 1) / RASTER_GM;
    return 8 * ((groups + 7) / 8) * RASTER_GM * ntn;
}

// Weight gradients: each expert's ntm x ntn tiles in column strips of 4
// n-tiles (the last strip of what is left), walked n fastest, all experts in
// one numbering, in chunks of 16 tiles: a 4 x 4 block sharing 4 A and 4 B
// panels, or 8 x 2 in a strip of two.  A tile costs its expert's route count,
// so an expert's chunks go to different XCDs.  (Numbering 4 x 4 blocks with
// room for missing tiles gave some XCDs only partial blocks: at 16 x 6 tiles
// per expert four XCDs ran 16 rounds and four ran 8.)
constexpr int WG_STRIP = 4, WG_CHUNK = 16;
DEV bool map_tile_wgrad(int b, int groups, int ntm, int ntn, int &cm, int &nt) {
    const int per = ntm * ntn;
    const int t = deal_tile(b, groups * per, WG_CHUNK);
    if (t < 0) return false;
    const int e = t / per, i = t % per;
    const int whole = ntn / WG_STRIP * WG_STRIP;       // n-tiles in strips of 4
    const int strip = i < whole * ntm ? i / (WG_STRIP * ntm) : whole / WG_STRIP;
    const int wid = i < whole * ntm ? WG_STRIP : ntn - whole;
    const int w = i - strip * WG_STRIP * ntm;
    cm = e * ntm + w / wid;
    nt = strip * WG_STRIP + w % wid;
    return true;
}

// Workgroups of a launch whose tiles map_tile_wgrad places.
inline long wgrad_grid(long groups, int ntm, int ntn) { return deal_grid(groups * ntm * ntn, WG_CHUNK); }

// The BM-row m-tiles of E <= 256 experts with plan rows offsets[e] ..
// offsets[e + 1], numbered expert by expert.  Every wave scans the tile counts
// for itself (no LDS, no barrier): lane l holds experts l, 64 + l, ...
template <int BM>
struct ExpertTiles {
    int tiles[4], first[4], total;
    DEV void scan(const int *__restrict__ offsets, int E, int lane) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ee = 64 * q + lane;
            const int cnt = ee < E ? offsets[ee + 1] - offsets[ee] : 0;
            tiles[q] = cnt > 0 ? (cnt + BM - 1) / BM : 0;
        }
        int cum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            first[q] = cum;
            if (64 * q >= E) continue;
            int x = tiles[q];
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off, 64);
                if (lane >= off) x += y;
            }
            first[q] = cum + x - tiles[q];
            cum += __shfl(x, 63, 64);
        }
        total = __builtin_amdgcn_readfirstlane(cum);
    }
    // expert of tile number mt < total, and the tile's number in it
    DEV int find(int mt, int &within) const {
        int e = 0;
        within = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned long long m = __ballot(mt >= first[q] && mt < first[q] + tiles[q]);
            if (m) {
                e = 64 * q + __builtin_ctzll(m);
                within = mt - __shfl(first[q], __builtin_ctzll(m), 64);
            }
        }
        within = __builtin_amdgcn_readfirstlane(within);
        return __builtin_amdgcn_readfirstlane(e);
    }
};

// The tile of workgroup b of a grouped row product with ntn n-tiles: the
// raster deals the tiles there are, not the launch's upper bound.
template <int BM>
DEV bool place_tile(const int *__restrict__ offsets, int E, int b, int ntn, int lane, int &e,
                    int &within, int &nt) {
    ExpertTiles<BM> x;
    x.scan(offsets, E, lane);
    int mt = 0;
    if (!map_tile(b, x.total, ntn, mt, nt)) return false;
    e = x.find(mt, within);
    return true;
}
