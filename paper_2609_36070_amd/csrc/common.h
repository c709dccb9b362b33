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

#include "raster.h"

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
