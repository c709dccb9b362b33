// Which path a forward takes: rules on sizes alone, host code without HIP.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>

// Small batches (skinny.hip): 16-row tiles per workgroup, 0 for the tile GEMMs.
//
// 64-row tiles from 17 tokens up: more rows per pass over the weights beat
// the smaller tiles' higher occupancy at every mean row count (128 experts, us
// with 16 / 32 / 64 rows: 256 tokens 306 / 284 / 280, 512: 393 / 338 / 315);
// up to 16 tokens no expert has more than 16 rows.
//
// Up to 64 rows per expert on average: there more experts take a second tile
// and the tile GEMMs catch up.  (us here / there) 128 experts of 768, d 2048:
// 512 tokens 276 / 333, 1000 330 / 353; 32 of 1536, d 4096: 100 tokens with a
// hot expert 259 / 334, 250 336 / 341; 200 of 768, one expert per token: 8000
// tokens 466 / 545, 12800 549 / 580.  The host sees the mean only, and an uneven
// load moves the crossing down: with a router bias of std 2 it lies near 40 rows
// (128 experts: 32 rows 167 / 185, 64 rows 237 / 216; 200 experts: 20 rows 182 /
// 201, 64 rows 325 / 271), and a router collapsed onto 8 of 128 experts runs 512
// tokens in 117 / 95.
//
// The shared expert's rows are all T tokens, re-reading its weights per 64 of
// them: past the first 64 its products count up to the routed ones' bound, T f_s
// <= 64 E f.  200 experts of 768, one per token, and a shared one of 2048 (us
// here / there): 4000 tokens (T f_s = 53 E f) 506 / 615, 8000 (107) 745 / 739,
// 12800 (171) 1003 / 892; of 1024: 8000 (53) 616 / 649, 12800 (85) 784 / 756; 32 of
// 1536 and one of 2048: 1000 (42) 387 / 418, 2000 (83) 512 / 506.
inline int skinny_tiles(long T, long k, long E, long f, long fs) {
    if (T <= 0) return 0;
    if (T <= 16) return 1;
    return T * k <= 64 * E && (T <= 64 || T * fs <= 64 * E * f) ? 4 : 0;
}
// Tokens past which skinny_tiles is 0 for every f and fs.
inline long skinny_max_tokens(long E, long k) { return 64 * E / k > 16 ? 64 * E / k : 16; }

// Tiles of bm rows that R routes to E experts fill at most.
inline long skinny_slots(long R, long E, long bm) { return (R < E ? R : E) + R / bm; }

// K slices of a small batch's up/gate product: its workgroups (64 columns of f
// each) run in rounds of the 256 CUs, so 288 of them (8 experts and a shared one
// of 2048 columns) take as long as 512.  K is split over two or four where that
// ends the launch earlier, if each slice keeps 1024 rows; the SwiGLU then moves to
// a launch of its own (4 us), the slices are at most five rounds and their sums
// take at most SK_SLICE_BYTES.
//
// Workgroups are counted for the experts that T balanced tokens reach, with a
// tenth for the ones they reach beyond that (if there are any left).  Slices that just fit one round do
// so only where the launch has no spare workgroups: those end at once and leave
// their CU to a second one.
//
// Forward at 1 / 2 / 4 slices (us), by workgroups: 16, d 5120: 36 / - / 25; 64, d
// 4096: 56 / 45 / 41; 96, d 2048: 32.5 / 30.2; 112, d 4096: 60 / 50 / 52; 128, d 2048:
// 40 / 37, with spare ones 42 / 45; 148, d 4096: 62 / 65 / 56; 288, d 7168: 1 token
// 186 / 169 / 160, 61 tokens 242 / 214 / 206; 344, d 7168: 186 / 175; 592, d
// 6144: whole call 326 / 315.  As many rounds
// either way: 175, d 4096: 71 / 82 / 78; 210: 73 / 70 / 79; 256: 92 / 96 / 100; 444: 139 /
// 144; 493, d 2048: 73 / 78.
constexpr long SK_SPLIT_MAX = 4;
constexpr size_t SK_SLICE_BYTES = size_t(48) << 20;

inline long skinny_max_slices(long d) {
    long s = 1;
    while (s < SK_SPLIT_MAX && d / (2 * s) >= 1024) s *= 2;
    return s;
}

inline int skinny_kslices(long T, long k, long E, long d, long f, long fs, long tt) {
    const long R = T * k, bm = 16 * tt, shared = (T + bm - 1) / bm * (fs / 64);
    double reached = E * (1.0 - std::pow(1.0 - (double)k / E, (double)T));
    if (reached < R / bm) reached = (double)(R / bm);
    const long wgs = (long)std::ceil(reached * (f / 64) - 1e-6) + shared;
    const long grid = skinny_slots(R, E, bm) * (f / 64) + shared;
    const long most = T <= bm ? (R < E ? R : E) * (f / 64) + shared : grid;   // T rows: one tile per expert
    long best = 1, rounds = (wgs + 255) / 256;        // of `best` slices each
    for (long s = 2; s <= skinny_max_slices(d); s *= 2) {
        const long n = wgs * s;
        if (wgs >= (s == 2 ? 640 : 320) || 8 * (size_t)s * ((size_t)R * f + (size_t)T * fs) > SK_SLICE_BYTES) break;
        const long r = n <= 252 ? 1 : n <= 256 ? 1 + (grid * s > 256) : (std::min(n + n / 10, most * s) + 255) / 256;
        if (r * best < rounds * s) {
            best = s;
            rounds = r;
        }
    }
    return (int)best;
}

// Dense routing on few token tiles: the folded down product has one workgroup
// per 256 x 256 tile of Y and a K loop over every expert, so a short batch
// leaves most CUs idle (200 tokens at d 7168: 28 workgroups of 288 K steps).
// The experts' products can run as tiles of their own into fp32 instead, with a
// small kernel that adds them in the same order of experts.  That shortens the
// chain of K steps from E f / 64 to `rounds` f / 64, rounds of the 256 CUs
// that E products of Y's tiles take, and costs a write and a read of fp32
// products, (E + shared) T d of them.  A K step of 64 takes about 1.4 us and
// the fp32 traffic runs at about 4.5 TB/s, so the two meet near 12000 values
// per column of f that the chain is shorter by.  Forward, folded / in parts
// (us): 8 experts and a shared one of 2048, d 7168: 200 tokens 706 / 387, 500
// 737 / 494; 8 of 1024, d 1024: 2048 tokens 253 / 128, 8192 450 / 481; 16 of
// 2048, d 256: 8192 tokens 1194 / 636; 8 of 256, d 1024: 2048 tokens 84 / 68,
// 8192 125 / 203; 2 of 256, d 256: 30000 tokens 49 / 71; over 306 shapes of 2
// to 16 experts the line is at most 10 % off the better side.
// Up to 64 tiles of Y a product of its own runs in quarter tiles, which the folded
// one cannot, in about two thirds of the time; that is all there is to gain with
// one expert, and for the shared expert's part of the chain: 1 expert of 2048, d
// 256: 300 tokens 62 / 34, 16000 138 / 122; of 512, d 1024: 2000 tokens 33.6 / 32.2,
// 4000 36 / 40; of 256, d 256, and a shared one of 1024: 2000 tokens 53 / 45, 16000
// 99 / 101; 2 of 512 and one of 1024, d 1024: 2000 tokens 85 / 70.
// Only up to half of the CUs' worth of Y tiles: past them the folded product
// fills the chip itself.
constexpr long DENSE_PARTS_MAX = 128, DENSE_PARTS_VALUES = 12000;
constexpr long DENSE_QUARTER_MAX = 64, DENSE_QUARTER_VALUES = 4500;

inline bool dense_parts(long T, long d, long E, long k, long f, long fs) {
    const long nt = (T + 255) / 256 * (d / 256);
    if (k != E || T <= 0 || nt > DENSE_PARTS_MAX) return false;
    const long rounds = (E * nt + 255) / 256;
    const long quarters = nt <= DENSE_QUARTER_MAX ? DENSE_QUARTER_VALUES * (fs + (E == 1 ? f : 0)) : 0;
    return (E + (fs > 0)) * T * d <= DENSE_PARTS_VALUES * f * (E - rounds) + quarters;
}

// Experts padded to the routers' tiles.
inline long route_padded(long E) {
    long p = 16;
    while (p < E) p *= 2;
    return p;
}

// The one-launch router: it re-reads W_r per 16 tokens, so up to 2048 tokens,
// and larger batches keep their logits' summation order.  Its loads of several
// expert columns need them aligned in every row.
//
// Up to 64 experts at every d (us here / the other routers): 32 experts, d
// 4096: 1 token 8.7 / 16.2, 1000 11.7 / 19.3, 2000 12.0 / 19.4; 64, d 16384:
// 1 token 37 / 74, 2048 50 / 83.  Past that a wave's chain of steps is long (8
// waves, 16 rows of W_r a lane in flight at 256) while the split router deals d
// to 8 blocks, and the two cross between d 3584 and 6144, later for more routes
// per token, which the split router's second launch selects on few CUs.
// 128 experts, top 1: d 4608 16 tokens 15.5 / 15.0, 2048 20 / 23; d 5120 16.6 / 15.4;
// top 8: d 5120 20 / 19, 500 tokens 22 / 24; d 7168 25 / 21, 29 / 26.  256 experts,
// top 1: d 3584 20 / 21, 28 / 29; d 4096 2048 tokens 32 / 30; d 4608 36 / 30; top 8:
// d 4608 30 / 30, 41 / 41; d 5120 740 tokens 34 / 40, 2048 45 / 41; d 7168 57 / 44;
// top 16, d 5120: 55 / 62.  W_r, re-read per 16 tokens, counts too: top 8, d 5120,
// 2048 tokens to 160 experts 38 / 42, 1600 to 200 40 / 42, to 256 44 / 43.  Over
// 3400 measured shapes at most 4 % (0.6 us) slower.
constexpr long ROUTE_DIRECT_MAX = 2048, ROUTE_DIRECT_ROWS = 160 * 2048;

inline bool route_direct(long T, long d, long E, long k) {
    const long ep = route_padded(E), cols = ep / 16 < 8 ? ep / 16 : 8;
    if (T <= 0 || T > ROUTE_DIRECT_MAX || E % cols) return false;
    if (ep <= 64) return true;
    if (ep == 128) return d <= (k >= 8 ? 5120 : 4608);
    const long top = k >= 8 ? 4608 : k >= 4 ? 4096 : 3584;
    return d <= top + (k >= 16 || (k >= 4 && T * E <= ROUTE_DIRECT_ROWS) ? 512 : 0);
}

// The third LDS stage of B in a row product of `rows` rows over `groups` experts
// (DEEP in gemm.hip) pays while an expert's weights serve few m-tiles and costs
// a little where they serve many (its loads then hit in L2 either way, and more
// of them queue).  Forward, two / three stages (us), mean rows per expert: 125:
// 394 / 369, 512 (128 experts): 906 / 878, 1000: 1315 / 1291, 1024 (128 experts):
// 1570 / 1541, 2048: 2461 / 2453, 3000: 3580 / 3607, 4096: 4752 / 4777.
//
// Short products have no K steps to hide it in: with 4 or 8 of 64 the loads
// ahead are the whole product, and its tiles start later.  Forward that keeps
// its activations, d = f, two / three stages (us): K 256, 128 experts: 16 rows
// 34.3 / 35.3, 300 76.5 / 77.9; K 512: 16 rows 67.7 / 69.8, 100 79.4 / 81.1, 300
// 164 / 161, 900 378 / 368; K 768: 16 rows 149 / 151, 300 326 / 311; K 1024, 64
// experts: 16 rows 124 / 119, 300 267 / 253.
constexpr long DEEP_ROWS = 1024, DEEP_K = 768, DEEP_SHORT_K = 512, DEEP_SHORT_ROWS = 200;

inline bool deep_stages(long K, long rows, long groups) {
    const long n = groups > 0 ? groups : 1;
    if (rows > DEEP_ROWS * n) return false;
    return K >= DEEP_K || (K >= DEEP_SHORT_K && rows >= DEEP_SHORT_ROWS * n);
}

// The MXFP8 up/gate product's kept pre-activations (fp32, two values per element
// of H) go past the L2, as every other output (gemm_mx.hip).  Not where they fit
// the Infinity Cache beside little else: a short K loop then waits for these
// stores, and past the L2 they run at 2.4 TB/s instead of 3.5.  Forward that keeps
// them, past / through the L2 (us): d 256, 1500 rows of 8 experts, f 1024 (98 MB)
// 87 / 79, f 2048 (197 MB) 139 / 124; d 512, f 1536 125 / 113; d 1024, f 1024 116 / 106,
// f 2048 189 / 186; d 2048, f 1536 224 / 232.  Fewer rows (256 of 32 experts, d 1024,
// f 1536: 122 / 134), smaller (49 MB, d 256: 56 / 58) and larger (393 MB, d 512: 0.92
// of the time) are faster past it.
inline bool mx_keep_l2(long R, long E, long K, long N) {
    const long bytes = 8 * R * N;
    return K <= 1024 && R >= 1024 * E && bytes >= (64L << 20) && bytes <= (208L << 20);
}
