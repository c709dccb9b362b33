// Which tile a workgroup of a GEMM launch runs: integer functions of its index,
// also compiled for the host by the test that walks them.  DEV and min come from
// the including file.
#pragma once

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
// What is left after the whole rounds goes in chunks of 4: a window of the
// bounded-memory backward has rows for some of the experts only, and contiguous
// shares left it on few XCDs (4 of 12 experts of 6 tiles, three products: 27 tiles
// on each of three XCDs, some CUs two deep; the launch 338 us, now 190).
constexpr int WG_STRIP = 4, WG_CHUNK = 16;
DEV bool map_tile_wgrad(int b, int groups, int ntm, int ntn, int &cm, int &nt) {
    const int per = ntm * ntn;
    const int n = groups * per, full = n / (8 * WG_CHUNK) * (8 * WG_CHUNK);
    int t = b < full ? deal_tile(b, full, WG_CHUNK) : deal_tile(b - full, n - full, WG_STRIP);
    if (t < 0) return false;
    if (b >= full) t += full;
    const int e = t / per, i = t % per;
    const int whole = ntn / WG_STRIP * WG_STRIP;       // n-tiles in strips of 4
    const int strip = i < whole * ntm ? i / (WG_STRIP * ntm) : whole / WG_STRIP;
    const int wid = i < whole * ntm ? WG_STRIP : ntn - whole;
    const int w = i - strip * WG_STRIP * ntm;
    cm = e * ntm + w / wid;
    nt = strip * WG_STRIP + w % wid;
    return true;
}

// Workgroups of a launch whose tiles map_tile_wgrad places, and no more of the
// last round than have one: several products follow each other in a launch, and
// places without a tile between them put one product's tiles on the same shader
// engines as the last one's.
inline long wgrad_grid(long groups, int ntm, int ntn) {
    const long n = groups * ntm * ntn, rounds = n / (8 * WG_CHUNK);
    return 8 * (rounds * WG_CHUNK + (n - rounds * 8 * WG_CHUNK + 7) / 8);
}
