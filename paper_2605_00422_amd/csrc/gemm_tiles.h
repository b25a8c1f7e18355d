// Which tile of the streaming GEMM (gemm_prefill.hip) serves M > 16 tokens and N channels.  Host arithmetic without HIP
// types: a CPU test compiles it by itself.
//
// Most tiles below win somewhere between 17 and 4096 tokens, and what decides is how their number comes out in rounds
// over the CUs: 257 tokens x 8192 channels are 104 to 128 large tiles (half the chip, half of the rows padding) or 430
// tiles of 64 x 96, two to a CU.  So each tile carries a small cost, in microseconds: a workgroup takes base[r - 1] +
// slice[r - 1] per 128-column slice of K that a wavefront contracts when r share the CU; full rounds run at the largest
// r, the last one at the r that it comes to, a slice being cheaper by `idle` for each of its workgroups that the CUs
// could still take; `start` is paid once.  With nibble codes, of which a slice moves half the bytes, all of it times
// `a4`.  And it takes no less than the codes need: workgroups are dealt out over the 8 XCDs in runs of tiles with the
// same token rows where their number is a multiple of eight, and each row enters one L2; otherwise up to eight L2s
// fetch it.  The smallest cost is taken.
//
// The constants are fitted to 852 shapes (the projections of the 4096-, 5120- and 8192-wide blocks at 17 to 4096
// tokens, the others at random: 17 .. 4096 tokens, K 128 .. 28672, N 32 .. 28672), each with plain and gated int8
// codes and with nibble codes, three layers in turn so that nothing stays in L2.  Over those the choice is within
// 0.4 / 0.7 / 0.4 % of the best of fifteen tiles on average, and takes 0.897 / 0.893 / 0.914 of the time that two
// thresholds between large and small private-ring tiles led to; 22 of the 2556 times are more than 2 % above those
// (the worst by 16 %).  Constants fitted to plain codes alone, without `idle` and the codes' own time, left 176 (the
// worst by 42 %; 18 tokens of nibble codes on 1280 columns 5.7 -> 7.1 us, 28672 -> 8192 at 1024 tokens, plain,
// 188 -> 216).  Five more tiles that were candidates (64 x 32 for one wavefront, 256 x 128 with rings of two and
// four, 256 x 160, 64 x 640 with private rings) moved no average by more than 0.1 % and are not built.
#pragma once

#include <stdint.h>

struct GdTile {
    int ntl, wk, nb, wn;          // 32-channel tiles a wavefront; wavefronts that share K; ring depth; wavefronts side by side
    int resident;                 // workgroups a CU holds (LDS of the tile rings, registers)
    float start, base[4], slice[4], idle, a4;
};
constexpr int GD_TILE_TOKENS = 64;
constexpr GdTile GD_TILES[] = {
    // few tokens: private rings, the wavefronts of a workgroup share out K
    {1, 4, 4, 1, 1, 0.87f, {10.42f}, {0.3377f}, 0.1405f, 0.875f},                                                     // 64 x 32, in four
    {2, 4, 4, 1, 1, 1.04f, {13.10f}, {0.5311f}, 0.1183f, 0.922f},                                                     // 64 x 64, in four
    {2, 2, 4, 1, 2, 3.07f, {9.94f, 12.94f}, {0.4594f, 0.4196f}, 0.0829f, 0.900f},                                     // 64 x 64, in two
    {3, 2, 4, 1, 2, 2.48f, {12.97f, 17.38f}, {0.5518f, 0.5312f}, 0.1100f, 0.945f},                                    // 64 x 96, in two
    // one ring of codes for four wavefronts (the first: two)
    {1, 1, 4, 2, 4, 2.24f, {7.25f, 10.34f, 13.53f, 12.25f}, {0.3176f, 0.3263f, 0.3504f, 0.4934f}, 0.0447f, 0.946f},   // 64 x 64
    {1, 1, 4, 4, 3, 4.07f, {6.03f, 9.79f, 11.68f}, {0.3383f, 0.4335f, 0.6751f}, 0.0834f, 1.000f},                     // 64 x 128
    {2, 1, 4, 4, 2, 2.31f, {9.69f, 13.60f}, {0.4123f, 0.6720f}, 0.1024f, 0.951f},                                     // 64 x 256
    {3, 1, 4, 4, 2, 3.83f, {12.73f, 19.44f}, {0.4759f, 0.9153f}, 0.1152f, 0.990f},                                    // 64 x 384
    {4, 1, 2, 4, 2, 1.80f, {15.40f, 24.53f}, {0.6896f, 1.3210f}, 0.2848f, 0.970f},                                    // 64 x 512, ring of two
    {5, 1, 4, 4, 1, 0.00f, {20.34f}, {0.7974f}, 0.1229f, 0.998f},                                                     // 64 x 640
};
constexpr int GD_NTILES = sizeof(GD_TILES) / sizeof(GD_TILES[0]);

inline float gd_cost(const GdTile& v, int64_t M, int64_t K, int64_t N, int64_t cus, bool a4) {
    const int64_t bn = v.wn * v.ntl * 32;
    const int64_t tiles_n = (N + bn - 1) / bn, tiles = (M + GD_TILE_TOKENS - 1) / GD_TILE_TOKENS * tiles_n;
    const int64_t cap = cus * v.resident;
    const float slices = (float)(((K >> 7) + v.wk - 1) / v.wk);
    const int64_t full = tiles / cap, rem = tiles - full * cap;
    float t = v.start + (float)full * (v.base[v.resident - 1] + v.slice[v.resident - 1] * slices);
    if (rem > 0) {
        const int r = (int)((rem + cus - 1) / cus);
        t += v.base[r - 1] + (v.slice[r - 1] - v.idle * ((float)r - (float)rem / (float)cus)) * slices;
    }
    if (a4) t *= v.a4;
    // codes at 5 MB a microsecond (a large read's rate), behind the launch and the first round trips
    const float fetched = (float)(M * K) * (a4 ? 0.5e-6f : 1.0e-6f) * (tiles % 8 == 0 ? 1.0f : (float)(tiles_n < 8 ? tiles_n : 8));
    const float least = 6.0f + fetched / 5.0f;
    return t > least ? t : least;
}

// index into GD_TILES
inline int gd_pick(int64_t M, int64_t K, int64_t N, int64_t cus, bool a4) {
    int best = 0;
    float cost = gd_cost(GD_TILES[0], M, K, N, cus, a4);
    for (int i = 1; i < GD_NTILES; ++i) {
        const float c = gd_cost(GD_TILES[i], M, K, N, cus, a4);
        if (c < cost) { cost = c; best = i; }
    }
    return best;
}
