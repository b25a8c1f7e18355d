// Which tile of the streaming GEMM (gemm_prefill.hip) serves M > 16 tokens and N channels.  Host arithmetic without HIP
// types: a CPU test compiles it by itself.
//
// Most tiles below win somewhere between 17 and 4096 tokens, and what decides is how their number comes out in rounds
// over the CUs: 257 tokens x 8192 channels are 104 to 128 large tiles (half the chip, half of the rows padding) or 430
// tiles of 64 x 96, two to a CU.  So each tile carries a small cost, in microseconds: a workgroup takes base[s - 1] +
// slice[s - 1] per 128-column slice of K that a wavefront contracts when s share the CU; full rounds run at the largest
// s, the last one at the s that it comes to, a slice being cheaper by `idle` for each of its workgroups that the CUs
// could still take; 16 ranks cost a round `low`; `start` is paid once.  With nibble codes, of which a slice moves half
// the bytes, all of it times `a4`.  And it takes no less than the codes need: workgroups are dealt out over the 8 XCDs
// in runs of tiles with the same token rows where their number is a multiple of eight, and each row enters one L2;
// otherwise up to eight L2s fetch it.  The smallest cost is taken.
//
// The constants are fitted to 924 shapes (the projections of the 4096-, 5120- and 8192-wide blocks at 17 to 4096
// tokens, the others at random: 17 .. 4096 tokens, K 128 .. 28672, N 32 .. 28672, ranks 0 .. 96), each with plain and
// gated int8 codes and with nibble codes, three layers in turn so that nothing stays in L2.  Over those the choice is
// within 0.4 / 0.7 / 0.5 % of the best of fifteen tiles on average, and takes 0.896 / 0.891 / 0.913 of the time that
// two thresholds between large and small private-ring tiles led to; 17 of the 2772 times are more than 2 % above those
// (the worst by 16 %).  Constants fitted to plain codes alone, without `idle`, `low` and the codes' own time, left 192
// (the worst by 42 %; 18 tokens of nibble codes on 1280 columns 5.7 -> 7.1 us, 28672 -> 8192 at 1024 tokens, plain,
// 188 -> 216; without `low` alone, 4096 -> 12288 at 4096 tokens and rank 96 245 -> 268).  Five more tiles that were
// candidates (64 x 32 for one wavefront, 256 x 128 with rings of two and four, 256 x 160, 64 x 640 with private
// rings) moved no average by more than 0.1 % and are not built.
#pragma once

#include <stdint.h>

struct GdTile {
    int ntl, wk, nb, wn;          // 32-channel tiles a wavefront; wavefronts that share K; ring depth; wavefronts side by side
    int resident;                 // workgroups a CU holds (LDS of the tile rings, registers)
    float start, base[4], slice[4], idle, low, a4;
};
constexpr int GD_TILE_TOKENS = 64;
constexpr GdTile GD_TILES[] = {
    // few tokens: private rings, the wavefronts of a workgroup share out K
    {1, 4, 4, 1, 1, 0.69f, {7.96f}, {0.3473f}, 0.1138f, 1.202f, 0.912f},                                                  // 64 x 32, in four
    {2, 4, 4, 1, 1, 0.62f, {10.30f}, {0.4917f}, 0.0945f, 1.326f, 1.002f},                                                 // 64 x 64, in four
    {2, 2, 4, 1, 2, 2.28f, {7.93f, 9.71f}, {0.4145f, 0.4223f}, 0.0694f, 1.332f, 0.946f},                                  // 64 x 64, in two
    {3, 2, 4, 1, 2, 2.11f, {10.44f, 13.07f}, {0.5221f, 0.5891f}, 0.1048f, 1.438f, 0.927f},                                // 64 x 96, in two
    // one ring of codes for four wavefronts (the first: two)
    {1, 1, 4, 2, 4, 2.27f, {4.46f, 7.54f, 8.57f, 8.88f}, {0.3572f, 0.3201f, 0.3833f, 0.4758f}, 0.0522f, 1.149f, 0.988f},  // 64 x 64
    {1, 1, 4, 4, 3, 4.91f, {2.49f, 6.66f, 10.52f}, {0.3331f, 0.4092f, 0.6233f}, 0.0662f, 1.323f, 1.020f},                 // 64 x 128
    {2, 1, 4, 4, 2, 3.39f, {4.37f, 12.24f}, {0.4005f, 0.6627f}, 0.0784f, 1.572f, 1.000f},                                 // 64 x 256
    {3, 1, 4, 4, 2, 3.60f, {7.23f, 17.55f}, {0.5550f, 0.9247f}, 0.1131f, 1.670f, 1.000f},                                 // 64 x 384
    {4, 1, 2, 4, 2, 3.85f, {11.71f, 22.08f}, {0.6995f, 1.3362f}, 0.2233f, 1.878f, 1.000f},                                // 64 x 512, ring of two
    {5, 1, 4, 4, 1, 0.00f, {19.87f}, {0.8199f}, 0.1241f, 2.171f, 0.980f},                                                 // 64 x 640
};
constexpr int GD_NTILES = sizeof(GD_TILES) / sizeof(GD_TILES[0]);

inline float gd_cost(const GdTile& v, int64_t M, int64_t K, int64_t N, int r, int64_t cus, bool a4) {
    const int64_t bn = v.wn * v.ntl * 32;
    const int64_t tiles_n = (N + bn - 1) / bn, tiles = (M + GD_TILE_TOKENS - 1) / GD_TILE_TOKENS * tiles_n;
    const int64_t cap = cus * v.resident;
    const float slices = (float)(((K >> 7) + v.wk - 1) / v.wk);
    const int64_t full = tiles / cap, rem = tiles - full * cap;
    float t = v.start + (float)full * (v.base[v.resident - 1] + v.slice[v.resident - 1] * slices);
    if (rem > 0) {
        const int share = (int)((rem + cus - 1) / cus);
        t += v.base[share - 1] + (v.slice[share - 1] - v.idle * ((float)share - (float)rem / (float)cus)) * slices;
    }
    t += (float)((full + (rem > 0 ? 1 : 0)) * ((r + 15) / 16)) * v.low;
    if (a4) t *= v.a4;
    // codes at 5 MB a microsecond (a large read's rate), behind the launch and the first round trips
    const float fetched = (float)(M * K) * (a4 ? 0.5e-6f : 1.0e-6f) * (tiles % 8 == 0 ? 1.0f : (float)(tiles_n < 8 ? tiles_n : 8));
    const float least = 6.0f + fetched / 5.0f;
    return t > least ? t : least;
}

// index into GD_TILES
inline int gd_pick(int64_t M, int64_t K, int64_t N, int r, int64_t cus, bool a4) {
    int best = 0;
    float cost = gd_cost(GD_TILES[0], M, K, N, r, cus, a4);
    for (int i = 1; i < GD_NTILES; ++i) {
        const float c = gd_cost(GD_TILES[i], M, K, N, r, cus, a4);
        if (c < cost) { cost = c; best = i; }
    }
    return best;
}

// Tiles of the sparse GEMM (gemm_sparse.hip), which serves codes of at most 7 bits and more than 64 tokens where it is
// the faster one.  The same kind of cost, `step` per superstep of 512 columns; in front of it the pass that turns the codes
// into sums and differences (a launch, and the codes once in and once out).  It contracts twice the columns an instruction
// but prepares its operands at more cost, in steps of 512 columns, and its wide tiles start and finish slowly: it wins where
// tiles are many and rows of K long.  Fitted to 279 shapes (65 .. 4096 tokens, K 256 .. 28672, N 64 .. 51200, 73 of them
// gated), three layers in turn; it is taken where its cost is 5 % below the dense kernel's.  Over those shapes the choice
// takes 0.974 of the dense kernel's time (0.968 with the best tile of both every time; 0.62 .. 0.9 where M K N > 1e11), with
// 2 of 279 times more than 2 % above it; without the 5 %, 9.  64 x 128, 64 x 384 and 128 x 384 tiles were candidates and
// move the average by less than 0.7 % at ten times as many wrong choices.
struct GsTile {
    int mt, nt, wn, ring;         // 32-token tiles and 32-channel tiles a wavefront; wavefronts side by side; pairs in the code ring
    int resident;                 // workgroups a CU holds
    float start, base[2], step[2], idle, low;
};
constexpr int GS_MIN_TOKENS = 64;
constexpr GsTile GS_TILES[] = {
    {2, 2, 4, 4, 2, 4.92f, {4.13f, 8.09f}, {1.500f, 2.401f}, 0.513f, 1.257f},       // 64 x 256
    {2, 5, 4, 4, 1, 0.77f, {16.83f}, {2.774f}, 0.829f, 1.675f},                     // 64 x 640
    {4, 4, 4, 4, 1, 0.69f, {24.61f}, {3.577f}, 1.122f, 2.267f},                     // 128 x 512
};
constexpr int GS_NTILES = sizeof(GS_TILES) / sizeof(GS_TILES[0]);

inline float gs_cost(const GsTile& v, int64_t M, int64_t K, int64_t N, int r, int64_t cus) {
    const int64_t bm = 32 * v.mt, bn = (int64_t)32 * v.nt * v.wn;
    const int64_t tiles = (M + bm - 1) / bm * ((N + bn - 1) / bn), cap = cus * v.resident;
    const float steps = (float)((K + 511) / 512);
    const int64_t full = tiles / cap, rem = tiles - full * cap;
    float t = v.start + (float)full * (v.base[v.resident - 1] + v.step[v.resident - 1] * steps);
    if (rem > 0) {
        const int share = (int)((rem + cus - 1) / cus);
        t += v.base[share - 1] + (v.step[share - 1] - v.idle * ((float)share - (float)rem / (float)cus)) * steps;
    }
    t += (float)((full + (rem > 0 ? 1 : 0)) * ((r + 15) / 16)) * v.low;
    return t + 1.5f + (float)(M * K) * 2.0f / 6.3e6f;
}

// index into GS_TILES, or -1: the dense kernel
inline int gs_pick(int64_t M, int64_t K, int64_t N, int r, int64_t cus) {
    if (M <= GS_MIN_TOKENS) return -1;
    int best = -1;
    float cost = gd_cost(GD_TILES[gd_pick(M, K, N, r, cus, false)], M, K, N, r, cus, false);
    for (int i = 0; i < GS_NTILES; ++i) {
        const float c = 1.05f * gs_cost(GS_TILES[i], M, K, N, r, cus);
        if (c < cost) { cost = c; best = i; }
    }
    return best;
}
