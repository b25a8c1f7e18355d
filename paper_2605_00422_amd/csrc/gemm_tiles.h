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
// The constants are fitted to 2500 shapes (the projections of the 4096-, 5120- and 8192-wide blocks and others at random:
// 17 .. 4096 tokens, K 128 .. 28672, N 32 .. 40000, ranks 0 .. 128), each with plain and gated int8 codes and with nibble
// codes, three layers in turn so that nothing stays in L2, short launches from a graph.  Over those the choice is within
// 0.7 / 0.8 / 0.4 % of the best of the ten on average, and more than a tenth above it at 1.3 / 1.5 / 1.2 % of them.  (Constants fitted
// to an epilogue that took longer and to fewer short launches: 1.6 / 1.7 / 0.9 % and 4.6 / 5.5 / 2.9 %; with these 11 % of the
// calls take 2 % less time or better and 0.5 % that much more.  24 tokens of 512 columns, 270 channels, rank 0 5.4 -> 4.6 us.)  Five more tiles
// that were candidates (64 x 32 for one wavefront, 256 x 128 with rings of two and four, 256 x 160, 64 x 640 with private
// rings) moved no average by more than 0.1 % and are not built.
#pragma once

#include <stddef.h>
#include <stdint.h>

// bytes of LDS that the epilogue's rows of T fill (EpRows in gemm_epilogue.h)
inline size_t ep_rows_bytes(int tokens, int r) { return (size_t)tokens * ((r + 15) / 16 * 64 + 12); }

struct GdTile {
    int ntl, wk, nb, wn;          // 32-channel tiles a wavefront; wavefronts that share K; ring depth; wavefronts side by side
    int resident;                 // workgroups a CU holds (LDS, registers) up to rank 112
    float start, base[4], slice[4], idle, low, a4;
};
constexpr int GD_TILE_TOKENS = 64;
constexpr GdTile GD_TILES[] = {
    // few tokens: private rings, the wavefronts of a workgroup share out K
    {1, 4, 4, 1, 1, 1.42f, {4.76f}, {0.3940f}, 0.0963f, 0.353f, 0.954f},                                                  // 64 x 32, in four
    {2, 4, 4, 1, 1, 1.78f, {4.58f}, {0.4895f}, 0.1293f, 0.541f, 1.030f},                                                  // 64 x 64, in four
    {2, 2, 4, 1, 2, 1.71f, {5.25f, 6.94f}, {0.3802f, 0.3879f}, 0.0872f, 0.711f, 0.931f},                                  // 64 x 64, in two
    {3, 2, 4, 1, 2, 1.95f, {7.29f, 10.01f}, {0.5066f, 0.5755f}, 0.0908f, 0.838f, 0.944f},                                 // 64 x 96, in two
    // one ring of codes for four wavefronts (the first: two)
    {1, 1, 4, 2, 4, 3.15f, {2.24f, 3.61f, 5.04f, 7.02f}, {0.2804f, 0.3010f, 0.4477f, 0.4147f}, 0.0345f, 0.654f, 1.102f},  // 64 x 64
    {1, 1, 4, 4, 3, 3.52f, {1.99f, 5.13f, 7.93f}, {0.3036f, 0.4222f, 0.5095f}, 0.0809f, 0.552f, 1.103f},                  // 64 x 128
    {2, 1, 4, 4, 2, 1.69f, {8.81f, 9.37f}, {0.3710f, 0.6488f}, 0.0786f, 0.769f, 1.027f},                                  // 64 x 256
    {3, 1, 4, 4, 2, 3.77f, {8.62f, 13.44f}, {0.4060f, 0.8893f}, 0.1199f, 0.869f, 1.089f},                                 // 64 x 384
    {4, 1, 2, 4, 2, 4.46f, {9.33f, 15.62f}, {0.6637f, 1.2518f}, 0.1257f, 1.119f, 1.044f},                                 // 64 x 512, ring of two
    {5, 1, 4, 4, 1, 0.00f, {16.35f}, {0.8438f}, 0.2189f, 1.854f, 1.089f},                                                 // 64 x 640
};
constexpr int GD_NTILES = sizeof(GD_TILES) / sizeof(GD_TILES[0]);

// LDS of a workgroup: the code rings, then in their place the epilogue's tiles and rows of T
inline size_t gd_lds_bytes(const GdTile& v, int r) {
    const size_t ring = (size_t)v.wk * v.nb * (GD_TILE_TOKENS * 128);
    const size_t tail = (size_t)(v.wk > 1 ? v.wk * (GD_TILE_TOKENS / 32) * v.ntl : v.wn) * 4096 + ep_rows_bytes(GD_TILE_TOKENS, r);
    return ring > tail ? ring : tail;
}
// Workgroups that a CU's 160 KiB hold: the rows of T grow with the rank, and from 113 on 64 x 96 in two no longer goes
// twice, nor 64 x 64 with one ring four times.  (Taken for resident as before, they were chosen where half of them had to wait:
// 2810 tokens of 19968 columns, 906 channels, rank 120 102.7 -> 64.2 us; 335 of 9728, 6927 channels 67.7 -> 39.0; 24 such
// shapes 0.65 of the time on average, 0.83 at most.)
inline int gd_resident(const GdTile& v, int r) {
    const int fit = (int)(160 * 1024 / gd_lds_bytes(v, r));
    return fit < v.resident ? fit : v.resident;
}

inline float gd_cost(const GdTile& v, int64_t M, int64_t K, int64_t N, int r, int64_t cus, bool a4) {
    const int64_t bn = v.wn * v.ntl * 32;
    const int64_t tiles_n = (N + bn - 1) / bn, tiles = (M + GD_TILE_TOKENS - 1) / GD_TILE_TOKENS * tiles_n;
    const int resident = gd_resident(v, r);
    const int64_t cap = cus * resident;
    const float slices = (float)(((K >> 7) + v.wk - 1) / v.wk);
    const int64_t full = tiles / cap, rem = tiles - full * cap;
    float t = v.start + (float)full * (v.base[resident - 1] + v.slice[resident - 1] * slices);
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

// index into GD_TILES (*least: its cost)
inline int gd_pick(int64_t M, int64_t K, int64_t N, int r, int64_t cus, bool a4, float* least = nullptr) {
    int best = 0;
    float cost = gd_cost(GD_TILES[0], M, K, N, r, cus, a4);
    for (int i = 1; i < GD_NTILES; ++i) {
        const float c = gd_cost(GD_TILES[i], M, K, N, r, cus, a4);
        if (c < cost) { cost = c; best = i; }
    }
    if (least != nullptr) *least = cost;
    return best;
}

// Tiles of the sparse GEMM (gemm_sparse.hip), which serves codes of at most 7 bits and more than 64 tokens where it is
// the faster one.  The same kind of cost, `step` per superstep of 512 columns; in front of it the pass that turns the codes
// into sums and differences (a launch, and the codes once in and once out).  It contracts twice the columns an instruction
// but prepares its operands at more cost, in steps of 512 columns, and its wide tiles start and finish slowly: it wins where
// tiles are many and rows of K long.  Fitted to 945 pairs of shape and form (65 .. 4096 tokens, K 128 .. 28672, N 32 .. 51200,
// plain and gated), three layers in turn; it is taken where its cost is 3 % below the dense kernel's.  Over those the choice
// took 0.992 of the time of the dense kernel as it was then (0.988 with the best tile of both every time), with 2 times more than
// 2 % above it; without the 3 %, 16.  Long ones against the dense kernel as it is, rank 64: 0.72 (28672 -> 28672 at 4096
// tokens), 0.75 (28672 -> 8192), 0.87 (8192 -> 28672), 0.90 (25600 -> 5120 at 2048), 0.96 (4096 -> 22016 gated).  64 x 128,
// 64 x 384 and 128 x 384 tiles were candidates and move the average by less than 0.7 % at ten times as many wrong choices.
struct GsTile {
    int mt, nt, wn, ring;         // 32-token tiles and 32-channel tiles a wavefront; wavefronts side by side; pairs in the code ring
    int resident;                 // workgroups a CU holds
    float start, base[2], step[2], idle, low;
};
constexpr int GS_MIN_TOKENS = 64;
constexpr GsTile GS_TILES[] = {
    {2, 2, 4, 4, 2, 6.00f, {3.51f, 7.60f}, {1.289f, 2.061f}, 0.264f, 1.256f},       // 64 x 256
    {2, 5, 4, 4, 1, 2.33f, {15.80f}, {2.557f}, 0.618f, 2.203f},                     // 64 x 640
    {4, 4, 4, 4, 1, 1.17f, {23.09f}, {3.298f}, 0.894f, 3.621f},                     // 128 x 512
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

// index into GS_TILES, or -1: the dense kernel (*dense: its tile, so that the launch need not pick again)
inline int gs_pick(int64_t M, int64_t K, int64_t N, int r, int64_t cus, int* dense = nullptr) {
    if (M <= GS_MIN_TOKENS) return -1;
    int best = -1;
    float cost;
    const int d = gd_pick(M, K, N, r, cus, false, &cost);
    if (dense != nullptr) *dense = d;
    for (int i = 0; i < GS_NTILES; ++i) {
        const float c = 1.03f * gs_cost(GS_TILES[i], M, K, N, r, cus);
        if (c < cost) { cost = c; best = i; }
    }
    return best;
}
