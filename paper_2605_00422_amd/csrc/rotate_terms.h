// Shapes of the rotation by strips for any even factor pair (rotate_terms.hip).
#pragma once
#include "rotate_args.h"

// what it multiplies: bf16 tokens with three bf16 terms of the factors, or (128 x 64) two fp16 ones; fp32 tokens in fp32
enum RtKind { RT_BF16, RT_H16, RT_F32 };

struct RtShape {
    int at, k1, ch2, strips;         // 16-row tiles along n1 (padded to 32), 32-deep steps along n2 and n1, 16-column strips
    int G, threads;                  // groups of strip wavefronts (a token each), threads with the wavefronts that fetch R1
    int pitch, r1_bytes, xt_bytes, cb_bytes;
    bool stream, own;                // R1 terms a step at a time; room for the codes beside the token rows
    size_t lds_bytes;
};

struct RtArgs {
    RqArgs q;
    const uint16_t* R1h; const uint16_t* R2h;
    RtShape s;
    int rounds;
};

namespace {

// M > 1: workgroups walk over that many tokens
inline RtShape rt_shape(int n1, int n2, int64_t M, int cus, RtKind kind) {
    RtShape s;
    s.ch2 = (n1 + 31) >> 5; s.at = 2 * s.ch2;
    s.strips = (n2 + 15) >> 4; s.k1 = (n2 + 31) >> 5;
    s.pitch = (kind == RT_F32 ? s.strips : s.k1) * 64 + 16;
    s.stream = n1 > 128;             // (three terms of 160 x 160 are 150 KiB)
    s.r1_bytes = (s.stream ? 2 : s.ch2) * (kind == RT_BF16 ? 3 : 2) * s.at * 1024;
    s.xt_bytes = s.ch2 * 32 * s.pitch;
    s.cb_bytes = (n1 * n2 + 255) & ~255;
    const int limit = (int)RQ_LDS_LIMIT;
    int loaders = s.stream ? 0 : s.strips <= 4 ? 4 : s.strips <= 8 ? 8 - s.strips + (s.strips == 8 ? 2 : 0) : 2;
    if (!s.stream && s.r1_bytes >= 65536) loaders = 12 - s.strips;       // (128 x 86: 14.7 us with two, 12.9 with six)
    s.G = 1; s.own = false; s.threads = 64 * (s.strips + loaders);
    if (M > 1) {
        // as many groups as the registers and LDS hold, and as there are tokens for
        const int most = s.stream ? 8 : 12;
        s.threads = 0;
        for (int g = 4; g >= 1; --g) {
            int w = g * s.strips, extra = s.stream ? 0 : most - w < loaders ? most - w : loaders;
            if (g > 1 && (w > most || (!s.stream && extra < 1) || (int64_t)(g - 1) * cus >= M)) continue;
            // (fp32: nor more than the same number of rounds takes; 96 x 48, 1024 tokens: three a workgroup 32.4 us, two 25.0)
            auto rounds = [&](int g) { return (M + (int64_t)g * cus - 1) / ((int64_t)g * cus); };
            if (kind == RT_F32 && g > 1 && rounds(g - 1) == rounds(g)) continue;
            const int plain = s.r1_bytes + g * (s.xt_bytes + 256), full = plain + g * s.cb_bytes;
            if (plain > limit) continue;
            s.G = g; s.own = full <= limit; s.threads = 64 * (w + extra);
            break;
        }
    }
    s.lds_bytes = (size_t)s.r1_bytes + (size_t)s.G * (s.xt_bytes + (s.own ? s.cb_bytes : 0) + 256);
    return s;
}

// fp32 tokens that rotate_f32_device.h rotates sooner.  (riders: the projection's workgroups in the same launch)
inline bool rt_f32_sooner(int n1, int n2, int64_t M, int64_t cus, int64_t riders, const RtShape& one) {
    // Tiles that one SIMD works off one after the other: here a wavefront takes a strip of tiles, padded to pairs; there eight
    // wavefronts share all tiles, and whole tiles have no edges to look after.
    const bool whole = ((n1 | n2) & 15) == 0;
    const int here = (one.strips + 3) / 4 * one.at, there = 2 * ((n1 / 16 * one.strips + 7) / 8);
    const bool uneven = whole && here >= 6 && 2 * here >= 3 * there;
    // 64 tokens, here / there: 80 x 16 8.9 / 7.6, 96 x 32 10.0 / 8.7, 128 x 32 12.6 / 11.2, 80 x 48 9.9 / 8.7, 112 x 80 20.1 / 18.6;
    // not uneven: 64 x 64 8.0 / 8.6, 96 x 64 10.9 / 14.1, 128 x 48 13.2 / 15.3, with ragged tiles 96 x 40 10.5 / 14.4
    const bool crowded = riders > 0 && M + riders > cus;
    if (uneven && M <= cus && !crowded) return true;
    // one workgroup a CU that the projection's have to wait for where two go there (rank 32: 256 tokens 112 x 32 18.3 / 12.0,
    // 104 x 24 17.8 / 14.7, 512 tokens 28.7 / 20.3 and 28.0 / 22.8; 96 x 32, two a CU in both, 10.6 / 12.1)
    const size_t half = RQ_LDS_LIMIT / 2;
    const bool alone = one.lds_bytes > half && rq_shape(n1, n2).lds_bytes <= half;
    if (crowded && n1 > 96 && n2 <= 32 && (uneven || alone)) return true;
    // (two a CU in both, few strips behind many rows, 256 tokens: 104 x 16 14.3 / 12.7; one in both: 112 x 80 32.1 / 31.8, 257 tokens
    // 37.9 / 35.3, but 400 tokens 44.5 / 49.4)
    if (crowded && n1 > 96 && n1 <= 112 && (n2 <= 16 || (uneven && 2 * M <= 3 * cus))) return true;
    // walking, an uneven pair of small factors: a last round that is hardly half full (48 x 80 and 80 x 80, 700 tokens 20.7 / 19.0 and
    // 34.6 / 32.2, 512 tokens 13.1 / 13.2 and 21.4 / 21.9), six strips on four SIMDs (80 x 48: 512 tokens 14.6 / 13.1, 700 17.9 / 19.0)
    if (uneven && riders == 0 && M > cus && n1 <= 80 && n2 >= 48 && n2 <= 80) {
        if (one.strips == 3 && M <= 2 * cus) return true;
        const int64_t a_round = rt_shape(n1, n2, M, (int)cus, RT_F32).G * cus, rounds = (M + a_round - 1) / a_round;
        return 10 * M < 7 * rounds * a_round;
    }
    return false;
}

// the calls that it takes: rows of whole pairs of values, and everything fits (fp32 tokens: up to 128 x 96).  Not those of nine or
// ten strips whose registers would not do: with R1 streamed (64 tokens: 160 x 160 32.9 us, rotate_bf16_device.h 26.3; 144 x 144
// 31.2, 25.3), or walking over few tokens (96 x 148: 257 tokens 42.1, 33.3; 400 tokens 42.1, 41.5; but 700 tokens 57.9, 61.0), or
// ten with n1 above 96 and a token a workgroup (112 x 160: 128 tokens 21.8, 20.4; 96 x 160 14.2, 16.2).
inline bool rt_fits(int n1, int n2, bool f32) {
    return (n2 & 1) == 0 && n1 <= (f32 ? 128 : 256) && n2 <= (f32 ? 96 : n1 > 128 ? 128 : 160) &&
           rt_shape(n1, n2, 1, 1, f32 ? RT_F32 : RT_BF16).lds_bytes <= RQ_LDS_LIMIT;
}
inline bool rt_serves(const bwla_layer_t* L, int xdtype, int64_t M, int64_t cus, int64_t riders) {
    const int n1 = L->n1, n2 = L->n2;
    const bool f32 = xdtype != BWLA_X_BF16;
    if (!rt_fits(n1, n2, f32)) return false;
    const RtShape one = rt_shape(n1, n2, 1, 1, f32 ? RT_F32 : RT_BF16);
    if (f32) return !rt_f32_sooner(n1, n2, M, cus, riders, one);
    if (n2 > 128 && M > cus && M < 2 * cus) return false;
    if (n2 > 144 && n1 > 96 && M <= cus) return false;
    // R1 streamed by one wavefront or two: it waits for every step of it, where rotate_bf16_device.h keeps R1 or has the rows in
    // more hands.  One (n2 up to 16): 64 tokens 144 x 16 20.8, 11.7, 256 x 16 43.1, 17.4; 300 tokens, walking 160 x 16 17.5, 23.9,
    // 192 x 16 22.5, 18.7, 256 x 16 34.5, 24.5; 1024 tokens 224 x 16 23.1, 41.1, 256 x 16 56.0, 47.1; 2048 tokens 82.6, 90.2.
    if (one.stream && one.strips == 1)
        if (M <= cus || riders > 0 || (n1 > 176 && M <= 2 * cus) || (n1 > 224 && M < 8 * cus)) return false;
    // Two: 64 tokens 224 x 32 23.6, 22.2, 256 x 24 28.8, 26.6; 192 x 32 18.7, 19.3, but with 256 tokens and the projection 25.0, 22.5
    if (one.stream && one.strips == 2 && M <= cus && (n1 > 192 || (n1 > 176 && riders > 0 && 2 * M > cus))) return false;
    return true;
}
// 128 x 64 with a token or two a CU: on the terms of rotate_planes.hip, which takes more tokens of that pair, in its order
inline bool rt_as_planes(const bwla_layer_t* L, int xdtype, int64_t M, int64_t cus) {
    return xdtype == BWLA_X_BF16 && L->n1 == 128 && L->n2 == 64 && L->off_Rd != 0 && M >= cus && M < 2 * cus;
}

}  // namespace

hipError_t bwla_launch_rotate_terms(const bwla_layer_t* L, const RqArgs& a, int64_t pblocks, bool rides, bool f32, hipStream_t st);
hipError_t bwla_launch_rotate_terms_many(const RtArgs& b, RtKind kind, int64_t blocks, int threads, size_t lds, hipStream_t st);
hipError_t bwla_launch_rotate_terms_f32(const RtArgs& b, bool many, int64_t blocks, int threads, size_t lds, hipStream_t st);
