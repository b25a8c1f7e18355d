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
            const int plain = s.r1_bytes + g * (s.xt_bytes + 256), full = plain + g * s.cb_bytes;
            if (plain > limit) continue;
            s.G = g; s.own = full <= limit; s.threads = 64 * (w + extra);
            break;
        }
    }
    s.lds_bytes = (size_t)s.r1_bytes + (size_t)s.G * (s.xt_bytes + (s.own ? s.cb_bytes : 0) + 256);
    return s;
}

// the calls that it takes: rows of whole pairs of values, and everything fits (fp32 tokens: up to 128 x 96).  Not those of nine or
// ten strips whose registers would not do: with R1 streamed (64 tokens: 160 x 160 32.9 us, rotate_bf16_device.h 26.3; 144 x 144
// 31.2, 25.3), or walking over few tokens (96 x 148: 257 tokens 42.1, 33.3; 400 tokens 42.1, 41.5; but 700 tokens 57.9, 61.0).
inline bool rt_serves(const bwla_layer_t* L, int xdtype, int64_t M, int64_t cus) {
    const int n1 = L->n1, n2 = L->n2;
    const bool f32 = xdtype != BWLA_X_BF16;
    if ((n2 & 1) != 0 || n1 > (f32 ? 128 : 256) || n2 > (f32 ? 96 : n1 > 128 ? 128 : 160)) return false;
    if (n2 > 128 && M > cus && M < 2 * cus) return false;
    return rt_shape(n1, n2, 1, 1, f32 ? RT_F32 : RT_BF16).lds_bytes <= RQ_LDS_LIMIT;
}
// 128 x 64 with a token or two a CU: on the terms of rotate_planes.hip, which takes more tokens of that pair, in its order
inline bool rt_as_planes(const bwla_layer_t* L, int xdtype, int64_t M, int64_t cus) {
    return xdtype == BWLA_X_BF16 && L->n1 == 128 && L->n2 == 64 && L->off_Rd != 0 && M >= cus && M < 2 * cus;
}

}  // namespace

hipError_t bwla_launch_rotate_terms(const bwla_layer_t* L, const RqArgs& a, int64_t pblocks, bool rides, bool f32, hipStream_t st);
hipError_t bwla_launch_rotate_terms_many(const RtArgs& b, RtKind kind, int64_t blocks, int threads, size_t lds, hipStream_t st);
hipError_t bwla_launch_rotate_terms_f32(const RtArgs& b, bool many, int64_t blocks, int threads, size_t lds, hipStream_t st);
