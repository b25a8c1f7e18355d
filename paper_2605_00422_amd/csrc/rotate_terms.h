// Shapes of the rotation on 16-bit terms for any factor pair (rotate_terms.hip).
#pragma once
#include "rotate_args.h"

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
inline RtShape rt_shape(int n1, int n2, int64_t M, int cus, bool f32 = false) {
    RtShape s;
    s.ch2 = (n1 + 31) >> 5; s.at = 2 * s.ch2;
    s.strips = (n2 + 15) >> 4; s.k1 = (n2 + 31) >> 5;
    s.pitch = s.k1 * 64 + 16;
    s.stream = n1 > 160;
    s.r1_bytes = (s.stream ? 2 : s.ch2) * (s.at <= 4 && !f32 ? 3 : 2) * s.at * 1024;
    s.xt_bytes = s.ch2 * 32 * s.pitch * (f32 ? 3 : 1);
    s.cb_bytes = (n1 * n2 + 255) & ~255;
    const int limit = (int)RQ_LDS_LIMIT, loaders = s.stream ? 0 : s.strips <= 4 ? 4 : s.strips <= 8 ? 8 - s.strips + (s.strips == 8 ? 2 : 0) : 2;
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

// the pairs that it takes: the factors' terms exist, rows of whole pairs of values, and everything fits
// (fp32 tokens: as three terms beside resident factors, up to 128 x 96)
inline bool rt_serves(const bwla_layer_t* L, bool f32 = false) {
    if ((L->n2 & 1) != 0 || (L->off_Rd == 0 && (f32 || L->n1 > 64))) return false;
    const int strips = (L->n2 + 15) >> 4;
    if (L->n1 > 160 && strips > 8) return false;
    if (f32 && (L->n1 > 128 || L->n2 > 96)) return false;
    const RtShape s = rt_shape(L->n1, L->n2, 1, 1, f32);
    return s.lds_bytes <= RQ_LDS_LIMIT && s.strips <= 10;
}

}  // namespace

hipError_t bwla_launch_rotate_terms(const bwla_layer_t* L, const RqArgs& a, int64_t pblocks, bool rides, bool f32, hipStream_t st);
hipError_t bwla_launch_rotate_terms_many(const RtArgs& b, int64_t blocks, int threads, size_t lds, hipStream_t st);
hipError_t bwla_launch_rotate_terms_f32(const RtArgs& b, bool many, int64_t blocks, int threads, size_t lds, hipStream_t st);
