// Rotation + quantization of tokens (paper Sec. 3.1, Sec. 4.1) for any even n2 up to 160 and n1 up to 256 (fp32 tokens: up to
// 128 x 96), for the factor pairs and token counts that rotate_planes.hip has no kernel for.
//
//   stage 1  Z[a,d]  = sum_b V[a,b] R2[b,d]       V: the token's n1 x n2 reshape
//   stage 2  Yt[d,c] = sum_a Z[a,d] R1[a,c]       x~[c n2 + d] = Yt[d,c]
//
//   bf16 tokens   as they are; the factors and Z as three bf16 terms (24 bits), three and six products on the 16x16x32 MFMA.
//                 The sums of rotate_bf16_device.h in its order: the same values to the bit
//   fp32 tokens   fp32 MFMA, the sums of rotate_f32_device.h in its order: the same values to the bit
//   128 x 64, a token or two a CU   the two fp16 terms (22 bits) of rotate_planes.hip, which takes more tokens, to the bit again
// What the other kernels give is kept to the last bit so that a code on a rounding boundary does not depend on which of them runs.
// (Two fp16 terms for all pairs were nearer to the exact value with ordinary tokens, but not with those that have one channel far
// above the others, where nothing averages 22 bits out: a channel 1e8 above, 128 x 86, 700 tokens, the largest error of a scale
// 4.4e-7 against 2.1e-7 and 9.6e-6 of the 8-bit codes against 1.6e-6.  Pairs too long for rotate_bf16_device.h, whose bf16 tokens
// the fp32 kernel rotated: 172 x 64 at 128 tokens, rms of a scale's error 2.3e-7 there and 1.5e-7 on three bf16 terms.  Of those it
// rotates few tokens still where n2 is up to 16, or up to 32 with n1 above 192: rt_serves says which calls stay elsewhere, and why.)
//
// Factors and rows are padded with zeros to multiples of 32.  Wavefront w of a group owns the 16 columns d of
// strip w, and alternates between the stages per 32-deep step of the long product, so that Z is never whole anywhere.
//
// What bounds it at few tokens is a wavefront by itself: one workgroup a token, and in it one chain of loads, two stages,
// a maximum, codes and stores.  So the chain is kept short: the R1 terms are fetched by wavefronts that have no other errand
// (asynchronously into LDS; a rotating wavefront waits for its own few loads only), the loop over the steps is rolled
// (straight-line code is fetched once and not used again), two tiles' products take turns (a tile's own wait for each other:
// 128 x 64 10.4 -> 10.0 us), codes leave in whole lines.  With many tokens it is the MFMAs.  Against straight-line
// code with factors carried through registers (rotate_bf16_device.h, rotate_f32_device.h: odd n2, longer pairs), us a launch
// with the projection riding, rank 32:
//   tokens            16 x 32    64 x 64    64 x 80    128 x 64   128 x 86   224 x 128  172 x 64
//   16                6.2 / 5.2  7.7 / 5.7  8.9 / 6.4  12.9 / 9.9 (split)    (split)    28.6 / 16.8
//   64                6.3 / 5.3  7.8 / 5.8  9.0 / 6.5  13.2 /10.0 17.7/12.8  31.1/26.6  28.8 / 17.0
//   700 (walking)     15.9/ 5.2             30.3/22.2             59.9/43.2             94.2 / 53.8
//   2048 (walking)    19.6/13.5             67.5/35.3             135 / 82              236 / 91
//   fp32, 16          5.6 / 5.4  8.5 / 7.3  11.0/10.0  16.2 /13.1 30.9/23.1
//   fp32, 1024        20.3/14.7  34.9/29.3  44.2/37.0  77 / 55    155 / 96
#include "rotate_terms_device.h"

hipError_t bwla_launch_rotate_terms(const bwla_layer_t* L, const RqArgs& a, int64_t pblocks, bool rides, bool f32, hipStream_t st) {
    const char* blob = (const char*)L->d_blob;
    RtArgs b;
    b.q = a;                                            // (its R1p, R2p: the bf16 terms)
    b.R1h = (const uint16_t*)(blob + L->off_Rd + bwla_decode_planes_r2_bytes(L->n1, L->n2));
    b.R2h = b.R1h + bwla_planes_r1h_bytes(L->n1) / 2;
    const int cus = bwla_device_cus();
    const RtKind kind = f32 ? RT_F32 : !rides && rt_as_planes(L, BWLA_X_BF16, a.M, cus) ? RT_H16 : RT_BF16;
    const bool many = !rides && (a.M > cus || kind == RT_H16);
    b.s = rt_shape(L->n1, L->n2, many ? a.M : 1, cus, kind);
    int64_t wgs = (a.M + b.s.G - 1) / b.s.G;
    if (many && wgs > cus) wgs = cus;
    b.q.rot_blocks = wgs;
    b.rounds = (int)((a.M + wgs * b.s.G - 1) / (wgs * b.s.G));
    int threads = b.s.threads;
    if (rides && threads < 512) threads = 512;         // the projection's workgroups want eight wavefronts
    const size_t plds = rides ? pp_lds_bytes(a.r, threads / 64) : 0;
    const size_t lds = b.s.lds_bytes > plds ? b.s.lds_bytes : plds;
    if (f32) return bwla_launch_rotate_terms_f32(b, many, wgs + pblocks, threads, lds, st);
    return many ? bwla_launch_rotate_terms_many(b, kind, wgs + pblocks, threads, lds, st) : launch_terms<false>(b, wgs + pblocks, threads, lds, st);
}

// More tokens than CUs, in rows long enough that a token has a CU to itself: walking, with the projection in front, 128 x 64 at 300
// tokens takes 16.8 us, a workgroup a token with the projection riding 18.4; 16 x 32 at 512 tokens 11 and 6.7.  With R1 streamed
// where one token is in flight a workgroup, walking saves nothing that the projection could not ride behind: rank 32, 257 tokens,
// 144 x 112 42.3 walking and 32.8 riding, 200 x 80 58.8 and 47.6; two in flight 172 x 64 29.1 and 31.7.  Nor with R1 resident and seven
// strips or more (six and few rows), of which one token is in flight too, before the second round is half full:
// 257 tokens 48 x 96 17.9 and 8.8, 48 x 112 23.4 and 16.9, 128 x 112 39.1 and 31.2, 300 tokens 80 x 128 30.7 and 25.2.
bool bwla_rotation_walks(const bwla_layer_t* L, int xdtype, int64_t M) {
    if (bwla_rotate_planes_serves(L, xdtype, M)) return true;
    const int64_t cus = bwla_device_cus();
    if (xdtype != BWLA_X_BF16 || L->K < 2048 || M <= cus || (L->n1 > 128 && L->n2 > 64)) return false;
    if (2 * M <= 3 * cus && (L->n2 > 96 || (L->n2 > 80 && L->n1 <= 64))) return false;
    if (M < 2 * cus && L->n1 > 128 && L->n2 <= 16) return false;       // (rt_serves: not where the projection rides)
    return rt_serves(L, xdtype, M, cus, 0);
}
