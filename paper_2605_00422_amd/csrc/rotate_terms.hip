// Rotation + quantization of tokens (paper Sec. 3.1, Sec. 4.1) for any even n2 up to 160 and n1 up to 256 (fp32 tokens: up to
// 128 x 96), for the factor pairs and token counts that rotate_planes.hip has no kernel for.
//
//   stage 1  Z[a,d]  = sum_b V[a,b] R2[b,d]       V: the token's n1 x n2 reshape
//   stage 2  Yt[d,c] = sum_a Z[a,d] R1[a,c]       x~[c n2 + d] = Yt[d,c]
//
// Operands are sums of 16-bit terms on the 16x16x32 MFMA, accumulated in fp32:
//   n1 <= 64, bf16 tokens   the factors and Z as three bf16 terms, six products
//   else                    the token scaled by a power of two, exact in fp16 (fp32 tokens as three fp16 terms), both factors and
//                           Z as two fp16 terms (22 bits), as in rotate_planes.hip
// The factors come padded to multiples of 32 with zeros, one KiB an operand.  Wavefront w of a group owns the 16 columns d of
// strip w, and alternates between the stages per 32-deep step of the long product, so that Z is never whole anywhere.
//
// What bounds it at few tokens is a wavefront by itself: one workgroup a token, and in it one chain of loads, two stages,
// a maximum, codes and stores.  So the chain is kept short: operands need no address arithmetic, the R1 terms are fetched by
// wavefronts that have no other errand (asynchronously into LDS; a rotating wavefront waits for its own few loads
// only), the loop over the steps is rolled (straight-line code is fetched once and not used again), codes are rounded
// by an addition and leave in whole lines.  Against straight-line code, factors carried through registers and fp32 MFMA
// for fp32 tokens (rotate_bf16_device.h, rotate_f32_device.h: odd n2, longer pairs, layers packed without these
// terms), us a launch with the projection riding:
//   tokens            16 x 32   64 x 64   64 x 80   128 x 64   128 x 86   160 x 160   224 x 128
//   16, rank 0        6.5 / 4.4 8 / 6.0   9.4 / 6.2 13.6 / 7.1 12.8 / 9.4 15.2 / 14.3 16.0 / 15.8
//   64, rank 32       6.4 / 4.5 8.1 / 6.6 9.3 / 6.9 14.4 / 7.2 18.7 / 9.8 29.0 / 16.0 35.1 / 17.1
//   512 (walking)     14.6/ 6.7           20.8/11.6            41.6/19.9
//   2048 (walking)    13.6/ 8.3           59.6/24              130 / 57
//   fp32, 16, rank 32 6.4 / 4.9 9.3 / 8.3 11.4/ 8.1 16.7 / 8.8 31.3 / 12.1
//   fp32, 1024        12.9/ 6.8 25.5/14.5 34.2/18.9 68 / 33    146 / 45
// Error against fp64 (rms of a token's scale, relative; share of differing 8-bit codes), before / here: 16 x 32 6.2e-8 and
// 2.3e-6 / 6.2e-8 and 1.8e-6; 64 x 64 1.11e-7 and 3.8e-6 / 0.79e-7 and 2.4e-6; 128 x 86 1.47e-7 and 4.4e-6 / 1.07e-7 and 3.3e-6;
// 172 x 64 2.3e-7 and 6.2e-6 / 1.5e-7 and 4.1e-6; fp32 16 x 32 1.18e-7 and 4.0e-6 / 0.92e-7 and 3.6e-6, 128 x 64 2.1e-7 and 5.8e-6 /
// 1.1e-7 and 4.3e-6.
#include "rotate_terms_device.h"

hipError_t bwla_launch_rotate_terms(const bwla_layer_t* L, const RqArgs& a, int64_t pblocks, bool rides, bool f32, hipStream_t st) {
    const char* blob = (const char*)L->d_blob;
    RtArgs b;
    b.q = a;                                            // (its R1p, R2p: the bf16 terms)
    b.R1h = (const uint16_t*)(blob + L->off_Rd + bwla_decode_planes_r2_bytes(L->n1, L->n2));
    b.R2h = b.R1h + bwla_planes_r1h_bytes(L->n1) / 2;
    const int cus = bwla_device_cus();
    const bool many = !rides && a.M > cus;
    b.s = rt_shape(L->n1, L->n2, many ? a.M : 1, cus, f32);
    int64_t wgs = (a.M + b.s.G - 1) / b.s.G;
    if (many && wgs > cus) wgs = cus;
    b.q.rot_blocks = wgs;
    b.rounds = (int)((a.M + wgs * b.s.G - 1) / (wgs * b.s.G));
    int threads = b.s.threads;
    if (rides && threads < 512) threads = 512;         // the projection's workgroups want eight wavefronts
    const size_t plds = rides ? pp_lds_bytes(a.r, threads / 64) : 0;
    const size_t lds = b.s.lds_bytes > plds ? b.s.lds_bytes : plds;
    if (f32) return bwla_launch_rotate_terms_f32(b, many, wgs + pblocks, threads, lds, st);
    return many ? bwla_launch_rotate_terms_many(b, wgs + pblocks, threads, lds, st) : launch_terms<false>(b, wgs + pblocks, threads, lds, st);
}

// More tokens than CUs, in rows long enough that a token has a CU to itself: walking, with the projection in front, 128 x 64 at 300
// tokens takes 16.8 us, a workgroup a token with the projection riding 18.4; 16 x 32 at 512 tokens 11 and 6.7.
bool bwla_rotation_walks(const bwla_layer_t* L, int xdtype, int64_t M) {
    if (bwla_rotate_planes_serves(L, xdtype, M)) return true;
    return xdtype == BWLA_X_BF16 && L->K >= 2048 && M > bwla_device_cus() && rt_serves(L);
}
