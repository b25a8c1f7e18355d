// Rotation + quantization of bf16 tokens (paper Sec. 3.1, Sec. 4.1), any even n2 up to 160 and n1 up to 256: the
// arithmetic of rotate_planes.hip (the token scaled by a power of two and exact in fp16, both factors and the intermediate
// as two fp16 terms, 22 bits, fp32 accumulation) for factor pairs and token counts that it has no kernel for.
//
//   stage 1  Z[a,d]  = sum_b V[a,b] R2[b,d]       V: the token's n1 x n2 reshape
//   stage 2  Yt[d,c] = sum_a Z[a,d] R1[a,c]       x~[c n2 + d] = Yt[d,c]
//
// The factors come padded to multiples of 32 with zeros, in operand order (one contiguous KiB an MFMA operand).
// Wavefront w of a group owns the 16 columns d of strip w, and alternates between the stages per 32-deep step of the long
// product, so that Z is never whole anywhere.
//
// What bounds it at few tokens is a wavefront by itself: one workgroup a token, and in it one chain of loads, two stages,
// a maximum, codes and stores.  So the chain is kept short: operands need no address arithmetic, the R1 terms are fetched by
// wavefronts that have no other errand (asynchronously into LDS; a rotating wavefront waits for its own few loads
// only), the loop over the steps is rolled (straight-line code is fetched once and not used again), codes are rounded
// by an addition and leave in whole lines.  Against three exact bf16 terms and six products, straight-line code and factors
// carried through registers (rotate_bf16_device.h, which keeps odd n2 and layers packed without these factors), us a launch:
//   tokens            16 x 32   64 x 64   64 x 80   128 x 64   128 x 86   160 x 160   224 x 128
//   16, rank 0        6.5 / 4.4 8 / 5.7   9.4 / 5.8 13.6 / 7.1 12.8 / 9.4 15.2 / 14.3 16.0 / 15.8
//   64, rank 32       6.4 / 4.5 8.1 / 6.4 9.3 / 6.7 14.4 / 7.2 18.7 / 9.8 29.0 / 16.0 35.1 / 17.1
//   512 (walking)     14.6/ 6.7           20.8/11.1            41.6/19.9
//   2048 (walking)    13.6/ 8.3           59.6/22.9            130 / 57
// Error against fp64 (rms of a token's scale, relative; share of differing 8-bit codes): 64 x 64 1.11e-7 and 3.8e-6 with
// the three terms, 0.99e-7 and 3.2e-6 here; 128 x 86 1.47e-7 and 4.4e-6, 1.08e-7 and 3.1e-6; 172 x 64 2.3e-7 and 6.2e-6, 1.5e-7 and
// 4.1e-6; of 17 pairs the codes are nearer in 16 (512 values: 5 and 5 codes in two million).
#include "rotate_terms_device.h"

hipError_t bwla_launch_rotate_terms(const bwla_layer_t* L, const RqArgs& a, int64_t pblocks, bool rides, hipStream_t st) {
    const char* blob = (const char*)L->d_blob;
    RtArgs b;
    b.q = a;
    b.R1h = (const uint16_t*)(blob + L->off_Rd + bwla_decode_planes_r2_bytes(L->n1, L->n2));
    b.R2h = b.R1h + bwla_planes_r1h_bytes(L->n1) / 2;
    const int cus = bwla_device_cus();
    const bool many = !rides && a.M > cus;
    b.s = rt_shape(L->n1, L->n2, many ? a.M : 1, cus);
    int64_t wgs = (a.M + b.s.G - 1) / b.s.G;
    if (many && wgs > cus) wgs = cus;
    b.q.rot_blocks = wgs;
    b.rounds = (int)((a.M + wgs * b.s.G - 1) / (wgs * b.s.G));
    int threads = b.s.threads;
    if (rides && threads < 512) threads = 512;         // the projection's workgroups want eight wavefronts
    const size_t plds = rides ? pp_lds_bytes(a.r, threads / 64) : 0;
    const size_t lds = b.s.lds_bytes > plds ? b.s.lds_bytes : plds;
    return many ? bwla_launch_rotate_terms_many(b, wgs + pblocks, threads, lds, st) : launch_terms<false>(b, wgs + pblocks, threads, lds, st);
}

// More tokens than CUs, in rows long enough that a token has a CU to itself: walking, with the projection in front, 128 x 64 at 300
// tokens takes 16.8 us, a workgroup a token with the projection riding 18.4; 16 x 32 at 512 tokens 11 and 6.7.
bool bwla_rotation_walks(const bwla_layer_t* L, int xdtype, int64_t M) {
    if (bwla_rotate_planes_serves(L, xdtype, M)) return true;
    return xdtype == BWLA_X_BF16 && L->K >= 2048 && M > bwla_device_cus() && rt_serves(L);
}
