// Whether the projection T = X U of M > 16 tokens rides in the rotation's launch (psp_block_device.h) or has one of its
// own in front or behind (psp_prefill.hip).  Host arithmetic without HIP types: a CPU test compiles it by itself.
//
// It rides where its workgroups (`riders`) finish in the rotation's shadow: a rotation workgroup has a CU to itself, the CUs that
// the last round of them leaves free take a round of projection workgroups at a time.  A little beside the shadow is still less
// than the launch of its own that the projection needs otherwise (4 to 7 us), and so is a small round behind the rotation.
// Not where a kernel that walks over the tokens serves (planes), which is the faster one by more.
// The shadow of 9 us + K / 1050 and the 5.5 us a round are those of rotate_bf16_device.h and of projections on fp32 MFMA; with
// rotate_terms.hip and bf16 MFMA both are shorter, and it is their quotient that counts.  Rotation + projection, riding / in a launch
// of its own, us, * where the rule takes the second: 128 x 64, rank 64: 128 tokens 13.2 / 16.6, 158 15.6 / 16.9 *, 255 23.0 / 19.0 *;
// 160 x 160, rank 32: 128 tokens 26.9 / 32.6, 185 34.8 / 33.2 *; 64 x 80, rank 32: 185 tokens 7.7 / 12.4, rank 64: 158 tokens
// 8.9 / 13.4 *, 256 tokens 12.9 / 13.8 *; 128 x 86, rank 64: 96 tokens 13.7 / 20.6, 200 tokens 25.2 / 21.2 *.  Of 805 calls (15 pairs of
// bf16 tokens, 7 of fp32 ones, 17 to 650 tokens, ranks 8, 32, 64) in which the two differ by 0.3 us it takes the better one to
// within 5 % in 732; in the others, as those above, it does not ride where riding would be the better by up to a half.
//
// Those are bf16 tokens.  Of fp32 tokens the rotation takes longer, and the projection's own launch reads twice the bytes
// and hands its sums over inside (bwla_launch_rotate_quant): there it rides as well while that launch stays within about
// three workgroups a CU.  64 x 80, rank 32, 200 tokens 11.2 / 21.9, 333 tokens 16.1 / 26.2; 64 x 64, rank 32, 400 tokens
// 13.3 / 21.3, but rank 64 17.3 / 26.3 *; 128 x 64, rank 64, 173 tokens 21.1 / 30.6.
//
// And of bf16 tokens whose rotation is a slow one for its length (`slow`: factors too large for the LDS of rotate_bf16_device.h with
// five strips of wavefronts or fewer, or too long for it) the shadow is 1.75 times as long.  Rank 8, 185 tokens: 172 x 64
// 20.2 / 23.6, 200 x 80 29.0 / 31.8, 163 x 32 19.1 / 24.4, 256 x 48 26.5 / 32.1; 200 tokens 172 x 64 22.1 / 23.4 *; rank 64, 158 tokens
// 172 x 64 24.2 / 25.2, 256 x 48 28.8 / 33.5, 163 x 32 19.2 / 26.8.
#pragma once

#include <stdint.h>

inline bool psp_rides(int64_t M, int64_t K, int64_t riders, int64_t cus, bool planes, bool f32, bool slow = false) {
    if (planes || M > 768) return false;
    // (short rows leave room for several workgroups a CU: there it is their number that counts, up to three a CU; 512
    // columns, rank 64, 384 tokens 11.7 / 18.5)
    if (K < 2048 || f32) {
        if (M + riders <= 768) return true;
        if (K < 2048) return false;
    }
    const int64_t beside = (cus - M % cus) % cus;              // CUs that the last round leaves free
    const float length = slow ? 1.75f * (6.0f + (float)K / 1050.0f) : 9.0f + (float)K / 1050.0f;
    const bool shadow = beside > 0 && 5.5f * (float)((riders + beside - 1) / beside) <= length;
    return shadow || riders <= 192;
}
