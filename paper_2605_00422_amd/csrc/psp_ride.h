// Whether the projection T = X U of M > 16 tokens rides in the rotation's launch (psp_block_device.h) or has one of its
// own in front or behind (psp_prefill.hip).  Host arithmetic without HIP types: a CPU test compiles it by itself.
//
// It rides where its workgroups (`riders`) finish in the rotation's shadow: a rotation workgroup has a CU to itself and
// takes about 6 us + K / 1050, the CUs that the last round of them leaves free take a round of projection workgroups every
// 5.5 us.  A little beside the shadow is still less than the launch of its own that the projection needs otherwise (6 to
// 7 us), and so is a small round behind the rotation.  Not where the kernel that walks over the tokens serves (planes),
// which is the faster one by more.  Rotation + projection, riding / in a launch of its own, and the rotation alone: 8192
// columns, rank 64: 128 tokens 16.7 / 21 / 13.3; 255 tokens 29.8 / 22.7 / 14.3; 25600, rank 32: 128 tokens 28.3 / 34 / 26.6;
// 5120, rank 32: 257 tokens 16.8 / 23 / 17.
//
// Those are bf16 tokens.  Of fp32 tokens the rotation takes longer, and the projection's own launch reads twice the bytes
// and hands its sums over inside (bwla_launch_rotate_quant): there it rides as well while that launch stays within about
// three workgroups a CU.  5120 columns, rank 37, 192 tokens 13.9 / 26.7, 320 tokens 21.6 / 32.4; 4096, rank 37, 384 tokens
// 18.5 / 27.2; 8192, rank 64, 173 tokens 25.2 / 33.2; of 40 whole layers at random that ride by this alone 0.87 of the time
// on average, 0.99 at most.  (bf16 tokens in the same fp32 kernel, whose factors are too long for the other: 1.00, 1.10.)
//
// And of bf16 tokens whose rotation is a slow one (`slow`: factors too large for LDS with five strips of wavefronts or fewer, or
// that the fp32 kernel rotates) the shadow is 1.75 times as long: 172 x 64 29 us, 200 x 80 40, 163 x 32 25.  Rank 8, 185 tokens,
// riding / in a launch of its own: 172 x 64 30.4 / 35.8, 200 x 80 41.4 / 47.1; 163 x 32, 400 tokens 49.1 / 56.1, 172 x 64 57.8 / 62.6;
// rank 64, 158 tokens 172 x 64 34.7 / 36.9, 192 x 64 38.0 / 36.5, 256 x 48 39.6 / 40.0, 163 x 32 26.1 / 34.4.
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
