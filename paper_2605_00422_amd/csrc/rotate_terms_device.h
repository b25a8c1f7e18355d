// Device code of the rotation by a group of strip wavefronts (rotate_terms.hip has the design).
#pragma once
#include "rotate_bf16_device.h"
#include "rotate_terms.h"
#include "wave_dpp.h"

namespace {

typedef _Float16 v8h_t __attribute__((ext_vector_type(8)));

template <bool BF>
__device__ __forceinline__ v4f rt_mma(v4i a, v4i b, v4f c) {
    if constexpr (BF) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h_t, a), __builtin_bit_cast(v8h_t, b), c, 0, 0, 0);
}

// Both stages of an fp32 token on fp32 MFMA (16x16x4): a lane's four values of a 16-byte read are the contraction indices of four
// instructions, and the accumulators of stage 1 (Z[a = 4 lg + v][d = li]) are the A operands of stage 2 as they stand.  Each sum in
// the order of rotate_f32_device.h: the same values to the bit.  wait: the R1 terms have to be waited for.
template <int AT, int NB, typename Load>
__device__ __forceinline__ void rotate_terms_f32(Load ld_a, const v4i (&bh)[NB], const char* r1, v4f (&y)[AT], int n1, int n2, bool wait) {
    auto mul = [](float x, float w, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, w, c, 0, 0, 0); };
#pragma nounroll
    for (int ch = 0; ch < AT / 2; ++ch) {
        const bool two = 32 * ch + 16 < n1;             // (else the second tile is past the rows)
        v4f z0 = v4f{0.f, 0.f, 0.f, 0.f}, z1 = z0;
        v4i x0 = ld_a(ch, 0, 0), x1 = ld_a(ch, 0, 1);
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) {
            if (16 * kb < n2) {
                const v4i c0 = x0, c1 = x1;
                if (16 * (kb + 1) < n2) { x0 = ld_a(ch, kb + 1, 0); x1 = ld_a(ch, kb + 1, 1); }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    z0 = mul(__int_as_float(c0[v]), __int_as_float(bh[kb][v]), z0);
                    if (two) z1 = mul(__int_as_float(c1[v]), __int_as_float(bh[kb][v]), z1);
                }
            }
        }
        if (wait && ch == 0) bwla_lds_barrier();
        const char* rb = r1 + 2 * ch * AT * 1024;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (half == 0 || two) {
                const v4f z = half ? z1 : z0;
#pragma unroll
                for (int tc = 0; tc < AT; tc += 2) {
                    if (16 * tc < n1) {
                        const v4f w0 = *reinterpret_cast<const v4f*>(rb + (half * AT + tc) * 1024);
                        const v4f w1 = *reinterpret_cast<const v4f*>(rb + (half * AT + tc + 1) * 1024);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            y[tc] = mul(z[v], w0[v], y[tc]);
                            y[tc + 1] = mul(z[v], w1[v], y[tc + 1]);
                        }
                    }
                }
            }
        }
    }
}

// AT, K1M: the most 16-row tiles along n1 (padded to 32) and 32-deep steps along n2.  STREAM: the R1 terms of one step at a
// time (n1 > 160).  MANY: workgroups walk over their tokens, G groups of wavefronts side by side; else one token a workgroup.
template <int AT, int K1M, bool STREAM, bool MANY, RtKind KIND, int THREADS>
__global__ __launch_bounds__(THREADS) void rotate_terms_kernel(RtArgs b) {
    constexpr bool F32 = KIND == RT_F32, H16 = KIND == RT_H16, BF = KIND == RT_BF16;
    extern __shared__ __align__(16) float lds_f[];
    const RqArgs& a = b.q;
    if ((int64_t)blockIdx.x >= a.rot_blocks) {
        const int pb = (int)(blockIdx.x - a.rot_blocks);
        if constexpr (MANY) psp_sum_at(a, pb);
        else psp_block_at<!F32, !F32>(reinterpret_cast<char*>(lds_f), a, pb);
        return;
    }
    constexpr int VG = F32 ? 4 : 8, TW = BF && !MANY && K1M < 5 ? 2 : 1;       // values in 16 bytes; tiles of stage 2 side by side
    constexpr int CH2 = AT / 2, NI = CH2 * (8 / VG);    // 32-deep steps along n1; 16-byte granules of a token per thread
    char* lds = reinterpret_cast<char*>(lds_f);
    const int n1 = a.n1, n2 = a.n2, K = n1 * n2, k1 = b.s.k1, strips = b.s.strips;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nwaves = (int)blockDim.x >> 6;
    int grp = 0;
    if constexpr (MANY) {
        for (int w = wv; w >= strips && grp < b.s.G; w -= strips) ++grp;
    } else {
        grp = wv >= strips ? 1 : 0;
    }
    const int G = MANY ? b.s.G : 1;
    const bool helper = grp >= G;                       // carries R1 terms only
    const int wave = wv - grp * strips;
    const int TG = 64 * strips, tid = (int)threadIdx.x - grp * TG, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    char* r1 = lds;
    char* xt = lds + b.s.r1_bytes + grp * b.s.xt_bytes;
    char* cb = b.s.own ? lds + b.s.r1_bytes + G * b.s.xt_bytes + grp * b.s.cb_bytes : xt;
    float* red = reinterpret_cast<float*>(lds + b.s.r1_bytes + G * (b.s.xt_bytes + (b.s.own ? b.s.cb_bytes : 0))) + grp * 64;
    int* redi = reinterpret_cast<int*>(red) + 48;
    constexpr int CB = BF ? 3 * AT : 2 * AT, chunk_bytes = CB * 1024;     // blocks and bytes of a step of R1 (fp32: two rows of tiles)
    const int pitch = b.s.pitch;

    // ---- R1 terms, global -> LDS, one KiB a request.  Resident: all of them, by the wavefronts behind the groups.  STREAM: the
    // terms of step g into buffer g & 1, by all, requested while the step before is worked on.
    const int n1p16 = (n1 + 15) & ~15;
    auto r1_async = [&](int ch, int e, char* dst) {     // block e of step ch
        const int l = (int)threadIdx.x & 63;
        const uint16_t* src = b.R1h + ((ch * 2 * AT + e) * 64 + l) * 8;
        if constexpr (BF) {
            // (planes of whole rows: sixteen rows of 64 bytes make a block; there is no tile past the rows)
            const int p = e / AT, c = 16 * (e - p * AT);
            if (c >= n1p16) {
                *reinterpret_cast<v4i*>(dst + l * 16) = v4i{0, 0, 0, 0};
                return;
            }
            src = a.R1p + ((p * n1p16 + c + (l & 15)) * (CH2 * 32) + ch * 32 + (l >> 4) * 8);
        }
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    };
    auto request_chunk = [&](int g, int ch) {
        for (int e = wv; e < CB; e += G * strips) r1_async(ch, e, r1 + (g & 1) * chunk_bytes + e * 1024);
    };
    if (STREAM && helper) return;
    if (!STREAM && helper) {
        const int first = wv - G * strips, step = nwaves - G * strips;
        if constexpr (F32) {
            // block ta AT + tc: R1[a = 16 ta + 4 lg + v][c = 16 tc + li], v = 0..3, eight of them in flight
            const int l = (int)threadIdx.x & 63;
            for (int e0 = first; e0 < AT * AT; e0 += 8 * step) {
                v4f t[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = e0 + u * step < AT * AT ? e0 + u * step : e0, ta = e / AT;
                    const int row = 16 * ta + 4 * (l >> 4), c = 16 * (e - ta * AT) + (l & 15);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const bool in = row + v < n1 && c < n1;
                        const float f = a.R1[in ? (row + v) * n1 + c : 0];
                        t[u][v] = in ? f : 0.0f;
                    }
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (e0 + u * step < AT * AT) *reinterpret_cast<v4f*>(r1 + (e0 + u * step) * 1024 + l * 16) = t[u];
            }
        } else {
            for (int e = first; e < CH2 * CB; e += step) r1_async(e / CB, e % CB, r1 + e * 1024);
        }
        bwla_lds_barrier();                             // maxima
        bwla_lds_barrier();                             // token rows
        __builtin_amdgcn_s_waitcnt(0);
        bwla_lds_barrier();                             // R1 terms
        return;                                         // (the barriers behind count the wavefronts that are left)
    }

    auto my_tid = [&]() -> int {
        int x = (int)threadIdx.x;
        if constexpr (MANY) asm volatile("" : "+v"(x));
        return x - grp * TG;
    };
    // ---- the token, then the R2 terms of my strip
    const int items = K / VG;
    const int64_t tstep = a.rot_blocks * G, t0 = (int64_t)blockIdx.x * G + grp;
    v4i xpre[NI];
    auto request = [&](int64_t t) {
        const char* xrow = reinterpret_cast<const char*>(a.X) + (t < a.M ? t : a.M - 1) * K * (16 / VG);
        const int tid = my_tid();
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            const int it = tid + e * TG;                // (past the last one: the first again)
            xpre[e] = *reinterpret_cast<const v4i*>(xrow + (it < items ? it : 0) * 16);
        }
    };
    request(t0);
    constexpr int NB = F32 ? 2 * K1M : K1M;             // (fp32: R2[b = 16 kb + 4 lg + v][d] in bh[kb])
    v4i bh[NB], bl[F32 ? 1 : K1M], bx[BF ? K1M : 1];
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) {
        const int kc = kb < k1 ? kb : 0;
        if constexpr (F32) {
            const int row = 16 * kb + 4 * lg, d = 16 * wave + li;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const bool in = row + v < n2 && d < n2;
                const float f = a.R2[in ? (row + v) * n2 + d : 0];
                bh[kb][v] = __float_as_int(in ? f : 0.0f);
            }
        } else if constexpr (BF) {
            const uint16_t* src = a.R2p + ((wave * 16 + li) * (k1 * 32) + kc * 32 + 8 * lg);
            const int term = strips * 16 * k1 * 32;
            bh[kb] = *reinterpret_cast<const v4i*>(src);
            bl[kb] = *reinterpret_cast<const v4i*>(src + term);
            bx[kb] = *reinterpret_cast<const v4i*>(src + 2 * term);
        } else {
            const uint16_t* src = b.R2h + ((wave * k1 + kc) * 2 * 64 + lane) * 8;
            bh[kb] = *reinterpret_cast<const v4i*>(src);
            bl[kb] = *reinterpret_cast<const v4i*>(src + 512);
        }
    }
    if constexpr (STREAM) request_chunk(0, 0);

    // largest magnitude of the token in registers: bf16 magnitudes order like their 15 low bits
    auto token_max = [&]() -> float {
        typedef unsigned short us2 __attribute__((ext_vector_type(2)));
        us2 m = us2{0, 0};
#pragma unroll
        for (int e = 0; e < NI; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(us2, (uint32_t)xpre[e][i] & 0x7fff7fffu));
        const uint32_t top = m.x > m.y ? m.x : m.y;
        return dl_wave_max_nonneg(__uint_as_float(top << 16));
    };
    // H16: exponent field E of a token's largest magnitude: the token is scaled by 2^(129 - E), which puts that magnitude into
    // [2^2, 2^3), and what the two stages make of it by 2^(145 - E) then (256 R1, 256 R2).  Codes and zero points are the
    // same in that scale, so only the step that is stored goes back.
    auto exponent_of = [&](float xmax) -> int {
        const int E = (__float_as_int(xmax) >> 23) & 0xff;
        return E < 2 ? 2 : E;
    };
    // zeros where a token row ends inside a step along n2 (32 values; fp32: 16), and in rows past n1
    auto zero_pads = [&](int tz, int nz) {
        const int words = F32 ? ((n2 + 15) & ~15) : k1 * 16, used = F32 ? n2 : n2 >> 1, cols = words - used;
        const FastDiv dc(cols > 0 ? cols : 1);
        for (int i = tz; i < n1 * cols; i += nz) {
            const int row = dc.div(i);
            *reinterpret_cast<uint32_t*>(xt + row * pitch + 4 * (used + i - row * cols)) = 0u;
        }
        const int g = words >> 2, rows = CH2 * 32 - n1;                          // 16-byte granules
        const FastDiv dg(g);
        for (int i = tz; i < rows * g; i += nz) {
            const int row = dg.div(i);
            *reinterpret_cast<v4i*>(xt + (n1 + row) * pitch + (i - row * g) * 16) = v4i{0, 0, 0, 0};
        }
    };
    // the token in registers -> rows in LDS
    const bool whole = (n2 & (VG - 1)) == 0;
    const FastDiv drow(whole ? n2 / VG : n2 >> 1);
    auto land = [&](int E) {
        const int tid = my_tid();
        const float sx = __int_as_float((256 - E) << 23);
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            const int it = tid + e * TG;
            v4i o = xpre[e];
#pragma unroll
            for (int i = 0; H16 && i < 4; ++i) {
                const uint32_t w = (uint32_t)xpre[e][i];
                o[i] = __builtin_bit_cast(int, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w << 16) * sx, __uint_as_float(w & 0xffff0000u) * sx));
            }
            if (it < items) {
                if (whole) {
                    const int row = drow.div(it), g = it - row * (n2 / VG);
                    *reinterpret_cast<v4i*>(xt + row * pitch + g * 16) = o;
                } else {
                    // pairs of values: n2 is even
                    constexpr int PAIRS = VG / 2, W = 4 / PAIRS;                 // of 16 bytes; words of one
#pragma unroll
                    for (int i = 0; i < PAIRS; ++i) {
                        const int p = it * PAIRS + i, row = drow.div(p);
                        char* to = xt + row * pitch + (p - row * (n2 >> 1)) * (4 * W);
                        if constexpr (W == 1) *reinterpret_cast<int*>(to) = o[i];
                        else *reinterpret_cast<int2*>(to) = int2{o[2 * i], o[2 * i + 1]};
                    }
                }
            }
        }
    };
    const bool pads = (n2 & (F32 ? 15 : 31)) != 0 || (n1 & 31) != 0;
    if (pads) zero_pads(tid, TG);
    if constexpr (H16) {
        const float m = token_max();
        if (lane == 0) red[32 + wave] = m;
    }
    bwla_lds_barrier();
    // (a word a lane of a row of sixteen, at most ten strips)
    auto over_strips = [&](const float* p) -> float {
        const int w = (int)threadIdx.x & 15;
        return dl_wave_max_nonneg(w < strips ? p[w] : 0.0f);
    };
    int E = 145;
    if constexpr (H16) E = exponent_of(over_strips(red + 32));
    land(E);
    if constexpr (MANY) {
        if (b.rounds > 1) request(t0 + tstep);
    }
    bwla_lds_barrier();

    // the codes of token t from LDS to memory, in whole lines
    auto write_codes = [&](int64_t t) {
        int8_t* qrow = a.q + t * K;
#pragma nounroll
        for (int it = my_tid(); it < (K >> 4); it += TG) *reinterpret_cast<v4i*>(qrow + it * 16) = *reinterpret_cast<const v4i*>(cb + it * 16);
    };
    const int rounds = MANY ? b.rounds : 1;
#pragma nounroll
    for (int j = 0; j < rounds; ++j) {
        const int64_t t = t0 + (int64_t)j * tstep;
        const bool live = !MANY || t < a.M;
        if (MANY && b.s.own && j > 0 && t - tstep < a.M) write_codes(t - tstep);
        // (lane-derived values anew each round, from an opaque copy: every address of the body would be kept in registers else)
        int lane_o = (int)threadIdx.x & 63;
        if constexpr (MANY) asm volatile("" : "+v"(lane_o));
        const int lane = lane_o, li = lane & 15, lg = lane >> 4;
        v4f y[AT];
#pragma unroll
        for (int tc = 0; tc < AT; ++tc) y[tc] = v4f{0.f, 0.f, 0.f, 0.f};
        const char* xa = xt + li * pitch + lg * 16;
        auto ld_a = [&](int ch, int kb, int half) -> v4i {
            return *reinterpret_cast<const v4i*>(xa + (32 * ch + 16 * half) * pitch + kb * 64);
        };
        if constexpr (F32) rotate_terms_f32<AT, NB>(ld_a, bh, r1 + lane * 16, y, n1, n2, j == 0);
        v4i n0 = ld_a(0, 0, 0), n1_ = ld_a(0, 0, 1);
#pragma nounroll
        for (int ch = 0; !F32 && ch < CH2; ++ch) {
            v4f z0 = v4f{0.f, 0.f, 0.f, 0.f}, z1 = z0;
            v4i qa0[K1M + 1], qa1[K1M + 1], qb[3][AT];
            qa0[0] = n0; qa1[0] = n1_;
            if (k1 > 1) { qa0[1] = ld_a(ch, 1, 0); qa1[1] = ld_a(ch, 1, 1); }
#pragma unroll
            for (int kb = 0; kb < K1M; ++kb) {
                if (kb < k1) {
                    const v4i a0 = qa0[kb], a1 = qa1[kb];
                    if (kb + 2 < K1M && kb + 2 < k1) { qa0[kb + 2] = ld_a(ch, kb + 2, 0); qa1[kb + 2] = ld_a(ch, kb + 2, 1); }
                    if constexpr (BF) {                                          // small terms first
                        z0 = rt_mma<BF>(a0, bx[kb], z0);
                        z1 = rt_mma<BF>(a1, bx[kb], z1);
                    }
                    if constexpr (!F32) {
                        z0 = rt_mma<BF>(a0, bl[kb], z0);
                        z1 = rt_mma<BF>(a1, bl[kb], z1);
                        z0 = rt_mma<BF>(a0, bh[kb], z0);
                        z1 = rt_mma<BF>(a1, bh[kb], z1);
                    }
                }
            }
            const char* rb;
            if constexpr (STREAM) {
                // this step's R1 terms have landed, everybody's share; the other buffer is free (all are past the step
                // before): the next step's terms go there while this one is worked on
                const int g = j * CH2 + ch;
                __builtin_amdgcn_s_waitcnt(0);
                bwla_lds_barrier();
                if (ch + 1 < CH2) request_chunk(g + 1, ch + 1);
                else if (j + 1 < rounds) request_chunk(g + 1, 0);
                rb = r1 + (g & 1) * chunk_bytes + lane * 16;
            } else {
                if (j == 0 && ch == 0) bwla_lds_barrier();                       // the R1 terms are there
                rb = r1 + ch * chunk_bytes + lane * 16;
            }
            auto ld_b = [&](int tc) {
#pragma unroll
                for (int p = 0; p < (BF ? 3 : 2); ++p) qb[p][tc] = *reinterpret_cast<const v4i*>(rb + (p * AT + tc) * 1024);
            };
#pragma unroll
            for (int u = 0; u < TW; ++u) ld_b(u);
            // lane (li, lg) holds Z[a = 32 ch + 4 lg + v (z0), 32 ch + 16 + 4 lg + v (z1)][d = li]: the eight contraction
            // positions of an A operand, in the order the R1 terms were stored in
            v4i ah, al, ax;
            if constexpr (BF) {
                const float f[8] = {z0[0], z0[1], z0[2], z0[3], z1[0], z1[1], z1[2], z1[3]};
                v8bf h1, h2, h3;
                r3_split3(f, h1, h2, h3);
                ah = __builtin_bit_cast(v4i, h1); al = __builtin_bit_cast(v4i, h2); ax = __builtin_bit_cast(v4i, h3);
            } else {
                v8h_t h1, h2;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float f = e < 4 ? z0[e & 3] : z1[e & 3];
                    const _Float16 h = (_Float16)f;
                    h1[e] = h;
                    h2[e] = (_Float16)__builtin_fmaf((float)h, -1.0f, f);
                }
                ah = __builtin_bit_cast(v4i, h1); al = __builtin_bit_cast(v4i, h2);
            }
            const int cn = ch + 1 < CH2 ? ch + 1 : 0;
            n0 = ld_a(cn, 0, 0); n1_ = ld_a(cn, 0, 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int tc = 0; tc < AT; tc += TW) {       // (the products of TW tiles in turn: those of one wait for each other)
                if (tc + TW < AT) {
#pragma unroll
                    for (int u = 0; u < TW; ++u) ld_b(tc + TW + u);
                }
                auto mul = [&](v4i x, int p) {
#pragma unroll
                    for (int u = 0; u < TW; ++u) y[tc + u] = rt_mma<BF>(x, qb[p][tc + u], y[tc + u]);
                };
                if constexpr (BF) {                     // small ones first
                    mul(ax, 0);
                    mul(ah, 2);
                    mul(al, 1);
                }
                mul(al, 0);
                mul(ah, 1);
                mul(ah, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // ---- the token's range (padded rows and columns are exact zeros); the next token's largest value
        float mx = 0.0f, mn = 0.0f;
        if (a.asym) {
#pragma unroll
            for (int tc = 0; tc < AT; ++tc)
#pragma unroll
                for (int v = 0; v < 4; ++v) { mx = fmaxf(mx, y[tc][v]); mn = fminf(mn, y[tc][v]); }
            mx = dl_wave_max_nonneg(mx);
            mn = dl_wave_max_nonneg(-mn);
        } else {
#pragma unroll
            for (int tc = 0; tc < AT; ++tc)
#pragma unroll
                for (int v = 0; v < 4; ++v) mx = fmaxf(mx, fabsf(y[tc][v]));
            mx = dl_wave_max_nonneg(mx);
            mn = mx;
        }
        if (lane == 0) { red[wave] = mx; red[16 + wave] = mn; }
        if constexpr (MANY) {
            if (H16 && j + 1 < rounds) {
                const float nm = token_max();
                if (lane == 0) red[32 + wave] = nm;
            }
        }
        bwla_lds_barrier();                             // also: everybody is done with the token rows
        const float hi = over_strips(red), lo = -over_strips(red + 16);
        float xmax = 0.0f;
        if constexpr (MANY && H16) xmax = over_strips(red + 32);
        const QuantPlan qp = quant_plan(hi, lo, a.qmax, a.asym != 0);
        // ---- codes, to LDS in k order.  Lane holds Yt[d = 16 strip + 4 lg + v][c = 16 tc + li]: four consecutive k.
        // The integer next to y * inv (ties to even) plus 1.5 * 2^23 and the zero point, clamped as a float, has the code in its
        // low byte.  (H16: one rounding for the product and the sum, as in rotate_planes.hip; else quant_code's two.)
        const float inv = qp.inv, addc = 12582912.0f + qp.zc;
        const float cmin = 12582912.0f + qp.cmin, cmax = 12582912.0f + qp.cmax;
        int lsum = 0;
        const int d0 = 16 * wave + 4 * lg;
        const bool words = (n2 & 3) == 0;
#pragma unroll
        for (int tc = 0; tc < AT; ++tc) {
            const int c = 16 * tc + li;
            {
                uint32_t c4[4];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    c4[v] = __float_as_uint(__builtin_amdgcn_fmed3f(H16 ? __builtin_fmaf(y[tc][v], inv, addc) : rintf(y[tc][v] * inv) + addc,
                                                                    cmin, cmax));
                const uint32_t wlo = __builtin_amdgcn_perm(c4[1], c4[0], 0x0c0c0400u);     // bytes: c4[0], c4[1], 0, 0
                const uint32_t whi = __builtin_amdgcn_perm(c4[3], c4[2], 0x04000c0cu);     // bytes: 0, 0, c4[2], c4[3]
                uint32_t word = wlo | whi;
                if (c < n1 && d0 < n2) {
                    char* p = cb + c * n2 + d0;
                    if (words) {
                        *reinterpret_cast<uint32_t*>(p) = word;
                    } else {
                        *reinterpret_cast<uint16_t*>(p) = (uint16_t)word;
                        if (d0 + 2 < n2) *reinterpret_cast<uint16_t*>(p + 2) = (uint16_t)(word >> 16);
                        else word &= 0xffffu;
                    }
                    lsum = __builtin_amdgcn_sdot4((int)word, 0x01010101, lsum, false);
                }
            }
        }
        lsum = dl_wave_sum(lsum);
        if (lane == 0) redi[wave] = lsum;
        float sc = quant_scale(hi, lo, a.qmax, a.asym != 0);
        if constexpr (H16) sc = ldexpf(sc, E - 145);
        if constexpr (MANY) {
            if (!b.s.own) {                             // the codes lie where the next token goes: out first
                bwla_lds_barrier();
                if (live) write_codes(t);
                bwla_lds_barrier();
            }
            if (j + 1 < rounds) {
                if constexpr (H16) E = exponent_of(xmax);
                if (pads && !b.s.own) zero_pads(tid, TG);
                land(E);
                if (j + 2 < rounds) request(t + 2 * tstep);
            }
        }
        bwla_lds_barrier();
        if constexpr (!MANY) write_codes(t);
        if (wave == 0 && live) {
            const int tot = dl_wave_sum(lane < strips ? redi[lane] : 0);
            if (lane == 0) {
                a.qsum[t] = tot;
                a.scale[t] = sc;
                quant_extras(a.tmode, a.tp, t, a.asym != 0, a.shift != 0, qp, sc, tot, K);
            }
        }
    }
    if constexpr (MANY) {
        const int64_t tl = t0 + (int64_t)(rounds - 1) * tstep;
        if (b.s.own && tl < a.M) write_codes(tl);
    }
}

template <int AT, int K1M, bool STREAM, bool MANY, RtKind KIND, int THREADS>
hipError_t launch_v(const RtArgs& b, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    if (threads > THREADS) return hipErrorInvalidValue;
    const auto kern = rotate_terms_kernel<AT, K1M, STREAM, MANY, KIND, THREADS>;
    hipError_t e = bwla_ensure_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    kern<<<dim3((unsigned)blocks), dim3((unsigned)threads), lds, st>>>(b);
    return hipGetLastError();
}

// (k1: the shape's; the kernel's is at least as large)
template <bool MANY>
hipError_t launch_terms(const RtArgs& b, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    const RtShape& s = b.s;
#define RT_STREAM(A) if (s.stream && s.at == A) return launch_v<A, 4, true, MANY, RT_BF16, 512>(b, blocks, threads, lds, st);
    RT_STREAM(10) RT_STREAM(12) RT_STREAM(14) RT_STREAM(16)
#undef RT_STREAM
#define RT_CASE(A)                                                                                         \
    if (s.at == A) return s.k1 <= 2   ? launch_v<A, 2, false, MANY, RT_BF16, MANY || A >= 8 ? 768 : 512>(b, blocks, threads, lds, st) \
                          : s.k1 <= 3 ? launch_v<A, 3, false, MANY, RT_BF16, MANY || A >= 8 ? 768 : 512>(b, blocks, threads, lds, st) \
                                      : launch_v<A, 5, false, MANY, RT_BF16, 768>(b, blocks, threads, lds, st);
    RT_CASE(2) RT_CASE(4) RT_CASE(6) RT_CASE(8)
#undef RT_CASE
    return hipErrorInvalidValue;
}
template <bool MANY>
hipError_t launch_terms_f32(const RtArgs& b, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    const RtShape& s = b.s;
#define RT_CASE(A)                                                                                         \
    if (s.at == A) return s.k1 <= 2 ? launch_v<A, 2, false, MANY, RT_F32, MANY || A >= 8 ? 768 : 512>(b, blocks, threads, lds, st) \
                                    : launch_v<A, 3, false, MANY, RT_F32, MANY || A >= 8 ? 768 : 512>(b, blocks, threads, lds, st);
    RT_CASE(2) RT_CASE(4) RT_CASE(6) RT_CASE(8)
#undef RT_CASE
    return hipErrorInvalidValue;
}

}  // namespace
