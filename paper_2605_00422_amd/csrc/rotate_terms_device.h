// Device code of the rotation on two fp16 terms (rotate_terms.hip has the design).
#pragma once
#include "rotate_terms.h"
#include "wave_dpp.h"

namespace {

typedef _Float16 v8h_t __attribute__((ext_vector_type(8)));

// AT, K1M: the most 16-row tiles along n1 (padded to 32) and 32-deep steps along n2.  STREAM: the R1 terms of one step at a
// time (n1 > 160).  MANY: workgroups walk over their tokens, G groups of wavefronts side by side; else one token a workgroup.
template <int AT, int K1M, bool STREAM, bool MANY, int THREADS>
__global__ __launch_bounds__(THREADS) void rotate_terms_kernel(RtArgs b) {
    extern __shared__ __align__(16) float lds_f[];
    const RqArgs& a = b.q;
    if ((int64_t)blockIdx.x >= a.rot_blocks) {
        const int pb = (int)(blockIdx.x - a.rot_blocks);
        if constexpr (MANY) psp_sum_at(a, pb);
        else psp_block_at<true, true>(reinterpret_cast<char*>(lds_f), a, pb);
        return;
    }
    // (the small terms of a product are added up apart where registers allow: fewer roundings at the sum's own magnitude)
    constexpr bool APART = AT <= 4 || (AT <= 8 && K1M <= 3 && !MANY);
    constexpr bool LOLO = AT <= 4;
    constexpr int NI = AT / 2, CH2 = AT / 2;            // 16-byte granules of a token per thread; 32-deep steps along n1
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
    constexpr int chunk_bytes = 2 * AT * 1024;
    const int pitch = b.s.pitch;

    // ---- R1 terms, global -> LDS, one KiB a request.  Resident: all of them, by the wavefronts behind the groups.  STREAM: the
    // terms of step g into buffer g & 1, by all, requested while the step before is worked on.
    auto r1_async = [&](int block, char* dst) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(b.R1h + (block * 64 + (int)(threadIdx.x & 63)) * 8),
                                         (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    };
    auto request_chunk = [&](int g, int ch) {
        for (int e = wv; e < 2 * AT; e += G * strips) r1_async(ch * 2 * AT + e, r1 + (g & 1) * chunk_bytes + e * 1024);
    };
    if (STREAM && helper) return;
    if (!STREAM && helper) {
        const int first = wv - G * strips, step = nwaves - G * strips;
        for (int e = first; e < CH2 * 2 * AT; e += step) r1_async(e, r1 + e * 1024);
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
    const int items = K >> 3;
    const int64_t tstep = a.rot_blocks * G, t0 = (int64_t)blockIdx.x * G + grp;
    v4i xpre[NI];
    auto request = [&](int64_t t) {
        const uint16_t* xrow = reinterpret_cast<const uint16_t*>(a.X) + (t < a.M ? t : a.M - 1) * K;
        const int tid = my_tid();
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            const int it = tid + e * TG;                // (past the last one: the first again)
            xpre[e] = *reinterpret_cast<const v4i*>(xrow + (it < items ? it : 0) * 8);
        }
    };
    request(t0);
    v8h_t bh[K1M], bl[K1M];
#pragma unroll
    for (int kb = 0; kb < K1M; ++kb) {
        const int kc = kb < k1 ? kb : 0;
        bh[kb] = __builtin_bit_cast(v8h_t, *reinterpret_cast<const v4i*>(b.R2h + (((wave * k1 + kc) * 2 + 0) * 64 + lane) * 8));
        bl[kb] = __builtin_bit_cast(v8h_t, *reinterpret_cast<const v4i*>(b.R2h + (((wave * k1 + kc) * 2 + 1) * 64 + lane) * 8));
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
    // power of two that puts a token's largest magnitude into [2^2, 2^3) (1 for an all-zero token)
    auto scale_of = [&](float xmax) -> float {
        int E = (__float_as_int(xmax) >> 23) & 0xff;
        E = E < 40 ? 40 : (E > 230 ? 230 : E);
        return xmax > 0.0f ? __int_as_float((127 + 2 + 127 - E) << 23) : 1.0f;
    };
    // zeros where a token row ends inside a 32-deep step, and in rows past n1
    auto zero_pads = [&](int tz, int nz) {
        const int cols = (k1 * 32 - n2) >> 1, prow = cols > 0 ? n1 : 0;          // words
        const FastDiv dc(cols > 0 ? cols : 1);
        for (int i = tz; i < prow * cols; i += nz) {
            const int row = dc.div(i);
            *reinterpret_cast<uint32_t*>(xt + row * pitch + 2 * n2 + 4 * (i - row * cols)) = 0u;
        }
        const int g = k1 * 4, rows = CH2 * 32 - n1;                              // 16-byte granules
        const FastDiv dg(g);
        for (int i = tz; i < rows * g; i += nz) {
            const int row = dg.div(i);
            *reinterpret_cast<v4i*>(xt + (n1 + row) * pitch + (i - row * g) * 16) = v4i{0, 0, 0, 0};
        }
    };
    // the token in registers -> fp16 rows in LDS, scaled by sx = 2^ex
    const bool whole = (n2 & 7) == 0;
    const FastDiv drow(whole ? n2 >> 3 : n2 >> 1);
    auto land = [&](float sx) {
        const int tid = my_tid();
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            {
                const int it = tid + e * TG;
                v4i o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = (uint32_t)xpre[e][i];
                    o[i] = __builtin_bit_cast(int, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w << 16) * sx, __uint_as_float(w & 0xffff0000u) * sx));
                }
                if (it < items) {
                    if (whole) {
                        const int row = drow.div(it), g = it - row * (n2 >> 3);
                        *reinterpret_cast<v4i*>(xt + row * pitch + g * 16) = o;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {                            // pairs of values: n2 is even
                            const int p = it * 4 + i, row = drow.div(p);
                            *reinterpret_cast<int*>(xt + row * pitch + (p - row * (n2 >> 1)) * 4) = o[i];
                        }
                    }
                }
            }
        }
    };
    const bool pads = (n2 & 31) != 0 || (n1 & 31) != 0;
    if (pads) zero_pads(tid, TG);
    {
        const float m = token_max();
        if (lane == 0) red[32 + wave] = m;
    }
    bwla_lds_barrier();
    // (a word a lane of a row of sixteen, at most ten strips)
    auto over_strips = [&](const float* p) -> float {
        const int w = (int)threadIdx.x & 15;
        return dl_wave_max_nonneg(w < strips ? p[w] : 0.0f);
    };
    float sx = scale_of(over_strips(red + 32));
    land(sx);
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
        v4f y[AT], ys[APART ? AT : 1];
#pragma unroll
        for (int tc = 0; tc < AT; ++tc) y[tc] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tc = 0; tc < (APART ? AT : 1); ++tc) ys[tc] = v4f{0.f, 0.f, 0.f, 0.f};
        const char* xa = xt + li * pitch + lg * 16;
        auto ld_a = [&](int ch, int kb, int half) -> v4i {
            return *reinterpret_cast<const v4i*>(xa + (32 * ch + 16 * half) * pitch + kb * 64);
        };
        v4i n0 = ld_a(0, 0, 0), n1_ = ld_a(0, 0, 1);
#pragma nounroll
        for (int ch = 0; ch < CH2; ++ch) {
            v4f z0 = v4f{0.f, 0.f, 0.f, 0.f}, z1 = z0, s0 = z0, s1 = z0;
            v4i qa0[K1M + 1], qa1[K1M + 1], qb[2][AT];
            qa0[0] = n0; qa1[0] = n1_;
            if (k1 > 1) { qa0[1] = ld_a(ch, 1, 0); qa1[1] = ld_a(ch, 1, 1); }
#pragma unroll
            for (int kb = 0; kb < K1M; ++kb) {
                if (kb < k1) {
                    const v8h_t a0 = __builtin_bit_cast(v8h_t, qa0[kb]), a1 = __builtin_bit_cast(v8h_t, qa1[kb]);
                    if (kb + 2 < K1M && kb + 2 < k1) { qa0[kb + 2] = ld_a(ch, kb + 2, 0); qa1[kb + 2] = ld_a(ch, kb + 2, 1); }
                    if constexpr (APART) {
                        s0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, bl[kb], s0, 0, 0, 0);
                        s1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, bl[kb], s1, 0, 0, 0);
                    } else {
                        z0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, bl[kb], z0, 0, 0, 0);      // small term first
                        z1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, bl[kb], z1, 0, 0, 0);
                    }
                    z0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, bh[kb], z0, 0, 0, 0);
                    z1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, bh[kb], z1, 0, 0, 0);
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
            qb[0][0] = *reinterpret_cast<const v4i*>(rb);
            qb[1][0] = *reinterpret_cast<const v4i*>(rb + AT * 1024);
            // lane (li, lg) holds Z[a = 32 ch + 4 lg + v (z0), 32 ch + 16 + 4 lg + v (z1)][d = li]: the eight contraction
            // positions of an A operand, in the order the R1 terms were stored in
            v8h_t ah, al;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float f = APART ? (e < 4 ? z0[e & 3] + s0[e & 3] : z1[e & 3] + s1[e & 3]) : (e < 4 ? z0[e & 3] : z1[e & 3]);
                const _Float16 h = (_Float16)f;
                ah[e] = h;
                al[e] = (_Float16)__builtin_fmaf((float)h, -1.0f, f);
            }
            const int cn = ch + 1 < CH2 ? ch + 1 : 0;
            n0 = ld_a(cn, 0, 0); n1_ = ld_a(cn, 0, 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int tc = 0; tc < AT; ++tc) {
                {
                    const v8h_t ch_ = __builtin_bit_cast(v8h_t, qb[0][tc]), cl_ = __builtin_bit_cast(v8h_t, qb[1][tc]);
                    if (tc + 1 < AT) {                 // (a tile past the last one reads what lies behind; never used)
                        qb[0][tc + 1] = *reinterpret_cast<const v4i*>(rb + (tc + 1) * 1024);
                        qb[1][tc + 1] = *reinterpret_cast<const v4i*>(rb + (AT + tc + 1) * 1024);
                    }
                    v4f& small = APART ? ys[tc] : y[tc];
                    if constexpr (LOLO) small = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, cl_, small, 0, 0, 0);
                    small = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, ch_, small, 0, 0, 0);
                    small = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, cl_, small, 0, 0, 0);
                    y[tc] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, ch_, y[tc], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if constexpr (APART) {
#pragma unroll
            for (int tc = 0; tc < AT; ++tc) y[tc] += ys[tc];
        }
        // ---- the token's range (padded rows and columns are exact zeros); the next token's largest value
        const float yun = 1.52587890625e-05f / sx;      // back from 256 R2, 256 R1 and the token's scale
        float mx = 0.0f, mn = 0.0f;
        if (a.asym) {
#pragma unroll
            for (int tc = 0; tc < AT; ++tc)
#pragma unroll
                for (int v = 0; v < 4; ++v) { mx = fmaxf(mx, y[tc][v]); mn = fminf(mn, y[tc][v]); }
            mx = dl_wave_max_nonneg(mx) * yun;
            mn = dl_wave_max_nonneg(-mn) * yun;
        } else {
#pragma unroll
            for (int tc = 0; tc < AT; ++tc)
#pragma unroll
                for (int v = 0; v < 4; ++v) mx = fmaxf(mx, fabsf(y[tc][v]));
            mx = dl_wave_max_nonneg(mx) * yun;
            mn = mx;
        }
        if (lane == 0) { red[wave] = mx; red[16 + wave] = mn; }
        if constexpr (MANY) {
            if (j + 1 < rounds) {
                const float nm = token_max();
                if (lane == 0) red[32 + wave] = nm;
            }
        }
        bwla_lds_barrier();                             // also: everybody is done with the token rows
        const float hi = over_strips(red), lo = -over_strips(red + 16);
        float xmax = 0.0f;
        if constexpr (MANY) xmax = over_strips(red + 32);
        const QuantPlan qp = quant_plan(hi, lo, a.qmax, a.asym != 0);
        // ---- codes, to LDS in k order.  Lane holds Yt[d = 16 strip + 4 lg + v][c = 16 tc + li]: four consecutive k.
        // y * inv + (1.5 * 2^23 + zero point) rounds once, to an integer (ties to even) in the low mantissa bits; clamped as a
        // float, its low byte is the code.
        const float inv = qp.inv * yun, addc = 12582912.0f + qp.zc;
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
                    c4[v] = __float_as_uint(__builtin_amdgcn_fmed3f(__builtin_fmaf(y[tc][v], inv, addc), cmin, cmax));
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
        if constexpr (MANY) {
            if (!b.s.own) {                             // the codes lie where the next token goes: out first
                bwla_lds_barrier();
                if (live) write_codes(t);
                bwla_lds_barrier();
            }
            if (j + 1 < rounds) {
                sx = scale_of(xmax);
                if (pads && !b.s.own) zero_pads(tid, TG);
                land(sx);
                if (j + 2 < rounds) request(t + 2 * tstep);
            }
        }
        bwla_lds_barrier();
        if constexpr (!MANY) write_codes(t);
        if (wave == 0 && live) {
            const int tot = dl_wave_sum(lane < strips ? redi[lane] : 0);
            if (lane == 0) {
                a.qsum[t] = tot;
                const float sc = quant_scale(hi, lo, a.qmax, a.asym != 0);
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

template <int AT, int K1M, bool STREAM, bool MANY, int THREADS>
hipError_t launch_v(const RtArgs& b, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    if (threads > THREADS) return hipErrorInvalidValue;
    const auto kern = rotate_terms_kernel<AT, K1M, STREAM, MANY, THREADS>;
    hipError_t e = bwla_ensure_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    kern<<<dim3((unsigned)blocks), dim3((unsigned)threads), lds, st>>>(b);
    return hipGetLastError();
}

// (k1, at: the shape's, the kernels' are at least as large)
template <bool MANY>
hipError_t launch_terms(const RtArgs& b, int64_t blocks, int threads, size_t lds, hipStream_t st) {
    const RtShape& s = b.s;
#define RT_STREAM(A) if (s.stream && s.at == A) return launch_v<A, 4, true, MANY, 512>(b, blocks, threads, lds, st);
    RT_STREAM(12) RT_STREAM(14) RT_STREAM(16)
#undef RT_STREAM
#define RT_CASE(A)                                                                                         \
    if (s.at == A) return s.k1 <= 2   ? launch_v<A, 2, false, MANY, MANY ? 768 : 512>(b, blocks, threads, lds, st) \
                          : s.k1 <= 3 ? launch_v<A, 3, false, MANY, MANY ? 768 : 512>(b, blocks, threads, lds, st) \
                                      : launch_v<A, 5, false, MANY, 768>(b, blocks, threads, lds, st);
    RT_CASE(2) RT_CASE(4) RT_CASE(6) RT_CASE(8) RT_CASE(10)
#undef RT_CASE
    return hipErrorInvalidValue;
}

}  // namespace
