// Epilogue of the streaming GEMMs for token batches:
//
//   Y[t,n] = scale_t * alpha_n * acc[t,n] + sum_j T[t,j] V[n,j]       (paper Eq. 4; Sec. 3.2)
//
// or, gated, h[t,i] = silu(Y[t,2i]) * Y[t,2i+1] as bf16.
//
// Low-rank term on fp16 MFMA 32x32x16: V is stored in fp16 and is an operand as it stands; a token's row of T is scaled
// by a power of two 2^k (largest entry near 2^13) and split into two fp16 terms, T 2^k = hi + lo to 2^-22: two products
// per 16 ranks and channel tile.  The main term is formed first, times 2^k of its row, the MFMAs add the low-rank
// products onto it, and 2^-k is applied at the store (powers of two: exact).
//
// What bounds it is a wavefront by itself: instructions one after the other, 4 to 5 cycles each, and requests to memory
// that nothing hides.  So nothing is done twice and every request is of whole lines: T is fetched row by row, split once
// for the workgroup and left in LDS as operands (fetched by each wavefront in operand order, 16 bytes of 32 rows a request,
// its first loads alone took 2000 to 4000 cycles, and twice that when they were asked for at once: lines that are on their
// way are asked for again); V comes as the contiguous rows of a tile; a tile leaves through LDS as 16-byte stores of whole
// rows.  Cycles behind the loop (workgroups of 48000 to 77000 in all), rank 64, before and after: 64 x 128 tiles 22100 and
// 11000, 64 x 256 27600 and 19000, 64 x 64 with K in two 25600 and 12700.  Whole launches: 64 tokens of 8192 columns, 28672
// channels, rank 64 28.1 -> 23.7 us; 257 tokens, 8192 channels 34.8 -> 30.2; 333 of 4096, 11008 channels, rank 32 31.1 ->
// 25.8; 64 of 4096, 4096 channels 13.3 -> 8.7; 4096 of 28672, 8192 channels 663 -> 647.  And nothing waits behind a branch:
// a store under a condition is one, and so is a look at acc_out for every value; with the reads of a tile's rows each behind the
// store before, and the branches for sums that nobody asked for, wide tiles of low ranks were slower than with stores straight
// from registers (806 tokens of 512 columns, 11140 channels, rank 16, 64 x 640 tiles 22.6, 25.9 us; now 21.3; 385 of 1408,
// 21018, rank 0 26.8, 31.0, 28.1; rank 64, 64 tokens of 8192, 28672 channels 25.3 -> 24.4, 257 of 8192, 8192 30.9 -> 30.0, 2048 of
// 25600, 5120 193.4 -> 187.7).  Taken back: a loop over tiles out
// of LDS (less code; its round trips come one after the other: 25.5 -> 27.9 us in the first of these); the weights as the
// first MFMA operand, so that a lane holds one token (0.5 us less for a single tile, but long products run 8 % slower: the
// matrix cores' power is the limit there, and the operand that changes from one MFMA to the next costs more on that side).
#pragma once

#include "bwla_internal.h"
#include "gemm_tiles.h"

namespace {

typedef _Float16 ep_v8h __attribute__((ext_vector_type(8)));
typedef _Float16 ep_v4h __attribute__((ext_vector_type(4)));

struct EpArgs {
    const float* scale; const int32_t* qsum; const __half* alpha; const __half* V; const float* T; int r;
    float* Y; int M, N; int32_t* acc_out; uint16_t* H;
};
constexpr int EP_JC = 4;                                         // steps of 16 ranks at a time

// The rows of T of a workgroup's tokens as MFMA operands in LDS: [token / 32][16 ranks][hi, lo][lane][8] fp16, and behind
// them, for each token, 2^k scale, 2^-k and the code sum.
template <int THREADS, int TOKENS>
struct EpRows {
    static constexpr int TPT = THREADS / TOKENS, MAXP = 4 * (BWLA_MAX_RANK / 16) / TPT;     // threads a token; 4-rank pieces a thread
    const EpArgs& e;
    const int tid, token, part, JT;
    float x[MAXP][4], sc;
    int qs;
    __device__ __forceinline__ EpRows(const EpArgs& e_, int tid_)
        : e(e_), tid(tid_), token(tid_ / TPT), part(tid_ % TPT), JT((e_.r + 15) >> 4) {}
    __device__ __forceinline__ void request(int m_base) {
        const int t = m_base + token < e.M ? m_base + token : e.M - 1;
        sc = e.scale[t];
        qs = e.qsum != nullptr ? e.qsum[t] : 0;
        if (JT == 0) return;
        const float* row = e.T + (int64_t)t * e.r;
        if ((e.r & 3) == 0) {
#pragma unroll
            for (int i = 0; i < MAXP; ++i)
                if (i * TPT < 4 * JT) {
                    const int k = 4 * (part + TPT * i);
                    const float4 v = *reinterpret_cast<const float4*>(row + (k < e.r ? k : 0));
                    x[i][0] = v.x; x[i][1] = v.y; x[i][2] = v.z; x[i][3] = v.w;
                }
        } else {
#pragma unroll
            for (int i = 0; i < MAXP; ++i)
                if (i * TPT < 4 * JT) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int k = 4 * (part + TPT * i) + c;
                        x[i][c] = row[k < e.r ? k : 0];
                    }
                }
        }
    }
    __device__ __forceinline__ void put(char* lds) {
        float tmax = 0.0f;                                       // the row's largest magnitude
#pragma unroll
        for (int i = 0; i < MAXP; ++i)
            if (i * TPT < 4 * JT) {
#pragma unroll
                for (int c = 0; c < 4; ++c) tmax = fmaxf(tmax, fabsf(x[i][c]));         // (past the rank: the row's first entries)
            }
#pragma unroll
        for (int d = 1; d < TPT; d *= 2) tmax = fmaxf(tmax, __shfl_xor(tmax, d, 64));
        int kexp = 0;
        if (tmax > 0.0f && tmax < 3.0e38f) kexp = 13 + 127 - (int)(__float_as_uint(tmax) >> 23);
        kexp = kexp > 60 ? 60 : (kexp < -60 ? -60 : kexp);
        const float up = __int_as_float((127 + kexp) << 23);
        char* to = lds + (token >> 5) * (JT * 2048) + (token & 31) * 16;
#pragma unroll
        for (int i = 0; i < MAXP; ++i)
            if (i * TPT < 4 * JT) {
                const int p = part + TPT * i;                    // ranks 4 p .. 4 p + 3
                ep_v4h hi, lo;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float v = 4 * p + c < e.r ? x[i][c] * up : 0.0f;
                    hi[c] = (_Float16)v;
                    lo[c] = (_Float16)(v - (float)hi[c]);
                }
                char* at = to + (p >> 2) * 2048 + ((p >> 1) & 1) * 512 + (p & 1) * 8;
                *reinterpret_cast<ep_v4h*>(at) = hi;
                *reinterpret_cast<ep_v4h*>(at + 1024) = lo;
            }
        if (part == 0) {
            float* info = reinterpret_cast<float*>(lds + TOKENS * 64 * JT);
            info[token] = sc * up;
            info[TOKENS + token] = __int_as_float((127 - kexp) << 23);
            info[2 * TOKENS + token] = __int_as_float(qs);
        }
    }
};

// A wavefront's MT x NT tiles of 32 tokens x 32 channels, sums u in registers (acc = 2 u - qsum): element v of lane
// (l32, lg) is channel l32 of token 8 (v / 4) + 4 lg + v % 4.
template <int MT, int NT, bool GATED>
struct Epilogue {
    const EpArgs& e;
    const int mrow0, n_base, lane, l32, lg, JT;
    char* const mine;                                            // 4 KiB of LDS, the wavefront's own
    const char* const rows_t;                                    // EpRows' operands ...
    const float* const info;                                     // ... and numbers of this wavefront's first row of tiles
    v4i vf[EP_JC];
    float al[NT];

    __device__ __forceinline__ Epilogue(const EpArgs& e_, int m_base, int mt0, int n_base_, int lane_, char* mine_, const char* t_)
        : e(e_), mrow0(m_base + mt0 * 32), n_base(n_base_), lane(lane_), l32(lane_ & 31), lg(lane_ >> 5), JT((e_.r + 15) >> 4),
          mine(mine_), rows_t(t_ + mt0 * (((e_.r + 15) >> 4) * 2048)),
          info(reinterpret_cast<const float*>(t_ + ((e_.r + 15) >> 4) * 4096) + mt0 * 32) {}

    // The rows of V of 32 channels lie one behind the other, and 64 j + lane counts their 16-byte pieces: whole lines a
    // request.  (Of longer rows, eight pieces a channel at a time.)
    __device__ __forceinline__ void load_v(int nt, int c0) {
        const int n0 = n_base + nt * 32 < e.N ? n_base + nt * 32 : e.N - 1;
        const int last = (e.N - n0) * 2 * JT - 1;
        const v4i* base = reinterpret_cast<const v4i*>(e.V) + (int64_t)n0 * JT * 2;
        const int c = c0 * 2 + (lane & 7), at = (lane >> 3) * 2 * JT + (c < 2 * JT ? c : 2 * JT - 1);
        const int step = JT <= EP_JC ? 64 : 16 * JT, first = JT <= EP_JC ? lane : at;
#pragma unroll
        for (int j = 0; j < EP_JC; ++j) {
            const int p = first + (j < JT ? j : 0) * step;
            vf[j] = base[p < last ? p : last];
        }
    }
    // where piece 64 j + lane goes: the operands of a step of 16 ranks are 1 KiB in lane order
    __device__ __forceinline__ int v_place(int j, int w, int inv) const {
        const int p = 64 * j + lane, ch = (int)(__umul24((uint32_t)p, (uint32_t)inv) >> 16), c = p - ch * 2 * w;     // p / (2 w) for p < 512
        return (c >> 1) * 1024 + (c & 1) * 512 + ch * 16;
    }
    __device__ __forceinline__ void request() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int n = n_base + nt * 32 + l32;
            al[nt] = __half2float(e.alpha[n < e.N ? n : e.N - 1]);
        }
        if (JT > 0) load_v(0, 0);
    }
    __device__ __forceinline__ void finish(v16i (&u)[MT][NT]) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int n0 = n_base + nt * 32;
            // the main term, times 2^k of its row
            const float a = al[nt];
            v16f y[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float* at = info + mt * 32 + 8 * g + 4 * lg;
                    const v4f scu = *reinterpret_cast<const v4f*>(at);
                    const v4i qs = *reinterpret_cast<const v4i*>(at + 128);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int w = 2 * u[mt][nt][4 * g + i] - qs[i];
                        y[mt][4 * g + i] = (float)w * (scu[i] * a);
                    }
                }
                if constexpr (!GATED) __builtin_amdgcn_sched_barrier(0);      // (a row of tiles at a time: registers)
            }
            if (!GATED && e.acc_out != nullptr) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const v4i qs = *reinterpret_cast<const v4i*>(info + mt * 32 + 8 * g + 4 * lg + 128);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int t = mrow0 + mt * 32 + 8 * g + 4 * lg + i;
                            if (t < e.M && n0 + l32 < e.N) e.acc_out[(int64_t)t * e.N + n0 + l32] = 2 * u[mt][nt][4 * g + i] - qs[i];
                        }
                    }
            }
#pragma unroll 1
            for (int c0 = 0; c0 < JT; c0 += EP_JC) {
                const int w = JT < EP_JC ? JT : EP_JC, inv = 32768 / w + 1;
#pragma unroll
                for (int j = 0; j < EP_JC; ++j)
                    if (j < w) *reinterpret_cast<v4i*>(mine + v_place(j, w, inv)) = vf[j];
                if (c0 + EP_JC < JT) load_v(nt, c0 + EP_JC);
                else if (nt + 1 < NT) load_v(nt + 1, 0);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int j = 0; j < EP_JC; ++j)
                    if (c0 + j < JT) {
                        const ep_v8h vb = *reinterpret_cast<const ep_v8h*>(mine + j * 1024 + lane * 16);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            if (mt > 0 && mrow0 + mt * 32 >= e.M) break;
                            const char* t = rows_t + mt * (JT * 2048) + (c0 + j) * 2048 + lane * 16;
                            const ep_v8h thi = *reinterpret_cast<const ep_v8h*>(t), tlo = *reinterpret_cast<const ep_v8h*>(t + 1024);
                            y[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(tlo, vb, y[mt], 0, 0, 0);
                            y[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(thi, vb, y[mt], 0, 0, 0);
                        }
                    }
                __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int row0 = mrow0 + mt * 32;
                if (mt > 0 && row0 >= e.M) break;
                const int rows = e.M - row0 < 32 ? e.M - row0 : 32, N2 = e.N >> 1;
                const float* down = info + 64 + mt * 32;
                if (GATED || (e.N & 3) == 0) {
                    // out through LDS, as whole rows of the tile's channels: token rows of 128 bytes, 16-byte pieces turned
                    // by the row
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = 8 * (v >> 2) + 4 * lg + (v & 3);
                        *reinterpret_cast<float*>(mine + row * 128 + (((l32 >> 2) ^ (row & 7)) << 4) + (l32 & 3) * 4) = y[mt][v];
                    }
                    __builtin_amdgcn_wave_barrier();
                    // (all four reads before the first store: a store is a branch, and reads behind it wait one by one)
                    v4f out[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int row = 8 * k + (lane >> 3);
                        out[k] = *reinterpret_cast<const v4f*>(mine + row * 128 + (((lane & 7) ^ (row & 7)) << 4)) * down[row];
                    }
                    const int n = n0 + (lane & 7) * 4;
                    if constexpr (!GATED) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const int row = 8 * k + (lane >> 3);
                            if (row < rows && n < e.N) *reinterpret_cast<v4f*>(e.Y + (int64_t)(row0 + row) * e.N + n) = out[k];
                        }
                    } else {
                        auto gate = [&](const v4f& o) -> uint32_t {
                            uint32_t hh = 0;
#pragma unroll
                            for (int i = 0; i < 2; ++i) {
                                const float h = o[2 * i] / (1.0f + __expf(-o[2 * i])) * o[2 * i + 1];
                                hh |= (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)h) << (16 * i);
                            }
                            return hh;
                        };
                        uint16_t* const to = e.H + (int64_t)row0 * N2 + (n >> 1);
                        if ((N2 & 1) == 0) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const int row = 8 * k + (lane >> 3);
                                const uint32_t hh = gate(out[k]);
                                if (row < rows && n < e.N) *reinterpret_cast<uint32_t*>(to + (int64_t)row * N2) = hh;
                            }
                        } else {                                 // rows that start on a single value
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const int row = 8 * k + (lane >> 3);
                                const uint32_t hh = gate(out[k]);
                                if (row < rows && n < e.N) to[(int64_t)row * N2] = (uint16_t)hh;
                                if (row < rows && n + 2 < e.N) to[(int64_t)row * N2 + 1] = (uint16_t)(hh >> 16);
                            }
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                } else {
                    // rows that do not start on whole vectors: channel by channel
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const v4f d = *reinterpret_cast<const v4f*>(down + 8 * g + 4 * lg);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int row = 8 * g + 4 * lg + i, n = n0 + l32;
                            if (row < rows && n < e.N) e.Y[(int64_t)(row0 + row) * e.N + n] = y[mt][4 * g + i] * d[i];
                        }
                    }
                }
            }
        }
    }
};

}  // namespace
