// Binary-weight GEMM for many tokens on the sparse INT8 matrix instructions, which contract twice the columns of the
// dense ones in the same time.  A +-1 weight matrix becomes 2:4 sparse in another basis: for a pair of columns
//
//     w1 x1 + w2 x2 = w1 (x1 + (w1 w2) x2)  =  w1 s  where the signs agree,  w1 d  where they differ,
//     s = x1 + x2,  d = x1 - x2,
//
// so with the codes turned into (s, d) every pair of weights picks one of two values and a sign: one of every two, two of
// every four, which is what v_smfmac_i32_32x32x64_i8 takes.  The sums stay exact int32: codes in [-64, 63] (every width up
// to 7 bits, symmetric or asymmetric) give s and d that fit int8.
//   pair_codes_kernel   codes -> (s, d) in the order in which the GEMM copies them to LDS, and one flag per 16 tokens
//                       and 512 columns for codes outside [-64, 63]
//   gemm_sparse_kernel  the contraction; same epilogue arithmetic as gemm_prefill.hip, to the bit.  A workgroup that finds
//                       a flag set contracts its tile on the dense instructions from the codes themselves (slowly).
//
// Operand A of the instruction is the weights (rows: channels), compressed: 16 values a lane and an index of two bits for
// each.  The values are the sign bits as bytes of +-64 (they differ in bit 7 alone: one shift and one bit select per four
// of them); the accumulators are therefore -64 times the sums.  The index wants the agreement bits of four words side by
// side in one byte, where a packed word (see bwla_internal.h) has them eight bits apart: a 4 x 4 transposition of bits, 20
// instructions per 256 weights of a row (convert_w).  The two columns of a pair are 4 apart (words d and d + 1 of a
// 128-column group, whose bits are aligned); value 4 g + b of lane half h in contraction m of a superstep of 512 columns is
// the pair at 128 g + 16 m + 8 h + b.  Operand B (columns: tokens): lane half H holds the pairs of groups 2 H and 2 H + 1.
#include "bwla_internal.h"
#include "gemm_tiles.h"
#include "gemm_epilogue.h"

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v2i __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t gs_bfi(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }
// Constants that the compiler is not to fold, so that they stay operands of three-input instructions.  (An instruction
// takes one scalar register; the thread index makes the second constant a lane's own in the compiler's eyes.)
__device__ __forceinline__ uint32_t gs_sgpr(uint32_t x) { asm("" : "+s"(x)); return x; }
__device__ __forceinline__ uint32_t gs_vgpr(uint32_t x) { asm("" : "+v"(x) : "v"(threadIdx.x)); return x; }
__device__ __forceinline__ uint32_t gs_xad(uint32_t x, uint32_t sk, uint32_t vk) {
    uint32_t o = (x ^ sk) + vk;
    asm("" : "+v"(o));                                       // kept together: one instruction
    return o;
}

// (s, d) of the codes: [64 tokens][superstep][m 0..7][h][H][64 tokens][16 bytes], 32 KiB per 64 tokens and superstep.
// Four bytes at a time: with v = sum (x + 64) 256^i, sums and differences of two such words do not carry between bytes while
// the codes are in [-64, 63], and bit 7 of a byte of v is set by any code that is not.  Bound by memory: as many bytes out
// as codes in, 117 MB each way in 36 us at 4096 tokens of 28672 columns.  Calls that overlap on one scratch with the same
// codes (two layers on the same rotated tokens) write the same bytes.
__global__ __launch_bounds__(256) void pair_codes_kernel(const int8_t* __restrict__ q, int M, int K, int nss, uint8_t* __restrict__ z,
                                                         uint32_t* __restrict__ flags) {
    // a wavefront: 8 tokens x 8 m; a workgroup: 16 tokens of a superstep
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 7, H = wave & 1;
    const int ks = blockIdx.x % nss, group = blockIdx.x / nss;
    const int row = group * 16 + (wave >> 1) * 8 + (lane >> 3);
    const uint32_t s80 = gs_sgpr(0x80808080u), vk = gs_vgpr(0x40404040u - 0x80808080u);
    const int c0 = ks * 512 + H * 256 + m * 16;
    uint4 a = make_uint4(0, 0, 0, 0), b = a;                 // tokens past the end and columns past K: zeros
    if (row < M) {
        if (c0 < K) a = *reinterpret_cast<const uint4*>(q + (int64_t)row * K + c0);
        if (c0 + 128 < K) b = *reinterpret_cast<const uint4*>(q + (int64_t)row * K + c0 + 128);
    }
    uint32_t bad = 0;
    auto pair = [&](uint32_t x, uint32_t y) -> uint2 {
        const uint32_t va = gs_xad(x, s80, vk), vb = gs_xad(y, s80, vk);
        bad |= va | vb;
        const uint32_t s = (va + vb) ^ s80, d = ((va | s80) - vb) ^ s80;
        return make_uint2(__builtin_amdgcn_perm(d, s, 0x05010400u), __builtin_amdgcn_perm(d, s, 0x07030602u));
    };
    uint8_t* dst = z + ((int64_t)((row >> 6) * nss + ks) * 8 + m) * 4096 + H * 1024 + (row & 63) * 16;
    const uint2 p0 = pair(a.x, a.y), p1 = pair(b.x, b.y), p2 = pair(a.z, a.w), p3 = pair(b.z, b.w);
    *reinterpret_cast<uint4*>(dst) = make_uint4(p0.x, p0.y, p1.x, p1.y);
    *reinterpret_cast<uint4*>(dst + 2048) = make_uint4(p2.x, p2.y, p3.x, p3.y);
    const int any = __syncthreads_or((int)(bad & 0x80808080u));
    if (threadIdx.x == 0) flags[blockIdx.x] = any != 0 ? 1u : 0u;
}

__device__ __forceinline__ v4i gs_read128(uint32_t addr, int ofs) {
    v4i r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(ofs));
    return r;
}
__device__ __forceinline__ v2i gs_read64(uint32_t addr, int ofs) {
    v2i r;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(ofs));
    return r;
}
// s_waitcnt immediate for vmcnt(n) alone
static_assert(BWLA_MAX_K <= 64 * BWLA_CHUNK_COLS, "a lane for every superstep");
constexpr int gs_vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// A wavefront owns MT x 32 tokens by NT x 32 channels; WN of them stand side by side over the same tokens and share one
// ring of code tiles in LDS, RING pairs of contractions deep, filled by asynchronous copies, one barrier a pair.  Each
// wavefront copies the sign bits of its own channels there too, two supersteps deep.  Nothing in the loop loads to registers
// from memory, so the waits are counted by hand; LDS reads are inline assembly, which the compiler does not order against the
// copies (see gemm_prefill.hip).
// What bounds it is power and instruction issue: on registers alone 1024 wavefronts of these instructions run at 1.5 GHz
// (21.6 ns each; dense ones at 1.8, 17.6 ns for half the columns), and beyond four vector instructions for each every
// further one costs its four cycles.  Hence wide wavefront tiles (the 13 instructions that prepare an operand of weights
// serve MT contractions) and codes prepared once for all channels: prepared per workgroup on the way to LDS they took a
// fifth of the instructions and a register-staged copy (28672 -> 8192 at 4096 tokens 545 us; 477 + 36 this way).
// Pass and GEMM against the dense kernel, in turn on one card, rank 64: 28672 -> 8192 at 4096 tokens 653 -> 490 us, 28672 ->
// 28672 2288 -> 1643, 25600 -> 5120 at 2048 186 -> 168, 4096 -> 22016 gated at 2048 174 -> 168.
template <int MT, int NT, int WN, int RING, int RESIDENT, bool GATED>
__global__ __launch_bounds__(64 * WN, RESIDENT) void gemm_sparse_kernel(
    const uint4* __restrict__ bits, int chunks, int row_tiles, const uint8_t* __restrict__ z, const uint32_t* __restrict__ flags,
    const int8_t* __restrict__ q, int M, int K,
    const float* __restrict__ scale, const __half* __restrict__ alpha, const __half* __restrict__ V,
    const float* __restrict__ T, int r, float* __restrict__ Y, int N, int32_t* __restrict__ acc_out, int tiles_n,
    uint16_t* __restrict__ H) {
    constexpr int BM = 32 * MT, BN = 32 * NT * WN;
    constexpr int SLOT = BM * 64;                            // bytes of an m
    constexpr int PAIR = 2 * SLOT;
    constexpr int CP = PAIR / 1024 / WN;                     // copies of codes a pair and wavefront
    static_assert(CP * WN * 1024 == PAIR, "");
    constexpr int WU = 2 * NT;                               // weight units a superstep and wavefront
    constexpr int WP = (WU + 3) / 4;                         // copies of weights a pair
    constexpr int PER = CP + WP;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lg = lane >> 5;
    int pid = blockIdx.x;
    const int nblocks = gridDim.x;
    if ((nblocks & 7) == 0) pid = (pid & 7) * (nblocks >> 3) + (pid >> 3);
    const int tm = pid / tiles_n, tn = pid - tm * tiles_n;
    const int m_base = tm * BM, n_base = tn * BN + wave * (32 * NT);
    const int nss = chunks;
    const uint32_t s80 = gs_sgpr(0x80808080u), v40 = gs_vgpr(0x40404040u), s55 = gs_sgpr(0x55555555u), v88 = gs_vgpr(0x88888888u);

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    char* wbuf = smem + RING * PAIR + wave * (2 * WU * 1024);                  // this wavefront's weights, two supersteps
    const uint32_t wlds = lds0 + RING * PAIR + wave * (2 * WU * 1024) + (l32 >> 4) * 1024 + (l32 & 15) * 16 + lg * 8;
    const uint32_t zlds = lds0 + lg * 1024 + l32 * 16;

    // ---- copies
    const int rbs = (M + 63) >> 6;                           // blocks of 64 tokens
    const int rb0 = m_base >> 6;
    auto copy_z = [&](int t, int pos) {                      // pair t of supersteps 0 .. nss - 1 (past the end: the last one)
        int ks = t >> 2;
        if (ks > nss - 1) ks = nss - 1;
        const int pr = t & 3;
#pragma unroll
        for (int c = 0; c < CP; ++c) {
            const int piece = wave * CP + c;                 // of the pair: [m][row block][4]
            const int mm = piece / (SLOT / 1024), rest = piece % (SLOT / 1024);
            int rb = rb0 + (rest >> 2);
            if (rb > rbs - 1) rb = rbs - 1;
            const uint8_t* src = z + ((int64_t)(rb * nss + ks) * 8 + 2 * pr + mm) * 4096 + (rest & 3) * 1024 + lane * 16;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)(smem + pos * PAIR + piece * 1024), 16, 0, 0);
        }
    };
    const int rt0 = n_base >> 4;
    auto copy_w = [&](int ks, int pr) {                      // WP units of superstep ks
        const int kc = ks < nss ? ks : nss - 1;
#pragma unroll
        for (int c = 0; c < WP; ++c) {
            int u = pr * WP + c;
            if (u > WU - 1) u = WU - 1;
            int rt = rt0 + u;
            if (rt > row_tiles - 1) rt = row_tiles - 1;
            const uint4* src = bits + ((int64_t)rt * chunks + kc) * 64 + lane;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)(wbuf + ((ks & 1) * WU + u) * 1024), 16, 0, 0);
        }
    };
    // ---- weights of a tile: sign words and index words
    struct Wraw { v2i w[4]; };
    auto read_w = [&](Wraw& o, int ks, int nt) {
        const uint32_t a = wlds + (uint32_t)((ks & 1) * WU * 1024);
#pragma unroll
        for (int g = 0; g < 4; ++g) o.w[g] = gs_read64(a, nt * 2048 + g * 256);
    };
    auto settle_w = [&](Wraw& o) {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(o.w[0]), "+v"(o.w[1]), "+v"(o.w[2]), "+v"(o.w[3]));
    };
    uint32_t S[NT][4], P[NT][4];
    auto convert_w = [&](int nt, const Wraw& w) {
        uint32_t E[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            S[nt][g] = (uint32_t)w.w[g][0];
            E[g] = (uint32_t)(w.w[g][0] ^ w.w[g][1]);
        }
        const uint32_t t0 = __builtin_amdgcn_perm(E[1], E[0], 0x05010400u), t1 = __builtin_amdgcn_perm(E[1], E[0], 0x07030602u);
        const uint32_t t2 = __builtin_amdgcn_perm(E[3], E[2], 0x05010400u), t3 = __builtin_amdgcn_perm(E[3], E[2], 0x07030602u);
        const uint32_t F0 = __builtin_amdgcn_perm(t2, t0, 0x05040100u), F1 = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
        const uint32_t F2 = __builtin_amdgcn_perm(t3, t1, 0x05040100u), F3 = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
        const uint32_t lo02 = gs_bfi(0x0f0f0f0fu, F0, F2 << 4), hi02 = gs_bfi(0x0f0f0f0fu, F0 >> 4, F2);
        const uint32_t lo13 = gs_bfi(0x0f0f0f0fu, F1, F3 << 4), hi13 = gs_bfi(0x0f0f0f0fu, F1 >> 4, F3);
        P[nt][0] = gs_bfi(0x33333333u, lo02, lo13 << 2);
        P[nt][1] = gs_bfi(0x33333333u, lo02 >> 2, lo13);
        P[nt][2] = gs_bfi(0x33333333u, hi02, hi13 << 2);
        P[nt][3] = gs_bfi(0x33333333u, hi02 >> 2, hi13);
    };
    struct Aop { v4i a[NT]; int x[NT]; };
    auto expand = [&](Aop& o, int nt, int m) {
#pragma unroll
        for (int g = 0; g < 4; ++g) o.a[nt][g] = (int)gs_bfi(s80, S[nt][g] << (7 - m), v40);
        o.x[nt] = (int)gs_bfi(s55, P[nt][m >> 1] >> (m & 1), v88);
    };
    // ---- code operands of two token tiles
    struct Zop { v4i lo[2], hi[2]; };
    auto read_z = [&](Zop& o, uint32_t base, int mm, int mp) {                 // m of the pair, pair of token tiles
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int mt = 2 * mp + e;
            o.lo[e] = gs_read128(base, mm * SLOT + (mt >> 1) * 4096 + (mt & 1) * 512);
            o.hi[e] = gs_read128(base, mm * SLOT + (mt >> 1) * 4096 + (mt & 1) * 512 + 2048);
        }
    };
    auto settle_z = [&](Zop& o) {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(o.lo[0]), "+v"(o.hi[0]), "+v"(o.lo[1]), "+v"(o.hi[1]));
    };
    v16i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mt][nt][v] = 0;

    // Codes that do not fit the pairs?  Every wavefront looks at all flags of the tile, a lane a superstep (there are at
    // most 64; past the end an existing one again).
    uint32_t fl[BM / 16];
#pragma unroll
    for (int f = 0; f < BM / 16; ++f) {
        const int fr = (m_base >> 4) + f;                    // (16-token flags exist for whole blocks of 64 tokens)
        const uint32_t* src = flags + (fr < 4 * rbs ? fr : 4 * rbs - 1) * nss + (lane < nss ? lane : 0);
        asm volatile("global_load_dword %0, %1, off" : "=v"(fl[f]) : "v"(src) : "memory");
    }
    // Issue order of the copies: weights of superstep 0; then for every pair t its codes and a quarter of the weights of
    // the next superstep but one (of superstep 1 for the first pairs), PER operations together.  At the end of pair t the
    // codes of pair t + 1 are needed: the operations younger than those are the RING - 2 groups behind them.
#pragma unroll
    for (int pr = 0; pr < 4; ++pr) copy_w(0, pr);
#pragma unroll
    for (int pr = RING; pr < 4; ++pr) copy_w(1, pr);
#pragma unroll
    for (int t = 0; t < RING; ++t) { copy_z(t, t); copy_w(1, t); }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(gs_vmcnt_imm((RING - 1) * PER));
    uint32_t wide = 0;
#pragma unroll
    for (int f = 0; f < BM / 16; ++f) {
        asm volatile("" : "+v"(fl[f]));                      // (has landed: it is older than every copy)
        wide |= fl[f];
    }
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (__ballot(wide != 0) != 0) {                          // the tile from the codes themselves, on the dense instructions
#pragma unroll 1
        for (int k = 0; k < K; k += 32) {
            const int c = k + 16 * lg;
            v4i b[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m = m_base + mt * 32 + l32;
                b[mt] = *reinterpret_cast<const v4i*>(q + (int64_t)(m < M ? m : M - 1) * K + c);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                int rt = (n_base + nt * 32 + l32) >> 4;
                if (rt > row_tiles - 1) rt = row_tiles - 1;
                const uint4 w = bits[((int64_t)rt * chunks + (c >> 9)) * 64 + ((c >> 7) & 3) * 16 + (l32 & 15)];
                const int up = 7 - ((c >> 4) & 7);
                const v4i a = {(int)gs_bfi(s80, w.x << up, v40), (int)gs_bfi(s80, w.y << up, v40),
                               (int)gs_bfi(s80, w.z << up, v40), (int)gs_bfi(s80, w.w << up, v40)};
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[mt], acc[mt][nt], 0, 0, 0);
            }
        }
    } else {
    Zop zc;
    Aop op[2];
    Wraw w[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        read_w(w[nt], 0, nt);
        settle_w(w[nt]);
        convert_w(nt, w[nt]);
        expand(op[0], nt, 0);
    }
    read_z(zc, zlds, 0, 0);
    settle_z(zc);
    constexpr int MP = MT / 2;
    int pos = 0;                                             // of the current pair in the ring
    int t = 0;
    for (int ks = 0; ks < nss; ++ks) {
#pragma unroll
        for (int pr = 0; pr < 4; ++pr) {
            const int npos = pos + 1 == RING ? 0 : pos + 1;
            const uint32_t zb = zlds + (uint32_t)(pos * PAIR), zn = zlds + (uint32_t)(npos * PAIR);
#pragma unroll
            for (int i = 0; i < 2 * MP; ++i) {
                const int mm = i / MP, mp = i % MP, m = 2 * pr + mm;
                Zop nx;
                if (i + 1 < 2 * MP) {
                    read_z(nx, zb, (i + 1) / MP, (i + 1) % MP);
                } else {
                    __builtin_amdgcn_s_waitcnt(gs_vmcnt_imm((RING - 2) * PER));   // the next pair has landed: mine, then everybody's
                    __builtin_amdgcn_s_barrier();
                    read_z(nx, zn, 0, 0);
                }
                if (m == 6 && mp == MP - 1) {                // the weights of the next superstep, settled with the codes below
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) read_w(w[nt], ks + 1, nt);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    if (nt * MP / NT == mp) {                // operands of the next m
                        if (m == 7) convert_w(nt, w[nt]);
                        expand(op[(m + 1) & 1], nt, (m + 1) & 7);
                    }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const v8i zz = __builtin_shufflevector(zc.lo[e], zc.hi[e], 0, 1, 2, 3, 4, 5, 6, 7);
                        acc[2 * mp + e][nt] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(op[m & 1].a[nt], zz, acc[2 * mp + e][nt],
                                                                                     op[m & 1].x[nt], 0, 0);
                    }
#pragma unroll
                for (int e = 0; e < 2 * NT; ++e) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                settle_z(nx);
                if (m == 6 && mp == MP - 1) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(w[nt].w[0]), "+v"(w[nt].w[1]), "+v"(w[nt].w[2]), "+v"(w[nt].w[3]));
                }
                zc = nx;
            }
            copy_z(t + RING, pos);
            copy_w(ks + 2, pr);
            __builtin_amdgcn_sched_barrier(0);
            pos = npos;
            ++t;
        }
    }
    __builtin_amdgcn_s_waitcnt(gs_vmcnt_imm(0));             // copies that nobody reads have landed before LDS is used anew
    }
    __syncthreads();

    // ---- epilogue: element v of lane (l32, lg) is channel 8 (v / 4) + 4 lg + v % 4 of token l32; acc = -64 sum.
    // T, once for the workgroup, as operands in LDS (gemm_epilogue.h).  Then one row of tiles (32 tokens) at a time: its
    // accumulators go to the wavefront's part of LDS, 4 KiB a tile, and a loop takes tile after tile from there -- the code
    // is one tile's, not MT x NT copies of it.
    constexpr int JC = EP_JC;
    const int JT = (r + 15) >> 4, w = JT < JC ? JT : JC, inv = w > 0 ? 32768 / w + 1 : 0;
    char* mine = smem + wave * (NT * 4096);
    char* const rows_lds = smem + WN * NT * 4096;
    const float* const info = reinterpret_cast<const float*>(rows_lds + BM * 64 * JT);
    {
        const EpArgs ep{scale, nullptr, alpha, V, T, r, Y, M, N, acc_out, H};
        EpRows<64 * WN, BM> rows(ep, tid);
        rows.request(m_base);
        rows.put(rows_lds);
    }
    // V as the contiguous rows of a tile's channels, whole lines a request; alpha of my channels
    struct Vop { v4i v[JC]; uint2 al[4]; };
    auto load_v = [&](Vop& o, int nt, int c0) {
        const int n0 = n_base + nt * 32 < N ? n_base + nt * 32 : N - 1;
        const int last = (N - n0) * 2 * JT - 1;
        const v4i* base = reinterpret_cast<const v4i*>(V) + (int64_t)n0 * JT * 2;
        const int c = c0 * 2 + (lane & 7), at = (lane >> 3) * 2 * JT + (c < 2 * JT ? c : 2 * JT - 1);
        const int step = JT <= JC ? 64 : 16 * JT, first = JT <= JC ? lane : at;
        if (JT > 0) {
#pragma unroll
            for (int j = 0; j < JC; ++j) {
                const int p = first + (j < JT ? j : 0) * step;
                o.v[j] = base[p < last ? p : last];
            }
        }
    };
    auto load_al = [&](Vop& o, int nt) {
        // (alpha is padded to a multiple of 256 bytes: quadruples of a tile that starts inside are readable)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            int ch = n_base + nt * 32 + 8 * g + 4 * lg;
            if (ch > N - 1) ch = (N - 1) & ~3;
            o.al[g] = *reinterpret_cast<const uint2*>(alpha + ch);
        }
    };
    __syncthreads();
#pragma unroll 1
    for (int mt = 0; mt < MT; ++mt) {
        const int mrow0 = m_base + mt * 32;
        if (mrow0 >= M) break;
        const int rows = M - mrow0 < 32 ? M - mrow0 : 32;
        const int tmr = mrow0 + (l32 < rows ? l32 : rows - 1);
        Vop vo;
        load_v(vo, 0, 0);
        load_al(vo, 0);
#pragma unroll
        for (int mm = 0; mm < MT; ++mm)
            if (mm == mt) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        *reinterpret_cast<v4i*>(mine + nt * 4096 + g * 1024 + lane * 16) =
                            v4i{acc[mm][nt][4 * g], acc[mm][nt][4 * g + 1], acc[mm][nt][4 * g + 2], acc[mm][nt][4 * g + 3]};
            }
        const float scu = info[mt * 32 + l32] * 0.015625f, down = info[BM + mt * 32 + l32];       // scale 2^k / 64, 2^-k
#pragma unroll 1
        for (int nt = 0; nt < NT; ++nt) {
            char* tile = mine + nt * 4096;
            v16f y;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4i u = *reinterpret_cast<const v4i*>(tile + g * 1024 + lane * 16);
                const __half2 a0 = __builtin_bit_cast(__half2, vo.al[g].x), a1 = __builtin_bit_cast(__half2, vo.al[g].y);
                // (multiples of 64 below 2^30: exact in fp32)
                y[4 * g + 0] = -(float)u[0] * (scu * __low2float(a0));
                y[4 * g + 1] = -(float)u[1] * (scu * __high2float(a0));
                y[4 * g + 2] = -(float)u[2] * (scu * __low2float(a1));
                y[4 * g + 3] = -(float)u[3] * (scu * __high2float(a1));
                if (!GATED && acc_out) {
                    const int n = n_base + nt * 32 + 8 * g + 4 * lg;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (l32 < rows && n + i < N) acc_out[(int64_t)tmr * N + n + i] = -(u[i] >> 6);
                }
            }
            if (nt + 1 < NT) load_al(vo, nt + 1);
#pragma unroll 1
            for (int c0 = 0; c0 < JT; c0 += JC) {
                // V in operand order, through the tile's place
#pragma unroll
                for (int j = 0; j < JC; ++j)
                    if (j < w) {
                        const int p = 64 * j + lane, ch = (int)(__umul24((uint32_t)p, (uint32_t)inv) >> 16), c = p - ch * 2 * w;
                        *reinterpret_cast<v4i*>(tile + (c >> 1) * 1024 + (c & 1) * 512 + ch * 16) = vo.v[j];
                    }
                if (c0 + JC < JT) load_v(vo, nt, c0 + JC);
                else if (nt + 1 < NT) load_v(vo, nt + 1, 0);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int j = 0; j < JC; ++j)
                    if (c0 + j < JT) {
                        const char* t = rows_lds + mt * (JT * 2048) + (c0 + j) * 2048 + lane * 16;
                        const ep_v8h vb = *reinterpret_cast<const ep_v8h*>(tile + j * 1024 + lane * 16);
                        const ep_v8h thi = *reinterpret_cast<const ep_v8h*>(t), tlo = *reinterpret_cast<const ep_v8h*>(t + 1024);
                        y = __builtin_amdgcn_mfma_f32_32x32x16_f16(vb, tlo, y, 0, 0, 0);
                        y = __builtin_amdgcn_mfma_f32_32x32x16_f16(vb, thi, y, 0, 0, 0);
                    }
                __builtin_amdgcn_wave_barrier();
            }
            if constexpr (!GATED) {
                // token rows of 128 bytes, 16-byte pieces turned by the row
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<v4f*>(tile + l32 * 128 + (((2 * g + lg) ^ (l32 & 7)) << 4)) =
                        v4f{y[4 * g] * down, y[4 * g + 1] * down, y[4 * g + 2] * down, y[4 * g + 3] * down};
            } else {
                // h of a token: rows of 32 bytes
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint32_t hh = 0;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const float gt = y[4 * g + 2 * i] * down, u = y[4 * g + 2 * i + 1] * down;
                        const float h = gt / (1.0f + __expf(-gt)) * u;
                        hh |= (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)h) << (16 * i);
                    }
                    *reinterpret_cast<uint32_t*>(tile + l32 * 32 + (2 * g + lg) * 4) = hh;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        // whole rows of the wavefront's channels
        if constexpr (!GATED) {
            if ((N & 3) == 0) {
                constexpr int PR = NT * 8;
#pragma unroll 4
                for (int p0 = 0; p0 < 32 * PR; p0 += 64) {
                    const int p = p0 + lane, row = p / PR, c = p % PR;
                    const v4f y = *reinterpret_cast<const v4f*>(mine + (c >> 3) * 4096 + row * 128 + (((c & 7) ^ (row & 7)) << 4));
                    if (row < rows && n_base + c * 4 < N)
                        *reinterpret_cast<v4f*>(Y + (int64_t)(mrow0 + row) * N + n_base + c * 4) = y;
                }
            } else {
                // rows that do not start on whole vectors: stores of four channels all the same, at the alignment of one.
                // (Value by value, every store behind its own read of LDS, such layers took 0.97 of the dense kernel's time,
                // 1.54 at most, over 103 shapes that the dispatch brings here; now 0.87 and 1.12: 1314 tokens of 2560
                // columns, 9554 channels 63.7 -> 46.3 us, 552 of 5504, 16725 channels, rank 32 68.7 -> 55.6.)
                typedef float v4f_one __attribute__((ext_vector_type(4), aligned(4)));
                constexpr int PR = NT * 8;
#pragma unroll 4
                for (int p0 = 0; p0 < 32 * PR; p0 += 64) {
                    const int p = p0 + lane, row = p / PR, c = p % PR, n = n_base + c * 4;
                    const v4f y = *reinterpret_cast<const v4f*>(mine + (c >> 3) * 4096 + row * 128 + (((c & 7) ^ (row & 7)) << 4));
                    float* to = Y + (int64_t)(mrow0 + row) * N + n;
                    if (row < rows) {
                        if (n + 3 < N) {
                            *reinterpret_cast<v4f_one*>(to) = y;
                        } else {
#pragma unroll
                            for (int i = 0; i < 3; ++i)
                                if (n + i < N) to[i] = y[i];
                        }
                    }
                }
            }
        } else {
            const int N2 = N >> 1, h_base = n_base >> 1;
            if ((N2 & 7) == 0) {
                constexpr int PR = NT * 2;
#pragma unroll 1
                for (int p0 = 0; p0 < 32 * PR; p0 += 64) {
                    const int p = p0 + lane, row = p / PR, c = p % PR;
                    const v4i y = *reinterpret_cast<const v4i*>(mine + (c >> 1) * 4096 + row * 32 + (c & 1) * 16);
                    if (row < rows && h_base + c * 8 < N2)
                        *reinterpret_cast<v4i*>(H + (int64_t)(mrow0 + row) * N2 + h_base + c * 8) = y;
                }
            } else {
                // (eight in flight: 3385 tokens of 512 columns, 10964 channels, rank 16 60.8 -> 56.8 us)
                constexpr int PR = NT * 16;
#pragma unroll 1
                for (int p0 = 0; p0 < 32 * PR; p0 += 8 * 64) {
                    uint32_t y[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        // (the pair, as it was written: the compiler takes a 16-bit read for one of something else)
                        const int p = p0 + 64 * i + lane, row = p / PR, c = p % PR;
                        y[i] = *reinterpret_cast<const uint32_t*>(mine + (c >> 4) * 4096 + row * 32 + ((c & 15) >> 1) * 4);
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int p = p0 + 64 * i + lane, row = p / PR, c = p % PR;
                        if (row < rows && h_base + c < N2)
                            H[(int64_t)(mrow0 + row) * N2 + h_base + c] = (uint16_t)(y[i] >> ((c & 1) * 16));
                    }
                }
            }
        }
    }
}


template <int I>
hipError_t launch_sparse(const bwla_layer_t* L, const int8_t* dq, const uint8_t* z, const uint32_t* flags, const float* dscale,
                         const float* dT, int64_t M, float* dY, int32_t* dacc, hipStream_t st, uint16_t* dH) {
    constexpr GsTile v = GS_TILES[I];
    constexpr int BM = 32 * v.mt, BN = 32 * v.nt * v.wn;
    const char* blob = (const char*)L->d_blob;
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((L->N + BN - 1) / BN);
    // code ring and two supersteps of weights; in the same place the epilogue turns 4 KiB a tile and wavefront and keeps T
    constexpr size_t ring = (size_t)v.ring * BM * 128 + (size_t)v.wn * 4 * v.nt * 1024, turn = (size_t)v.wn * v.nt * 4096;
    static_assert((ring > turn ? ring : turn) * v.resident <= 160 * 1024 && turn + BM * (BWLA_MAX_RANK / 16 * 64 + 12) <= 160 * 1024, "");
    const size_t tail = turn + ep_rows_bytes(BM, L->r), lds = ring > tail ? ring : tail;
    auto launch = [&](auto kern) -> hipError_t {
        hipError_t e = bwla_ensure_lds((const void*)kern, lds);
        if (e != hipSuccess) return e;
        kern<<<dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * v.wn), lds, st>>>(
            (const uint4*)(blob + L->off_bits), (int)bwla_chunks(L->K), (int)bwla_row_tiles(L->N), z, flags, dq, (int)M, (int)L->K,
            dscale, (const __half*)(blob + L->off_alpha), (const __half*)(blob + L->off_V), dT, L->r, dY, (int)L->N, dacc, tiles_n, dH);
        return hipGetLastError();
    };
    if (dH != nullptr) return launch(gemm_sparse_kernel<v.mt, v.nt, v.wn, v.ring, v.resident, true>);
    return launch(gemm_sparse_kernel<v.mt, v.nt, v.wn, v.ring, v.resident, false>);
}

template <int I>
hipError_t launch_pick(int pick, const bwla_layer_t* L, const int8_t* dq, const uint8_t* z, const uint32_t* flags, const float* dscale,
                       const float* dT, int64_t M, float* dY, int32_t* dacc, hipStream_t st, uint16_t* dH) {
    if (pick == I) return launch_sparse<I>(L, dq, z, flags, dscale, dT, M, dY, dacc, st, dH);
    if constexpr (I + 1 < GS_NTILES) return launch_pick<I + 1>(pick, L, dq, z, flags, dscale, dT, M, dY, dacc, st, dH);
    return hipErrorInvalidValue;
}

}  // namespace

// (s, d) of 64-token blocks, then the flags
static uint64_t gs_code_bytes(const bwla_layer_t* L, int64_t M) { return (uint64_t)((M + 63) / 64) * bwla_chunks(L->K) * 32768; }

uint64_t bwla_gemm_sparse_bytes(const bwla_layer_t* L, int64_t M) {
    if (M <= GS_MIN_TOKENS || !bwla_gemm_prefill_streams(L)) return 0;
    return gs_code_bytes(L, M) + bwla_align256((uint64_t)((M + 63) / 64) * 4 * bwla_chunks(L->K) * sizeof(uint32_t));
}

int bwla_gemm_sparse_pick(const bwla_layer_t* L, int64_t M, int* dense) {
    if (bwla_gemm_sparse_bytes(L, M) == 0) return -1;
    return gs_pick(M, L->K, L->N, L->r, bwla_device_cus(), dense);
}

hipError_t bwla_launch_gemm_sparse(const bwla_layer_t* L, int pick, const int8_t* dq, const float* dscale, const float* dT, int64_t M,
                                   float* dY, int32_t* dacc, hipStream_t st, void* dz, uint16_t* dH) {
    if (pick < 0 || bwla_gemm_sparse_bytes(L, M) == 0) return hipErrorInvalidValue;
    const int nss = (int)bwla_chunks(L->K);
    uint8_t* z = (uint8_t*)dz;
    uint32_t* flags = (uint32_t*)(z + gs_code_bytes(L, M));
    pair_codes_kernel<<<dim3((unsigned)(nss * ((M + 63) / 64 * 4))), dim3(256), 0, st>>>(dq, (int)M, (int)L->K, nss, z, flags);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_pick<0>(pick, L, dq, z, flags, dscale, dT, M, dY, dacc, st, dH);
}
