// fp64 GEMM of the offline quantizer (paper App. A.1 Algorithm 2: every dense contraction of the
// OKT rotation of the weight rows, of the Procrustes matrices C1 and C2 of App. A.2.2, and of the
// subspace iteration behind the truncated SVD of Sec. 3.2 runs through this one kernel).
//
// v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; result register v of
// lane l is D[4 v + l / 16][l % 16].  A workgroup of four wavefronts owns a 64 x 64 tile of C, each
// wavefront a 32 x 32 quarter (2 x 2 MFMA tiles); the operands of a 16-deep step of the contraction
// pass through LDS as [k][row] with rows padded to 72 doubles, so that the 16 lanes of a k share
// 128 contiguous bytes and the four k of an operand spread over all banks.  Global loads of the
// next step are in flight while the current one is multiplied.  Operands are read through strides
// (see quantizer_internal.h) in one of two ways:
//   k contiguous (AK, BK)  eight lanes read the 128 bytes of a row's step as pairs of doubles, so
//                          that a request of the wavefront takes eight whole lines (one row a lane
//                          touched 64 lines and was what the tall products were bound by)
//   otherwise              a lane reads its row at four k, a coalesced 512-byte run where the row
//                          index is contiguous
// A step's offset along k is the same for all lanes (EASY) unless a split contraction index changes
// its block inside a step; the general form computes it for every load.
#include "quantizer_internal.h"

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int TM = 64, TN = 64, TK = 16, LD = 72;

__device__ __forceinline__ long q_koff(int k, int kdiv, long kh, long kl) {
    if (kdiv > 0) {
        const int h = k / kdiv;
        return h * kh + (long)(k - h * kdiv) * kl;
    }
    return (long)k * kl;
}

__device__ __forceinline__ bool q_skipped(const QGemm& g) {
    const int v = g.skip ? *g.skip : 0;
    return v != 0 && v != g.skip_but;
}

// C[o] = alpha x + beta C0[o] (+ gamma C1[o])
__device__ __forceinline__ double q_combine(const QGemm& g, double x, long o) {
    const double beta = g.coef ? g.coef[1] : g.beta;
    x *= g.coef ? g.coef[0] : g.alpha;
    if (g.C0 && beta != 0.0) x += beta * g.C0[o];
    if (g.C1 && g.coef) x += g.coef[2] * g.C1[o];
    return x;
}

template <bool EASY, bool AK, bool BK>
__global__ __launch_bounds__(256) void qgemm_kernel(QGemm g) {
    if (q_skipped(g)) return;
    __shared__ double As[2][TK][LD];
    __shared__ double Bs[2][TK][LD];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int b = blockIdx.z / g.ksplit, s = blockIdx.z % g.ksplit;
    const int i0 = blockIdx.y * TM, j0 = blockIdx.x * TN;
    const int steps = (g.K + TK - 1) / TK;
    const int per = (steps + g.ksplit - 1) / g.ksplit;
    const int kbeg = min(g.K, s * per * TK), kend = min(g.K, (s + 1) * per * TK);
    const int li = t & 63, lk = (t >> 6) * 4;               // a row, four k
    const int pr = t >> 3, pk = (t & 7) * 2;                // rows pr and pr + 32, the k pair pk
    // rows past the matrix read its last one: what they contribute to is not stored
    auto rowptr = [](const double* base, int row, int rows, long stride) {
        return base + (long)(row < rows ? row : rows - 1) * stride;
    };
    const double* Ab = g.A + (long)b * g.bsA;
    const double* Bb = g.B + (long)b * g.bsB;
    const double* Ap = rowptr(Ab, i0 + (AK ? pr : li), g.M, g.rsA) + (EASY ? (long)(AK ? pk : lk) * g.klA : 0);
    const double* Bp = rowptr(Bb, j0 + (BK ? pr : li), g.N, g.csB) + (EASY ? (long)(BK ? pk : lk) * g.klB : 0);
    const double* Ap2 = AK ? rowptr(Ab, i0 + pr + 32, g.M, g.rsA) + pk : Ap;
    const double* Bp2 = BK ? rowptr(Bb, j0 + pr + 32, g.N, g.csB) + pk : Bp;
    double ra[4], rb[4];
    auto operand = [&](double (&r)[4], const double* p, const double* p2, int k0, int kdiv, long kh, long kl, bool pairs) {
        if (EASY) {
            const long off = q_koff(k0, kdiv, kh, kl);      // uniform
            p += off;
            p2 += off;
            if (pairs) {
                const int k = k0 + pk;
                if (k0 + TK <= kend) {
                    const double2 u = *reinterpret_cast<const double2*>(p), v = *reinterpret_cast<const double2*>(p2);
                    r[0] = u.x; r[1] = u.y; r[2] = v.x; r[3] = v.y;
                } else {
                    r[0] = k < kend ? p[0] : 0.0;
                    r[1] = k + 1 < kend ? p[1] : 0.0;
                    r[2] = k < kend ? p2[0] : 0.0;
                    r[3] = k + 1 < kend ? p2[1] : 0.0;
                }
            } else if (k0 + TK <= kend) {
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = p[u * kl];
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = k0 + lk + u < kend ? p[u * kl] : 0.0;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + lk + u;
                r[u] = k < kend ? p[q_koff(k, kdiv, kh, kl)] : 0.0;
            }
        }
    };
    auto gload = [&](int k0) {
        operand(ra, Ap, Ap2, k0, g.kdivA, g.khA, g.klA, AK);
        operand(rb, Bp, Bp2, k0, g.kdivB, g.khB, g.klB, BK);
    };
    auto put = [&](double (&S)[TK][LD], const double (&r)[4], bool pairs) {
        if (pairs) {
            S[pk][pr] = r[0];
            S[pk + 1][pr] = r[1];
            S[pk][pr + 32] = r[2];
            S[pk + 1][pr + 32] = r[3];
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) S[lk + u][li] = r[u];
        }
    };
    auto sstore = [&](int buf) {
        put(As[buf], ra, AK);
        put(Bs[buf], rb, BK);
    };
    const int wm = (w & 1) * 32, wn = (w >> 1) * 32, lr = lane & 15, lq = lane >> 4;
    d4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[a][c] = d4{0.0, 0.0, 0.0, 0.0};
    if (kbeg < kend) {
        gload(kbeg);
        sstore(0);
        __syncthreads();
        int buf = 0;
        for (int k0 = kbeg; k0 < kend; k0 += TK) {
            const bool more = k0 + TK < kend;
            if (more) gload(k0 + TK);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const double a0 = As[buf][ks * 4 + lq][wm + lr], a1 = As[buf][ks * 4 + lq][wm + 16 + lr];
                const double b0 = Bs[buf][ks * 4 + lq][wn + lr], b1 = Bs[buf][ks * 4 + lq][wn + 16 + lr];
                acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
            }
            if (more) sstore(buf ^ 1);
            __syncthreads();
            buf ^= 1;
        }
    }
    const bool direct = g.ksplit == 1;
    double* Cb = direct ? g.C + (long)b * g.bsC : g.partials + ((long)s * g.batch + b) * (long)g.M * g.N;
    const long rs = direct ? g.rsC : g.N;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = i0 + wm + a * 16 + 4 * v + lq, col = j0 + wn + c * 16 + lr;
                if (row < g.M && col < g.N) {
                    const long o = row * rs + col;
                    Cb[o] = direct ? q_combine(g, acc[a][c][v], (long)b * g.bsC + o) : acc[a][c][v];
                }
            }
}

// adds the ksplit partial products in range order and combines the sum with C0 and C1
__global__ __launch_bounds__(256) void qgemm_reduce_kernel(QGemm g) {
    if (q_skipped(g)) return;
    const long per = (long)g.M * g.N, total = per * g.batch;
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
        double x = 0.0;
        for (int s = 0; s < g.ksplit; ++s) x += g.partials[(long)s * total + e];
        const long b = e / per, rem = e - b * per;
        const long row = rem / g.N, col = rem - row * g.N;
        const long o = b * g.bsC + row * g.rsC + col;
        g.C[o] = q_combine(g, x, o);
    }
}

}  // namespace

hipError_t bwla_q_launch_gemm(const QGemm& g, hipStream_t st) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
    const dim3 grid((g.N + TN - 1) / TN, (g.M + TM - 1) / TM, g.batch * g.ksplit);
    if (grid.y > 65535u || grid.z > 65535u) return hipErrorInvalidValue;
    const bool easy = (g.kdivA == 0 || g.kdivA % TK == 0) && (g.kdivB == 0 || g.kdivB % TK == 0);
    // pairs of doubles along k: neighbours in memory, 16-byte aligned in every row, block and batch
    auto pairs = [&](const double* p, long rs, long kh, long kl, long bs, int kdiv) {
        return easy && kl == 1 && (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && rs % 2 == 0 && bs % 2 == 0 &&
               (kdiv == 0 || kh % 2 == 0);
    };
    const bool ak = pairs(g.A, g.rsA, g.khA, g.klA, g.bsA, g.kdivA), bk = pairs(g.B, g.csB, g.khB, g.klB, g.bsB, g.kdivB);
    const auto kern = !easy ? qgemm_kernel<false, false, false>
                      : ak ? (bk ? qgemm_kernel<true, true, true> : qgemm_kernel<true, true, false>)
                           : (bk ? qgemm_kernel<true, false, true> : qgemm_kernel<true, false, false>);
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || g.ksplit == 1) return e;
    const long total = (long)g.M * g.N * g.batch;
    const int blocks = (int)((total + 255) / 256 < 1024 ? (total + 255) / 256 : 1024);
    hipLaunchKernelGGL(qgemm_reduce_kernel, dim3(blocks), dim3(256), 0, st, g);
    return hipGetLastError();
}
