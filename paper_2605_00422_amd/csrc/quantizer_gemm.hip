// fp64 GEMM of the offline quantizer (paper App. A.1 Algorithm 2: every dense contraction of the
// OKT rotation of the weight rows, of the Procrustes matrices C1 and C2 of App. A.2.2, and of the
// subspace iteration behind the truncated SVD of Sec. 3.2 runs through these kernels).
//
// v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; result register v of
// lane l is D[4 v + l / 16][l % 16].  In the general kernel a workgroup of four wavefronts owns a 64 x 64 tile of C, each
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
typedef double d2 __attribute__((ext_vector_type(2)));
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

// alpha x + beta C0[o] (+ gamma C1[o]).  The factors are read once, ahead of the stores, behind which the compiler would
// read them again (rotations of 11008 x 4096: 192 us where they take 168)
struct QCombine {
    double alpha, beta, gamma;
    const double *C0, *C1;
    __device__ __forceinline__ explicit QCombine(const QGemm& g)
        : alpha(g.coef ? g.coef[0] : g.alpha), beta(g.coef ? g.coef[1] : g.beta), gamma(g.coef ? g.coef[2] : 0.0),
          C0(beta != 0.0 ? g.C0 : nullptr), C1(gamma != 0.0 ? g.C1 : nullptr) {}
    __device__ __forceinline__ double operator()(double x, long o) const {
        x *= alpha;
        if (C0) x += beta * C0[o];
        if (C1) x += gamma * C1[o];
        return x;
    }
};

// A workgroup's 16 x 16 tile of results: row(v) is the matrix row of register v of this lane (-1 past the matrix), col its
// column.  Into C, or a partial product of a split contraction.
template <typename Row>
__device__ __forceinline__ void q_store(const QGemm& g, const QCombine f, int b, int s, d4 x, Row row, int col) {
    if (col >= g.N) return;
    const bool direct = g.ksplit == 1;
    double* to = direct ? g.C + (long)b * g.bsC : g.partials + ((long)s * g.batch + b) * (long)g.M * g.N;
    const long rs = direct ? g.rsC : g.N;
    if (direct) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = row(v);
            x[v] = r >= 0 ? f(x[v], (long)b * g.bsC + r * rs + col) : 0.0;
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = row(v);
        if (r >= 0) to[r * rs + col] = x[v];
    }
}

// (Two wavefronts a SIMD at least, in all kernels here: within 256 registers the compiler keeps the accumulators where the
// MFMAs work on them; beyond, it moves them to accumulation registers and back at every step, a quarter of the MFMAs' time.)
template <bool EASY, bool AK, bool BK>
__global__ __launch_bounds__(256, 2) void qgemm_kernel(QGemm g) {
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
                    const d2 u = *reinterpret_cast<const d2*>(p), v = *reinterpret_cast<const d2*>(p2);
                    r[0] = u[0]; r[1] = u[1]; r[2] = v[0]; r[3] = v[1];
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
    const QCombine combine(g);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            q_store(g, combine, b, s, acc[a][c], [&](int v) {
                const int row = i0 + wm + a * 16 + 4 * v + lq;
                return row < g.M ? row : -1;
            }, j0 + wn + c * 16 + lr);
}

// ---------------------------------------------------------------- A from memory, B through LDS
// The order of the contraction index is free as long as A and B agree: with lane (r, q) = (l % 16, l / 16) taking k = 4 q + s
// in MFMA s of a step of 16, the A operand of all four is 32 contiguous bytes of row r (AK: k contiguous), or a double of
// four rows of k, 128 contiguous bytes each over the 16 lanes (rows contiguous), so that A goes straight from
// memory into operand registers, whole lines at a time, and only B, which the four wavefronts share (rows of 64 doubles, N
// contiguous), passes through LDS: 8 KiB a step of 16, in 16-byte pieces whose place is turned by 128 bytes for odd q, as
// a row is a multiple of all banks.  Wavefront w owns MT x 16 rows of the tile.  64 cycles an MFMA and four LDS reads for
// 4 MT of them: bound by the matrix cores where K is long, by memory where it is short (the rotations).  Against both
// operands through LDS in tiles of 64 x 64 (below), 11008 x 4096: Y Q with 64 columns 157 -> 132 us, Y^T Z 130 -> 131, with
// the sums of their partial products 9 -> 7 and 9 -> 6; rotations 170 -> 158 and 160 -> 152 (720 MB, 4.7 TB/s).
constexpr int SK = 16;

template <int MT, bool AK>
__global__ __launch_bounds__(256, 2) void qgemm_stream_kernel(QGemm g) {
    if (q_skipped(g)) return;
    __shared__ __align__(16) double Bs[2][SK][64];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), r = lane & 15, q = lane >> 4;
    const int b = blockIdx.z / g.ksplit, s = blockIdx.z % g.ksplit;
    const int i0 = blockIdx.y * 64 * MT + w * 16 * MT, j0 = blockIdx.x * 64;
    const int steps = (g.K + SK - 1) / SK, per = (steps + g.ksplit - 1) / g.ksplit;
    const int kbeg = min(g.K, s * per * SK), kend = min(g.K, (s + 1) * per * SK);
    // rows and columns past the matrix read its last ones: what they contribute to is not stored
    const double* Ap[MT];
    int rows[MT];
#pragma unroll
    for (int a = 0; a < MT; ++a) {
        rows[a] = i0 + a * 16 + r;
        const int row = rows[a] < g.M ? rows[a] : g.M - 1;
        Ap[a] = g.A + (long)b * g.bsA + (long)row * g.rsA + (AK ? 4L * q : 4L * q * g.klA);
    }
    const double* Bp[2];
    int brow[2], bat[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int id = t + 256 * u, piece = id & 31, col = j0 + 2 * piece;
        brow[u] = id >> 5;
        bat[u] = brow[u] * 64 + 2 * (piece ^ (((brow[u] >> 2) & 1) << 3));
        Bp[u] = g.B + (long)b * g.bsB + (col + 1 < g.N ? col : g.N - 2);
    }
    double a[MT][4], an[MT][4];
    d2 bn[2];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + brow[u];
            bn[u] = *reinterpret_cast<const d2*>(Bp[u] + (long)(k < kend ? k : kend - 1) * g.klB);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            if (k0 + SK <= kend) {
                if (AK) {
                    const d2 lo = *reinterpret_cast<const d2*>(Ap[i] + k0);
                    const d2 hi = *reinterpret_cast<const d2*>(Ap[i] + k0 + 2);
                    an[i][0] = lo[0]; an[i][1] = lo[1]; an[i][2] = hi[0]; an[i][3] = hi[1];
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) an[i][u] = Ap[i][(long)(k0 + u) * g.klA];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) an[i][u] = k0 + 4 * q + u < kend ? Ap[i][(long)(k0 + u) * (AK ? 1 : g.klA)] : 0.0;
            }
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 2; ++u) *reinterpret_cast<d2*>(&Bs[buf][0][0] + bat[u]) = bn[u];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) a[i][u] = an[i][u];
    };
    d4 acc[MT][4];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[i][c] = d4{0.0, 0.0, 0.0, 0.0};
    if (kbeg < kend) {
        fetch(kbeg);
        put(0);
        __syncthreads();
        int buf = 0;
        for (int k0 = kbeg; k0 < kend; k0 += SK) {
            const bool more = k0 + SK < kend;
            if (more) fetch(k0 + SK);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                double bv[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) bv[c] = Bs[buf][4 * q + u][(16 * c + r) ^ ((q & 1) << 4)];
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][u], bv[c], acc[i][c], 0, 0, 0);
            }
            if (more) put(buf ^ 1);
            __syncthreads();
            buf ^= 1;
        }
    }
    const QCombine combine(g);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            q_store(g, combine, b, s, acc[i][c], [&](int v) {
                const int row = i0 + i * 16 + 4 * v + q;
                return row < g.M ? row : -1;
            }, j0 + 16 * c + r);
}

// ---------------------------------------------------------------- small results of long contractions
// A 64 x 64 tile of C per wavefront, both operands straight from memory as above (KC: k contiguous in both, else the
// rows of A and the columns of B, two neighbours a load), no LDS and no barrier in the loop: a step of 16 is 16 KiB of
// operands and 64 MFMAs, so that the products over all rows of the layer (the Procrustes matrices, 720 MB) stream at the
// memory's rate.  The four wavefronts of a workgroup take neighbouring ranges of the contraction and are added in
// order through LDS.  Against tiles through LDS, whose partial products were added by one thread an element, at
// 11008 x 4096: 265 + 79 -> 180 + 6 us (k contiguous), 217 + 75 -> 174 + 6 (4.1 TB/s); Gram matrices of 64 columns 19 + 7 -> 15 + 5.
template <bool KC>
__global__ __launch_bounds__(256, 2) void qgemm_square_kernel(QGemm g) {
    if (q_skipped(g)) return;
    __shared__ __align__(16) double red[2][64][64];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), r = lane & 15, q = lane >> 4;
    const int s = blockIdx.z, i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    const int steps = (g.K + SK - 1) / SK, ranges = 4 * g.ksplit, per = (steps + ranges - 1) / ranges;
    const int kbeg = min(g.K, (4 * s + w) * per * SK), kend = min(g.K, (4 * s + w + 1) * per * SK);
    const double *Ap[4], *Bp[4];                            // KC: of a tile; else of tiles 2 i, 2 i + 1 (two of them)
#pragma unroll
    for (int i = 0; i < (KC ? 4 : 2); ++i) {
        const int ra = i0 + (KC ? 16 * i + r : 32 * i + 2 * r), rb = j0 + (KC ? 16 * i + r : 32 * i + 2 * r);
        const int last = KC ? 1 : 2;
        Ap[i] = g.A + (long)(ra + last <= g.M ? ra : g.M - last) * g.rsA + (KC ? 4 * q : 0);
        Bp[i] = g.B + (long)(rb + last <= g.N ? rb : g.N - last) * g.csB + (KC ? 4 * q : 0);
    }
    // a step in two halves of two MFMAs each, the next one's operands on their way: [tile][MFMA]
    double a[4][2], bb[4][2], an[4][2], bn[4][2];
    auto fetch = [&](int k0, int half) {
        if (KC) {
            const long oa = q_koff(k0, g.kdivA, g.khA, 1) + 2 * half, ob = q_koff(k0, g.kdivB, g.khB, 1) + 2 * half;   // uniform
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const d2 x = *reinterpret_cast<const d2*>(Ap[i] + oa), y = *reinterpret_cast<const d2*>(Bp[i] + ob);
                an[i][0] = x[0]; an[i][1] = x[1];
                bn[i][0] = y[0]; bn[i][1] = y[1];
            }
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = k0 + 4 * q + 2 * half + u, kk = k < kend ? k : kend - 1;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const d2 x = *reinterpret_cast<const d2*>(Ap[i] + (long)kk * g.klA);
                    const d2 y = *reinterpret_cast<const d2*>(Bp[i] + (long)kk * g.klB);
                    an[2 * i][u] = k < kend ? x[0] : 0.0;
                    an[2 * i + 1][u] = k < kend ? x[1] : 0.0;
                    bn[2 * i][u] = y[0];
                    bn[2 * i + 1][u] = y[1];
                }
            }
        }
    };
    d4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[i][c] = d4{0.0, 0.0, 0.0, 0.0};
    if (kbeg < kend) fetch(kbeg, 0);
    for (int k0 = kbeg; k0 < kend; k0 += SK) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    a[i][u] = an[i][u];
                    bb[i][u] = bn[i][u];
                }
            if (half == 0) fetch(k0, 1);
            else if (k0 + SK < kend) fetch(k0 + SK, 0);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][u], bb[c][u], acc[i][c], 0, 0, 0);
        }
    }
    // (w0 + w1) + (w2 + w3)
    for (int half = 1; half <= 2; ++half) {
        const bool gives = half == 1 ? (w & 1) : w == 2, takes = half == 1 ? !(w & 1) : w == 0;
        const int place = half == 1 ? w >> 1 : 0;
        if (half == 2) __syncthreads();
        if (gives)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[place][(i * 4 + c) * 4 + v][lane] = acc[i][c][v];
        __syncthreads();
        if (takes)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[i][c][v] += red[place][(i * 4 + c) * 4 + v][lane];
    }
    if (w) return;
    const QCombine combine(g);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            q_store(g, combine, 0, s, acc[i][c], [&](int v) {
                const int row = i0 + (KC ? 16 * i + 4 * v + q : 32 * (i >> 1) + 2 * (4 * v + q) + (i & 1));
                return row < g.M ? row : -1;
            }, j0 + (KC ? 16 * c + r : 32 * (c >> 1) + 2 * r + (c & 1)));
}

// Adds the ksplit partial products in range order, a range of them by each of G threads whose sums are added in order,
// and combines the sum with C0 and C1.  (With one thread an element 256 partial products of 64 x 64 took 79 us, one
// load after the other.)
template <int G>
__global__ __launch_bounds__(256) void qgemm_reduce_kernel(QGemm g) {
    if (q_skipped(g)) return;
    __shared__ double sh[G][256 / G];
    const long per = (long)g.M * g.N, total = per * g.batch;
    const QCombine combine(g);
    const int slot = threadIdx.x % (256 / G), part = threadIdx.x / (256 / G), each = (g.ksplit + G - 1) / G;
    const int sbeg = min(g.ksplit, part * each), send = min(g.ksplit, (part + 1) * each);
    for (long e0 = (long)blockIdx.x * (256 / G); e0 < total; e0 += (long)gridDim.x * (256 / G)) {
        const long e = e0 + slot;
        double x = 0.0;
        if (e < total) {
            int s = sbeg;
            for (; s + 4 <= send; s += 4) {
                const double* p = g.partials + (long)s * total + e;
                const double y0 = p[0], y1 = p[total], y2 = p[2 * total], y3 = p[3 * total];
                x = (((x + y0) + y1) + y2) + y3;
            }
            for (; s < send; ++s) x += g.partials[(long)s * total + e];
        }
        if (G > 1) {
            __syncthreads();
            sh[part][slot] = x;
            __syncthreads();
            if (part) continue;
#pragma unroll
            for (int i = 1; i < G; ++i) x += sh[i][slot];
        }
        if (e < total) {
            const long b = e / per, rem = e - b * per;
            const long row = rem / g.N, col = rem - row * g.N;
            const long o = b * g.bsC + row * g.rsC + col;
            g.C[o] = combine(x, o);
        }
    }
}

}  // namespace

hipError_t bwla_q_launch_gemm(QGemm g, size_t partial_bytes, hipStream_t st) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
    const auto tiles_of = [](int n, int t) { return (long)((n + t - 1) / t); };
    if (tiles_of(g.M, TM) > 65535 || g.batch > 65535) return hipErrorInvalidValue;
    const bool easy = (g.kdivA == 0 || g.kdivA % TK == 0) && (g.kdivB == 0 || g.kdivB % TK == 0);
    const auto aligned = [](const double* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    // pairs of doubles along k: neighbours in memory, 16-byte aligned in every row, block and batch
    auto pairs = [&](const double* p, long rs, long kh, long kl, long bs, int kdiv) {
        return easy && kl == 1 && aligned(p) && rs % 2 == 0 && bs % 2 == 0 && (kdiv == 0 || kh % 2 == 0);
    };
    const bool ak = pairs(g.A, g.rsA, g.khA, g.klA, g.bsA, g.kdivA), bk = pairs(g.B, g.csB, g.khB, g.klB, g.bsB, g.kdivB);
    // the most ranges of the contraction whose partial products fit
    long most = (long)(partial_bytes / ((size_t)g.batch * g.M * g.N * sizeof(double)));
    if (most > 256) most = 256;
    if (most * g.batch > 65535) most = 65535 / g.batch;
    if (most < 1) most = 1;
    const long steps = tiles_of(g.K, SK);
    const auto launch = [&](auto kern, dim3 grid) {
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, g);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || g.ksplit == 1) return e;
        const long total = (long)g.M * g.N * g.batch;
        const auto blocks = [&](int a_block) { const long n = (total + a_block - 1) / a_block; return dim3((unsigned)(n < 2048 ? n : 2048)); };
        if (g.ksplit >= 16) hipLaunchKernelGGL(qgemm_reduce_kernel<8>, blocks(32), dim3(256), 0, st, g);
        else hipLaunchKernelGGL(qgemm_reduce_kernel<1>, blocks(256), dim3(256), 0, st, g);
        return hipGetLastError();
    };
    // pairs of neighbouring rows of A, of columns of B
    const bool ra = g.rsA == 1 && g.kdivA == 0 && aligned(g.A) && g.klA % 2 == 0 && g.M % 2 == 0;
    const bool cb = g.csB == 1 && g.kdivB == 0 && aligned(g.B) && g.klB % 2 == 0 && g.bsB % 2 == 0 && g.N % 2 == 0;
    const long squares = tiles_of(g.M, 64) * tiles_of(g.N, 64);
    if (g.batch == 1 && squares <= 16 && g.K >= 2048 && ((ak && bk && g.K % SK == 0) || (ra && cb))) {
        // a result of few tiles, each of them by four wavefronts a workgroup: as many ranges as fill the chip once, of
        // at least two steps
        long S = 256 / squares;
        if (S > steps / 8) S = steps / 8;
        if (S > most) S = most;
        g.ksplit = (int)(S < 1 ? 1 : S);
        const dim3 grid((unsigned)tiles_of(g.N, 64), (unsigned)tiles_of(g.M, 64), g.ksplit);
        return ak && bk ? launch(qgemm_square_kernel<true>, grid) : launch(qgemm_square_kernel<false>, grid);
    }
    if (cb && ((ak && g.kdivA == 0) || (g.rsA == 1 && g.kdivA == 0))) {
        // Rows a tile and ranges of the contraction by the time that they take, us: a step of 16 of a tile of 64 rows is 1024
        // cycles of the four matrix cores, and a CU that has one workgroup waits for memory at times; a partial product
        // is written and read, and a launch adds them up.
        int mt = 1;
        long best = 1;
        double least = 1.0e30;
        for (int rows = 1; rows <= 2; ++rows) {
            const long tiles = tiles_of(g.N, 64) * tiles_of(g.M, 64 * rows) * g.batch;
            for (long S = 1; S <= most && (S == 1 || (tiles < 512 && S * 16 <= steps)); ++S) {
                const long together = tiles_of((int)(tiles * S), 256);
                const double cost = (double)together * tiles_of((int)steps, (int)S) * rows * 0.49 * (together == 1 ? 1.2 : 1.0) +
                                    (S > 1 ? 5.0 + 4.0e-6 * S * g.M * g.N * g.batch : 0.0);
                if (cost < least) { least = cost; best = S; mt = rows; }
            }
        }
        g.ksplit = (int)best;
        const dim3 grid((unsigned)tiles_of(g.N, 64), (unsigned)tiles_of(g.M, 64 * mt), (unsigned)(g.batch * best));
        if (ak) return mt == 1 ? launch(qgemm_stream_kernel<1, true>, grid) : launch(qgemm_stream_kernel<2, true>, grid);
        return mt == 1 ? launch(qgemm_stream_kernel<1, false>, grid) : launch(qgemm_stream_kernel<2, false>, grid);
    }
    // about 1024 workgroups, at least 256 of K per range
    const long tiles = tiles_of(g.M, TM) * tiles_of(g.N, TN) * g.batch;
    long S = 1;
    if (tiles < 512) {
        S = 1024 / tiles;
        if (S > g.K / 256) S = g.K / 256;
        if (S > most) S = most;
        if (S < 2) S = 1;
    }
    g.ksplit = (int)S;
    const dim3 grid((unsigned)tiles_of(g.N, TN), (unsigned)tiles_of(g.M, TM), (unsigned)(g.batch * S));
    const auto kern = !easy ? qgemm_kernel<false, false, false>
                      : ak ? (bk ? qgemm_kernel<true, true, true> : qgemm_kernel<true, true, false>)
                           : (bk ? qgemm_kernel<true, false, true> : qgemm_kernel<true, false, false>);
    return launch(kern, grid);
}
