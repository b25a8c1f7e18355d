// Polar factor U V^T of a small square matrix C = U S V^T in one workgroup: the orthogonal Procrustes updates of the OKT
// factors (paper App. A.2.2, "Alternating Procrustes Updates") up to 96 wide.
//
// Newton-Schulz iteration X <- X (3 I - X^T X) / 2: singular values in (0, 1] rise to 1, by 3/2 a step while small, then
// quadratically, and the singular vectors stay.  X and G = X^T X live in LDS (rows of n + 2 doubles: the 16 rows of an
// operand along k and the four of one along rows each spread over all banks), both products are fp64 MFMAs, tiles of
// 16 x 16 dealt to eight wavefronts.  X starts as C / ||C||_F; the first G gives a closer bound on the largest singular
// value, its largest absolute row sum, and the first step is scaled by it.  When every entry of G is that of I to 3e-9 the step that
// follows leaves 3/4 (G - I)^2, at most n x 0.75e-17 an entry and so I to rounding, and the last one is done.  A singular C, or one of condition beyond 1e9, does not get there in 64
// steps: `done` stays 0 and R as it was, unless `always`.
//
// Bound by the chain of steps: two products of 256 MFMAs (64 wide) on one CU's matrix cores, 4096 cycles each, and five
// barriers.  The Procrustes matrices of 11008 x 4096 with 64 x 64 factors: 97 us each, against 465 and 425 with the Jacobi
// SVD and the product of its factors; a 86 x 86 one was 200 launches of small products.
#include "bwla_internal.h"
#include "quantizer_internal.h"

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int PT = 512, PW = PT / 64, TILES = (BWLA_Q_POLAR_MAX / 16) * (BWLA_Q_POLAR_MAX / 16), OWN = (TILES + PW - 1) / PW;
constexpr int POLAR_STEPS = 64;

__global__ __launch_bounds__(PT) void polar_kernel(const double* C, int n, double* R, int* done, bool always) {
    extern __shared__ __align__(16) double lds[];
    __shared__ double sh[PW];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), r = lane & 15, q = lane >> 4;
    const int n16 = (n + 15) & ~15, ld = n16 + 2, T = n16 / 16;
    double *X = lds, *G = lds + n16 * ld;
    auto largest = [&](double v) {                          // over the workgroup, to every thread; a NaN stays
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_xor(v, off, 64);
            v = o > v || o != o ? o : v;
        }
        __syncthreads();
        if (lane == 0) sh[w] = v;
        __syncthreads();
        for (int i = 0; i < PW; ++i) v = sh[i] > v || sh[i] != sh[i] ? sh[i] : v;
        return v;
    };
    double s = 0.0;
    for (int e = t; e < n16 * n16; e += PT) {
        const int i = e / n16, j = e - i * n16;
        const double v = i < n && j < n ? C[(size_t)i * n + j] : 0.0;
        X[i * ld + j] = v;
        s = fma(v, v, s);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) sh[w] = s;
    __syncthreads();
    s = 0.0;
    for (int i = 0; i < PW; ++i) s += sh[i];
    double scale = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
    for (int e = t; e < n16 * n16; e += PT) X[(e / n16) * ld + e % n16] *= scale;
    __syncthreads();
    bool converged = false;
    for (int step = 0; step < POLAR_STEPS && !converged; ++step) {
        d4 acc[OWN];
        auto product = [&](const double* A, int ra, int ka, const double* B) {      // A(i, k) = A[i ra + k ka], B(k, j) = B[k ld + j]
#pragma unroll
            for (int o = 0; o < OWN; ++o) acc[o] = d4{0.0, 0.0, 0.0, 0.0};
            for (int k0 = 0; k0 < n16; k0 += 4)
#pragma unroll
                for (int o = 0; o < OWN; ++o) {
                    const int id = w + PW * o;
                    if (id < T * T) {
                        const double a = A[(16 * (id / T) + r) * ra + (k0 + q) * ka], b = B[(k0 + q) * ld + 16 * (id % T) + r];
                        acc[o] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[o], 0, 0, 0);
                    }
                }
        };
        auto each = [&](auto f) {                           // result <- f(result, row, column)
#pragma unroll
            for (int o = 0; o < OWN; ++o) {
                const int id = w + PW * o;
                if (id < T * T)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[o][v] = f(acc[o][v], 16 * (id / T) + 4 * v + q, 16 * (id % T) + r);
            }
        };
        product(X, 1, ld, X);
        double off = 0.0;
        each([&](double g, int i, int j) {
            G[i * ld + j] = g;
            const double d = fabs(g - (i == j && i < n ? 1.0 : 0.0));
            off = d > off || d != d ? d : off;
            return g;
        });
        off = largest(off);                                 // (its barriers are G's too)
        converged = off <= 3.0e-9;
        double f = 1.0;
        if (step == 0) {
            double sum = 0.0;
            if (t < n)
                for (int i = 0; i < n; ++i) sum += fabs(G[i * ld + t]);
            sum = largest(sum);
            f = sum > 0.0 ? 1.0 / sqrt(sum) : 0.0;
        }
        product(X, ld, 1, G);
        const double one = 1.5 * f, three = -0.5 * f * f * f;
        each([&](double g, int i, int j) { return fma(one, X[i * ld + j], three * g); });
        __syncthreads();
        each([&](double g, int i, int j) { return X[i * ld + j] = g; });
        __syncthreads();
    }
    if (converged || always)
        for (int e = t; e < n * n; e += PT) R[e] = X[(e / n) * ld + e % n];
    if (t == 0) *done = converged;
}

}  // namespace

hipError_t bwla_q_launch_polar(const double* C, int n, double* R, int* done, bool always, hipStream_t st) {
    if (n < 1 || n > BWLA_Q_POLAR_MAX) return hipErrorInvalidValue;
    const int n16 = (n + 15) & ~15;
    const size_t lds = (size_t)2 * n16 * (n16 + 2) * sizeof(double);
    const hipError_t e = bwla_ensure_lds((const void*)polar_kernel, lds + 64);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(polar_kernel, dim3(1), dim3(PT), lds, st, C, n, R, done, always);
    return hipGetLastError();
}
