// Internal declarations of the offline quantizer's translation units (not installed).
// Everything here computes in fp64 on device-resident arrays; the launchers enqueue on the given
// stream and never synchronize or allocate.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bwla_quantizer.h"

// ---------------------------------------------------------------- fp64 GEMM (quantizer_gemm.hip)
// C[b] = alpha * A[b] * B[b] + beta * C0[b], fp64 MFMA 16x16x4, 64 x 64 tiles.
// Operands are addressed through strides so that views of the quantizer's n x m arrays (rows
// reshaped to n1 x n2, transposes, sums over the rows of all reshaped matrices) need no copies:
//   A(i, k) = A[b * bsA + i * rsA + (k / kdivA) * khA + (k % kdivA) * klA]
//   B(k, j) = B[b * bsB + j * csB + (k / kdivB) * khB + (k % kdivB) * klB]
//   C(i, j) = C[b * bsC + i * rsC + j]            (C0 is addressed like C)
// kdiv = 0 stands for "no split of the contraction index" (k / kdiv = 0, k % kdiv = k).
// The launch picks a kernel and cuts the contraction into ksplit ranges where tiles are few, whose partial products go
// to `partials` (ksplit x batch x M x N, dense) and are added in range order by a second launch, which also
// applies alpha, beta and C0: deterministic whatever the launch order.
// `coef` (device, may be NULL): C = coef[0] A B + coef[1] C0 + coef[2] C1 instead, C1 addressed like C; C0 may be C.
// `skip` (device, may be NULL): the launches return without touching C when *skip is neither 0 nor skip_but.
struct QGemm {
    const double* A; const double* B; double* C; const double* C0;
    int M, N, K, batch;
    long rsA, khA, klA, bsA; int kdivA;
    long csB, khB, klB, bsB; int kdivB;
    long rsC, bsC;
    double alpha, beta;
    int ksplit; double* partials;
    const double* C1; const double* coef;
    const int* skip; int skip_but;
};
inline QGemm qgemm_plain(const double* A, const double* B, double* C, int M, int N, int K) {
    QGemm g{};
    g.A = A; g.B = B; g.C = C; g.C0 = nullptr; g.M = M; g.N = N; g.K = K; g.batch = 1;
    g.rsA = K; g.klA = 1; g.csB = 1; g.klB = N; g.rsC = N; g.alpha = 1.0; g.beta = 0.0; g.ksplit = 1;
    return g;
}
hipError_t bwla_q_launch_gemm(QGemm g, size_t partial_bytes, hipStream_t st);

// ---------------------------------------------------------------- row kernels (quantizer_rows.hip)
hipError_t bwla_q_launch_convert_f32_f64(const float* src, double* dst, size_t count, hipStream_t st);
hipError_t bwla_q_launch_convert_f64_f32(const double* src, float* dst, size_t count, hipStream_t st);
// The steps of one launch over the rows of an n x m array, in this order (all on x = y, or y - its mean with CENTER):
//   CENTER    ybar = the row means, X = the centered rows (each may be NULL)
//   INIT      c, s2 started from x (otherwise read, where a step needs them)
//   NLL       part[i] = the row's share of -n m L_GMM at (c, s2)
//   EM        one update of c, s2
//   NLL_EM    part_em[i] = the same after it
//   GRAD      out = H[(x - m) / s2], m = c tanh(c x / s2)
//   TARGETS   out = (H m + ybar 1) / s2
// f32 (may be NULL) gets y itself.  out may be Y.
enum : unsigned { QROWS_CENTER = 1, QROWS_INIT = 2, QROWS_NLL = 4, QROWS_EM = 8, QROWS_NLL_EM = 16, QROWS_GRAD = 32,
                  QROWS_TARGETS = 64 };
struct QRows {
    const double* Y; int m; unsigned steps;
    double* c; double* s2; double s2_min;
    double* X; double* ybar; double* part; double* part_em; double* out; float* f32;
};
hipError_t bwla_q_launch_rows(const QRows& g, int n, hipStream_t st);
// nll = scale sum(part), nll_em (and nll_again) = scale sum(part_em), and the proximal step's factor to fac[0], with
// fac[1] = fac[2] = 0, as QGemm::coef takes it (scale = 1 / (n m)); part, part_em, nll_again, fac may be NULL
struct QRowsFinish {
    const double* part; const double* part_em; double* nll; double* nll_em; double* nll_again;
    const double* s2; double* fac; double mu, scale; int n;
};
hipError_t bwla_q_launch_rows_finish(const QRowsFinish& f, hipStream_t st);
// Q[i] = uniform in [-1, 1) from a counter-based hash of (seed, i)
hipError_t bwla_q_launch_fill_hash(double* Q, size_t count, uint32_t seed, hipStream_t st);
hipError_t bwla_q_launch_fill_identity(double* R, int n, hipStream_t st);
// X = C / ||C||_F (count values, one workgroup; a zero matrix stays zero)
hipError_t bwla_q_launch_scale_inv_frob(const double* C, int count, double* X, hipStream_t st);
// out[0] = 1 / sqrt(max_j sum_i |G_ij|) for a Gram matrix G = X^T X (nn x nn): a bound on 1 / sigma_max(X)
// (0 for a zero matrix); one workgroup
hipError_t bwla_q_launch_gram_inv_norm(const double* G, int nn, double* out, hipStream_t st);
// X[e] *= s[0]
hipError_t bwla_q_launch_scale_by(double* X, size_t count, const double* s, hipStream_t st);
// *done = 1 once max |G - I| <= tol (G nn x nn); never cleared
hipError_t bwla_q_launch_near_identity(const double* G, int nn, double tol, int* done, hipStream_t st);
hipError_t bwla_q_launch_set_int(int* p, int v, hipStream_t st);
hipError_t bwla_q_launch_fill_value(double* p, size_t count, double v, hipStream_t st);
// dst[e] = src[e]^pw (0 where src <= 0)
hipError_t bwla_q_launch_pow_vec(const double* src, double pw, int count, double* dst, hipStream_t st);
// dst[i][j] = src[i][j] * pow(lam[j], pw) (fp32 out, n x k; lam <= 0 gives 0)
hipError_t bwla_q_launch_scale_cols_f32(const double* src, const double* lam, double pw, int n, int k, float* dst,
                                        hipStream_t st);

// ---------------------------------------------------------------- one-sided Jacobi (quantizer_jacobi.hip)
// Singular value decomposition G = U S V^T of a square n x n matrix (n <= 256) by Hestenes'
// one-sided Jacobi rotations in one workgroup.  Outputs, ordered by descending singular value:
//   sig[j]        singular values
//   Ws[j][:]      column j of G V = s_j u_j            (n x n, row j = that column)
//   Vs[j][:]      s_j^pw * v_j                          (n x n, row j = that vector; s_j = 0 gives 0)
// `work` holds 2 n^2 doubles.  it (may be NULL): the bookkeeping of the subspace iteration, below.  The launch
// returns immediately when *skip != 0.
// sym: G is symmetric positive semidefinite (a Gram matrix G = B^T B); Ws is not available.  Up to 136 wide the
// sweeps run in LDS, on the Cholesky factor G = L L^T, and the rotations are not accumulated; sig are eigenvalues:
//   ortho         the columns of L^T are rotated into X S; Vs[j] = column j of L^-T X, or those of L into V S and
//                 Vs[j] = v_j / s_j where columns of B are not far apart, so that B Vs^T has orthonormal columns, which
//                 are the left singular vectors of B (without `it`, and for a B that is orthonormal to 1e-8: some
//                 such columns, and no sig); quick: without sweeps, X = I, and of `it` power alone
//   otherwise     the columns of L; Vs[j] = eigenvector j (pw is not looked at)
// Wider ones (without ortho) are rotated themselves, v_j being the normalized column j of G V.
//
// The subspace iteration on S = Y^T Y filters its block by T_2(2 S / theta - 1), the Chebyshev polynomial
// that is at most 1 on [0, theta] and grows fastest beyond (Rutishauser's simultaneous iteration, 1970),
// theta being the smallest Ritz value of the block.  QRitz is what a Jacobi call on the Gram matrix of the
// filtered block leaves for the next iteration: theta, the coefficients of the filter's two products
// (QGemm::coef), and how far the leading values moved.  power > 0 says that the filter is (S / power)^2 instead, power < 0 that it is S / -power and the second product
// of no account; wide that the Ritz values are far apart, and the first product is to be deflated (below).
struct QRitz { double first[3], second[3], theta, power, moved; int wide; };
struct QJacobi {
    const double* G; int n; double pw;
    double* sig; double* Ws; double* Vs; double* work;
    const int* skip;
    bool sym, ortho, quick;
    // With it: prev holds n doubles, the squared Ritz values of the iteration before, and is replaced; degree says
    // whether the block was multiplied by S (1) or filtered (2), scale what its Ritz values are to be multiplied
    // with in the first case.  From the third call on (call counts from 1) *done is set to `call` once the leading `lead` values have
    // settled: they moved by at most tol relative, or the block is by now where plain iterations would be when theirs have.
    QRitz* it; double* prev; int lead, degree, call; double tol, scale; int* done;
};
hipError_t bwla_q_launch_jacobi(const QJacobi& j, hipStream_t st);
// Where it->wide: takes out of each column j of U (m x p, a filter's first product of the orthonormal block Q) what it has of the columns of Q whose
// Ritz values are 100 times its own and more: rounding, as Q^T S Q is diagonal.  prev: the squared Ritz values.
hipError_t bwla_q_launch_deflate(const double* Q, double* U, int m, int p, const QRitz* it, const double* prev, const int* skip,
                                 hipStream_t st);
constexpr int BWLA_Q_JACOBI_LDS = 96;        // largest matrix whose two work arrays fit LDS
constexpr int BWLA_Q_JACOBI_SYM_LDS = 136;   // ... whose one array does (sym)

// ---------------------------------------------------------------- polar factors (quantizer_polar.hip)
// R = U V^T of C = U S V^T (n x n, n <= BWLA_Q_POLAR_MAX) by the Newton-Schulz iteration in one workgroup; *done = 1, or 0
// where it has not converged, which leaves R as it was (always: gives what it has).
constexpr int BWLA_Q_POLAR_MAX = 96;         // two matrices of that size fit LDS
hipError_t bwla_q_launch_polar(const double* C, int n, double* R, int* done, bool always, hipStream_t st);
