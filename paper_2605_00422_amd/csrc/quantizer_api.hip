// C ABI of the offline quantizer (paper App. A.1 Algorithm 2): validation and scratch layout on the
// host, then the sequence of launches -- fp64 GEMMs on strided views (quantizer_gemm.hip), row-wise
// mixture kernels (quantizer_rows.hip), one-sided Jacobi SVDs (quantizer_jacobi.hip).  Nothing
// here allocates or synchronizes; a call is a chain of launches on the caller's stream.
#include <math.h>

#include "quantizer_internal.h"

namespace {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t al256(size_t x) { return (x + 255u) & ~(size_t)255; }
constexpr size_t PART_BYTES = (size_t)64 << 20;   // partial products of split contractions

// Scratch layout.  big[0..4]: W in fp64, W - M, the half-rotated rows (W - M) R2 viewed as
// (n n1) x n2, the rotated rows, and the centered rows / the MM targets.
struct QPlan {
    int n, m, n1, n2, k, p, jn;
    size_t big[5], R1, R2, C, A, Bt, A2, Bt2, c, s2, rowpart, rowpart2, scal, norm, ritz, Q, Q2, Zs, G, Vs, Ws, sig, prev, lam,
        jwork, flags, partials, bytes;
};

bwla_status_t make_plan(int64_t n, int64_t m, int32_t n1, int32_t n2, int32_t k, QPlan& P) {
    if (n <= 0 || m <= 0 || n1 <= 0 || n2 <= 0 || k < 0) return BWLA_ERR_SHAPE;
    // n1 = n2 = 1 with m > 1 is the sizing of the calls that take no factors (bwla_q_truncate_rank)
    const bool no_factors = n1 == 1 && n2 == 1;
    if (!no_factors && (int64_t)n1 * n2 != m) return BWLA_ERR_SHAPE;
    if (k > n || k > m) return BWLA_ERR_SHAPE;
    if (n1 > 256 || n2 > 256 || k > 128 || n > 65535 || m > 65536) return BWLA_ERR_UNSUPPORTED;
    P.n = (int)n; P.m = (int)m; P.n1 = n1; P.n2 = n2; P.k = k;
    int p = k > 0 ? (2 * k > k + 16 ? 2 * k : k + 16) : 0;
    if (p > n) p = (int)n;
    if (p > m) p = (int)m;
    P.p = p;
    P.jn = p > n1 ? p : n1;
    if (n2 > P.jn) P.jn = n2;
    const size_t D = sizeof(double), nm = (size_t)n * m, jj = (size_t)P.jn * P.jn;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off = al256(off + bytes); return o; };
    for (int i = 0; i < 5; ++i) P.big[i] = take(nm * D);
    P.R1 = take((size_t)n1 * n1 * D); P.R2 = take((size_t)n2 * n2 * D); P.C = take(jj * D);
    P.A = take((size_t)n * k * D); P.Bt = take((size_t)m * k * D);
    P.A2 = take((size_t)n * k * D); P.Bt2 = take((size_t)m * k * D);
    P.c = take(n * D); P.s2 = take(n * D); P.rowpart = take(n * D); P.rowpart2 = take(n * D);
    P.scal = take(64 * D); P.norm = take(D); P.ritz = take(sizeof(QRitz));
    P.Q = take((size_t)m * p * D); P.Q2 = take((size_t)m * p * D); P.Zs = take((size_t)n * p * D);
    P.G = take(jj * D); P.Vs = take(jj * D); P.Ws = take(jj * D);
    P.sig = take(P.jn * D); P.prev = take(P.jn * D); P.lam = take(P.jn * D);
    P.jwork = take(2 * jj * D);
    P.flags = take(256);
    P.partials = take(PART_BYTES);
    P.bytes = off;
    return BWLA_OK;
}

struct Ctx {
    QPlan P; char* ws; hipStream_t st; hipError_t err = hipSuccess;
    double* d(size_t off) const { return reinterpret_cast<double*>(ws + off); }
    int* done() const { return reinterpret_cast<int*>(ws + P.flags); }
    void ck(hipError_t e) { if (err == hipSuccess && e != hipSuccess) err = e; }
};

void gemm(Ctx& x, QGemm g, const int* skip = nullptr) {
    g.partials = x.d(x.P.partials);
    g.skip = skip;
    x.ck(bwla_q_launch_gemm(g, PART_BYTES, x.st));
}

// dst_i = R1^T src_i for every row as an n1 x n2 matrix (transposed: R1 src_i); src must differ from dst
void rotate_left(Ctx& x, const double* R1, const double* src, bool transposed, double* dst) {
    const QPlan& P = x.P;
    QGemm b{};
    b.A = R1; b.B = src; b.C = dst; b.M = P.n1; b.N = P.n2; b.K = P.n1; b.batch = P.n;
    if (transposed) { b.rsA = P.n1; b.klA = 1; } else { b.rsA = 1; b.klA = P.n1; }
    b.bsA = 0; b.csB = 1; b.klB = P.n2; b.bsB = P.m; b.rsC = P.n2; b.bsC = P.m; b.alpha = 1.0; b.beta = 0.0;
    gemm(x, b);
}

// dst rows = src rows times R1 (x) R2 (transposed = false) or times its transpose R1^T (x) R2^T;
// half = the (n n1) x n2 intermediate src_i R2.  src may equal dst; half must differ from both.
// coef (may be NULL): times coef[0]
void rotate_rows(Ctx& x, const double* src, const double* R1, const double* R2, bool transposed, double* half,
                 double* dst, const double* coef = nullptr) {
    const QPlan& P = x.P;
    QGemm a = qgemm_plain(src, R2, half, P.n * P.n1, P.n2, P.n2);
    a.coef = coef;
    if (transposed) { a.csB = P.n2; a.klB = 1; }
    gemm(x, a);
    rotate_left(x, R1, half, transposed, dst);
}

// Wres = W - A Bt^T (returns W itself when k == 0)
const double* residual(Ctx& x, const double* W, const double* A, const double* Bt, double* Wres) {
    const QPlan& P = x.P;
    if (P.k == 0) return W;
    QGemm g{};
    g.A = A; g.B = Bt; g.C = Wres; g.C0 = W; g.M = P.n; g.N = P.m; g.K = P.k; g.batch = 1;
    g.rsA = P.k; g.klA = 1; g.csB = P.k; g.klB = 1; g.rsC = P.m; g.alpha = -1.0; g.beta = 1.0;
    gemm(x, g);
    return Wres;
}

// the steps `r` of the rows of big[3], or of others (steps that write an array get it from the caller)
void rows(Ctx& x, QRows r) {
    const QPlan& P = x.P;
    if (!r.Y) r.Y = x.d(P.big[3]);
    r.m = P.m; r.part = x.d(P.rowpart); r.part_em = x.d(P.rowpart2);
    x.ck(bwla_q_launch_rows(r, P.n, x.st));
}
QRows row_steps(unsigned steps, const double* c, const double* s2, double* out) {
    QRows r{};
    // (written by INIT and EM alone, which callers with arrays of their own to write ask for)
    r.steps = QROWS_CENTER | steps; r.c = const_cast<double*>(c); r.s2 = const_cast<double*>(s2); r.out = out;
    return r;
}

// big[1] = W - M (when k > 0), big[2] = half-rotated, big[3] = Y = (W - M) R
const double* rotated(Ctx& x, const double* W, const double* A, const double* Bt, const double* R1, const double* R2) {
    const QPlan& P = x.P;
    const double* Wres = residual(x, W, A, Bt, x.d(P.big[1]));
    rotate_rows(x, Wres, R1, R2, false, x.d(P.big[2]), x.d(P.big[3]));
    return Wres;
}

// Polar factors come from the Newton-Schulz iteration: up to BWLA_Q_POLAR_MAX in one workgroup, above as a few dozen
// small products.  Up to this size, which the one-sided Jacobi SVD does in half a millisecond (86: 3 ms, 128: 11 ms), that
// takes over where the iteration does not converge.
constexpr int POLAR_JACOBI_MAX = 64;
constexpr int POLAR_NS_PAIRS = 32;

// polar factor of the jn-sized scratch matrix C (nn x nn) into R
void polar(Ctx& x, int nn, double* R) {
    const QPlan& P = x.P;
    if (nn > BWLA_Q_POLAR_MAX) {
        // X <- X (3 I - X^T X) / 2 from X = C / ||C||_F: singular values in (0, 1] rise to 1 (by 3/2 per
        // step while small, then quadratically), the singular vectors stay: X -> U V^T.  Steps come in
        // pairs so that X is back in the same buffer after each; before a pair X^T X is compared with I,
        // and once it is within 1e-13 the remaining launches return at once.  A singular C never gets
        // there and leaves a finite matrix that is not orthogonal.
        double *Xa = x.d(P.Ws), *Xb = x.d(P.Vs), *G = x.d(P.G);
        int* done = x.done();
        x.ck(bwla_q_launch_set_int(done, 0, x.st));
        x.ck(bwla_q_launch_scale_inv_frob(x.d(P.C), nn * nn, Xa, x.st));
        auto step = [&](const double* src, double* dst) {
            QGemm g = qgemm_plain(src, src, G, nn, nn, nn);       // G = src^T src
            g.rsA = 1; g.klA = nn;
            gemm(x, g, done);
            QGemm u = qgemm_plain(src, G, dst, nn, nn, nn);       // dst = 1.5 src - 0.5 src G
            u.C0 = src; u.alpha = -0.5; u.beta = 1.5;
            gemm(x, u, done);
        };
        for (int it = 0; it < POLAR_NS_PAIRS; ++it) {
            if (it > 0) {
                QGemm g = qgemm_plain(Xa, Xa, G, nn, nn, nn);
                g.rsA = 1; g.klA = nn;
                gemm(x, g, done);
                x.ck(bwla_q_launch_near_identity(G, nn, 1.0e-13, done, x.st));
            }
            step(Xa, Xb);
            step(Xb, Xa);
        }
        x.ck(hipMemcpyAsync(R, Xa, (size_t)nn * nn * sizeof(double), hipMemcpyDeviceToDevice, x.st));
        return;
    }
    x.ck(bwla_q_launch_polar(x.d(P.C), nn, R, x.done(), nn > POLAR_JACOBI_MAX, x.st));
    if (nn > POLAR_JACOBI_MAX) return;
    QJacobi j{};
    j.G = x.d(P.C); j.n = nn; j.pw = -1.0; j.sig = x.d(P.sig); j.Ws = x.d(P.Ws); j.Vs = x.d(P.Vs); j.work = x.d(P.jwork);
    j.skip = x.done();
    x.ck(bwla_q_launch_jacobi(j, x.st));
    QGemm g = qgemm_plain(x.d(P.Ws), x.d(P.Vs), R, nn, nn, nn);
    g.rsA = 1; g.klA = nn;
    gemm(x, g, x.done());
}

// The Procrustes update of one factor, from half = (W - M) R2 (which = 1), W - M and R1 (2), and big[4] = the
// weighted targets of the rotated rows.  which = 2 leaves R1^T (W - M) in big[2].
void procrustes_held(Ctx& x, int which, const double* half, const double* Wres, const double* R1, double* Rnew) {
    const QPlan& P = x.P;
    double *left = x.d(P.big[2]), *T = x.d(P.big[4]);
    QGemm g{};
    g.batch = 1; g.alpha = 1.0; g.beta = 0.0; g.C = x.d(P.C);
    if (which == 1) {
        // C1[a][c] = sum_i sum_d (V_i R2)[a][d] (lambda_i T_i)[c][d]
        g.A = half; g.B = T; g.M = P.n1; g.N = P.n1; g.K = P.n * P.n2;
        g.rsA = P.n2; g.kdivA = P.n2; g.khA = P.m; g.klA = 1;
        g.csB = P.n2; g.kdivB = P.n2; g.khB = P.m; g.klB = 1;
        g.rsC = P.n1;
        gemm(x, g);
        polar(x, P.n1, Rnew);
    } else {
        // P_i = R1^T V_i, then C2[b][d] = sum_(i,c) P[(i,c)][b] (lambda_i T_i)[(i,c)][d]
        rotate_left(x, R1, Wres, false, left);
        g.A = left; g.B = T; g.M = P.n2; g.N = P.n2; g.K = P.n * P.n1;
        g.rsA = 1; g.klA = P.n2; g.csB = 1; g.klB = P.n2; g.rsC = P.n2;
        gemm(x, g);
        polar(x, P.n2, Rnew);
    }
}

// The same at (Wres, R1, R2, c, s2); expects nothing of the scratch.
void procrustes(Ctx& x, int which, const double* Wres, const double* R1, const double* R2, const double* c,
                const double* s2, double* Rnew) {
    const QPlan& P = x.P;
    rotate_rows(x, Wres, R1, R2, false, x.d(P.big[2]), x.d(P.big[3]));
    rows(x, row_steps(QROWS_TARGETS, c, s2, x.d(P.big[4])));
    procrustes_held(x, which, x.d(P.big[2]), Wres, R1, Rnew);
}

// rank-k truncation of Y (n x m) into A2 (n x k), Bt2 (m x k); lam gets the k leading eigenvalues
// of Y^T Y restricted to the block (sigma^2)
void truncate(Ctx& x, const double* Y, int iters, double tol, double* A2, double* Bt2, double* lam) {
    const QPlan& P = x.P;
    const int n = P.n, m = P.m, p = P.p, k = P.k;
    double *Q = x.d(P.Q), *Q2 = x.d(P.Q2), *Zs = x.d(P.Zs), *G = x.d(P.G), *Vs = x.d(P.Vs);
    int* done = x.done();
    x.ck(bwla_q_launch_set_int(done, 0, x.st));
    x.ck(bwla_q_launch_fill_hash(Q, (size_t)m * p, 12345u, x.st));
    auto gram = [&](const double* B, int rows, const int* skip) {      // G = B^T B, B rows x p
        QGemm g = qgemm_plain(B, B, G, p, p, rows);
        g.rsA = 1; g.klA = p;
        gemm(x, g, skip);
    };
    QJacobi eig{};
    eig.G = G; eig.n = p; eig.sig = x.d(P.sig); eig.Vs = Vs; eig.work = x.d(P.jwork);
    eig.sym = true;                                          // a Gram matrix
    auto ritz_step = [&]() {                                 // eigenvectors, eigenvalues to lam
        eig.ortho = false; eig.sig = lam;
        x.ck(bwla_q_launch_jacobi(eig, x.st));
    };
    // out = B Vs^T[:, :cols]; with `skip`, skipped in iterations behind the one (`but`) that set it
    auto times_vs = [&](const double* B, int rows, int cols, double* out, const int* skip, int but) {
        QGemm g = qgemm_plain(B, Vs, out, rows, cols, p);
        g.csB = p; g.klB = 1; g.skip_but = but;
        gemm(x, g, skip);
    };
    if (p > BWLA_Q_JACOBI_SYM_LDS) {
        // Blocks too wide for the one-workgroup eigensolver to hold in LDS (ranks above 68): the block is
        // orthonormalized by the Newton-Schulz iteration X <- X (3 I - X^T X) / 2 instead (tall GEMMs; it
        // converges to the orthogonal polar factor of the block, a basis of the same subspace), there are
        // no Ritz values along the way, so every one of the `iters` iterations runs, and the eigensolver is
        // called once, for the Rayleigh-Ritz step.
        auto ns_ortho = [&](double* src, double* dst) {                 // src is overwritten; result in dst
            x.ck(bwla_q_launch_set_int(done, 0, x.st));
            gram(src, m, nullptr);
            // (not to scal: a proximal step's factor waits there for the truncation to end)
            x.ck(bwla_q_launch_gram_inv_norm(G, p, x.d(P.norm), x.st));
            x.ck(bwla_q_launch_scale_by(src, (size_t)m * p, x.d(P.norm), x.st));
            auto step = [&](const double* a, double* b, const int* skip) {
                gram(a, m, skip);
                QGemm u = qgemm_plain(a, G, b, m, p, p);                  // b = 1.5 a - 0.5 a G
                u.C0 = a; u.alpha = -0.5; u.beta = 1.5;
                gemm(x, u, skip);
            };
            step(src, dst, nullptr);
            for (int pair = 0; pair < POLAR_NS_PAIRS; ++pair) {
                gram(dst, m, done);
                x.ck(bwla_q_launch_near_identity(G, p, 1.0e-13, done, x.st));
                step(dst, src, done);
                step(src, dst, done);
            }
        };
        ns_ortho(Q, Q2);
        double* cur = Q2; double* oth = Q;
        for (int it = 0; it < iters; ++it) {
            gemm(x, qgemm_plain(Y, cur, Zs, n, p, m));                   // Zs = Y Q
            QGemm t = qgemm_plain(Y, Zs, oth, m, p, n);                  // oth = Y^T Zs
            t.rsA = 1; t.klA = m;
            gemm(x, t);
            ns_ortho(oth, cur);
        }
        gemm(x, qgemm_plain(Y, cur, Zs, n, p, m));
        gram(Zs, n, nullptr);
        ritz_step();
        times_vs(Zs, n, k, A2, nullptr, 0);
        times_vs(cur, m, k, Bt2, nullptr, 0);
        return;
    }
    // Iterations: the block U <- S Q, or T_2(2 S / theta - 1) Q = (4 / theta) S U - 2 U - Q with
    // U = (2 / theta) S Q - Q, then Q <- U orthonormalized in the basis of its Ritz vectors.  The first is S Q of the random
    // start as it is (S Q spans the same whatever the basis of Q) and is orthonormalized without Ritz vectors, which are
    // worth nothing yet (500 us of sweeps); theta is not known there, and the second is S^2 Q, or S Q where its pivots are far apart.
    //
    // `iters` counts products with S.  What two of them multiply sigma_k^2 / sigma_{p+1}^2 = q by is q^2 plain and
    // 8 q^2 - 8 q + 1 filtered: the filter needs half as many up to q = 2.1, a third up to q = 1.2, and for any gap wider than
    // these 24 and 64 of them leave nothing to be done (19.5^12, 2.9^32).  So half or a third as many are made, which are
    // fewer launches that return at once too.  11008 x 4096, rank 32: 13 iterations of 560 us and 14 calls of the
    // eigensolver became 11 products of 280 in 6 iterations, 1400 empty launches some 346; the truncation's error, tol 1e-12, rank 32 of
    // 900 x 640, gaps of 2, 10 and 50 %: 4.8e-7, 2.2e-7, 8.1e-8 -> 1.9e-7, 7.4e-8, 3.3e-9.  Values far apart: quantizer_jacobi.hip.
    QRitz* ritz = reinterpret_cast<QRitz*>(x.ws + P.ritz);
    const int half_of = iters / 2 > 24 ? iters / 2 : 24, third_of = iters / 3 > 64 ? iters / 3 : 64;
    int budget = iters < half_of ? iters : half_of;
    if (third_of < budget) budget = third_of;
    if (budget > 2) budget |= 1;            // (one, and pairs of which the first may count for one: a spectrum far apart)
    QJacobi turn = eig;
    turn.ortho = true; turn.it = ritz; turn.prev = x.d(P.prev); turn.lead = k; turn.tol = tol; turn.done = done; turn.skip = done;
    auto apply = [&](const double* src, double* dst, const double* coef, const double* c0, const double* c1) {
        gemm(x, qgemm_plain(Y, src, Zs, n, p, m), done);                 // dst = Y^T (Y src), combined with c0, c1
        QGemm t = qgemm_plain(Y, Zs, dst, m, p, n);
        t.rsA = 1; t.klA = m; t.coef = coef; t.C0 = c0; t.C1 = c1;
        gemm(x, t, done);
    };
    for (int used = 0, call = 1; used < budget; ++call) {
        const bool two = used > 0 && used + 2 <= budget;
        apply(Q, Q2, two ? ritz->first : nullptr, two ? Q : nullptr, nullptr);
        if (two) {
            x.ck(bwla_q_launch_deflate(Q, Q2, m, p, ritz, x.d(P.prev), done, x.st));
            apply(Q2, Q2, ritz->second, Q2, Q);
        }
        gram(Q2, m, done);
        turn.degree = two ? 2 : 1; turn.call = call;
        turn.quick = used == 0;
        turn.scale = used == 0 ? sqrt(3.0 / m) : 1.0;                   // (the start's columns are some sqrt(m / 3) long)
        x.ck(bwla_q_launch_jacobi(turn, x.st));
        times_vs(Q2, m, p, Q, done, call);
        used += two ? 2 : 1;
    }
    // one more orthonormalization (of a block that hardly needs it any more), then Rayleigh-Ritz
    gram(Q, m, nullptr);
    eig.ortho = true;
    x.ck(bwla_q_launch_jacobi(eig, x.st));
    times_vs(Q, m, p, Q2, nullptr, 0);
    gemm(x, qgemm_plain(Y, Q2, Zs, n, p, m));
    gram(Zs, n, nullptr);
    ritz_step();
    times_vs(Zs, n, k, A2, nullptr, 0);
    times_vs(Q2, m, k, Bt2, nullptr, 0);
}

// M <- truncation of M - (1/mu) dL/dM; A, Bt in place.  big[3] holds the gradient's rows (QROWS_GRAD) at the rotated rows
// of W - M, scal the factor that goes with them.  identity: both factors are I; zero: M is 0.  Leaves the scratch's
// big arrays stale.
void psp(Ctx& x, double* A, double* Bt, const double* R1, const double* R2, bool identity, bool zero, int iters, double tol,
         double* lam) {
    const QPlan& P = x.P;
    double *Y = x.d(P.big[3]), *fac = x.d(P.scal);
    if (identity && zero) {
        // the proximal point is the factor times the gradient's rows as they stand: it goes into the truncation's result
        truncate(x, Y, iters, tol, x.d(P.A2), x.d(P.Bt2), lam);
        x.ck(bwla_q_launch_scale_by(x.d(P.A2), (size_t)P.n * P.k, fac, x.st));
        x.ck(bwla_q_launch_scale_by(lam, P.k, fac, x.st));
        x.ck(bwla_q_launch_scale_by(lam, P.k, fac, x.st));
    } else {
        rotate_rows(x, Y, R1, R2, true, x.d(P.big[2]), Y, fac);           // back through R^T, sign folded in
        if (!zero) {
            QGemm g{};                                                    // Y <- Y + A Bt^T: the proximal point
            g.A = A; g.B = Bt; g.C = Y; g.C0 = Y; g.M = P.n; g.N = P.m; g.K = P.k; g.batch = 1;
            g.rsA = P.k; g.klA = 1; g.csB = P.k; g.klB = 1; g.rsC = P.m; g.alpha = 1.0; g.beta = 1.0;
            gemm(x, g);
        }
        truncate(x, Y, iters, tol, x.d(P.A2), x.d(P.Bt2), lam);
    }
    x.ck(hipMemcpyAsync(A, x.d(P.A2), (size_t)P.n * P.k * sizeof(double), hipMemcpyDeviceToDevice, x.st));
    x.ck(hipMemcpyAsync(Bt, x.d(P.Bt2), (size_t)P.m * P.k * sizeof(double), hipMemcpyDeviceToDevice, x.st));
}

bwla_status_t open_ctx(Ctx& x, int64_t n, int64_t m, int32_t n1, int32_t n2, int32_t k, void* d_ws, size_t ws_bytes,
                       void* stream) {
    const bwla_status_t s = make_plan(n, m, n1, n2, k, x.P);
    if (s != BWLA_OK) return s;
    if (!d_ws) return BWLA_ERR_NULL;
    if (!aligned16(d_ws)) return BWLA_ERR_ALIGN;
    if (ws_bytes < x.P.bytes) return BWLA_ERR_BUFSIZE;
    x.ws = static_cast<char*>(d_ws);
    x.st = static_cast<hipStream_t>(stream);
    return BWLA_OK;
}
inline bwla_status_t finish(const Ctx& x) { return x.err == hipSuccess ? BWLA_OK : BWLA_ERR_HIP; }

}  // namespace

extern "C" {

bwla_status_t bwla_quantizer_workspace_size(int64_t n, int64_t m, int32_t n1, int32_t n2, int32_t k, size_t* bytes) {
    if (!bytes) return BWLA_ERR_NULL;
    QPlan P;
    const bwla_status_t s = make_plan(n, m, n1, n2, k, P);
    if (s != BWLA_OK) return s;
    *bytes = P.bytes;
    return BWLA_OK;
}

bwla_status_t bwla_q_okt_rows(const double* d_W, const double* d_A, const double* d_Bt, int32_t k, const double* d_R1,
                              const double* d_R2, int64_t n, int64_t m, int32_t n1, int32_t n2, double* d_X,
                              double* d_ybar, void* d_ws, size_t ws_bytes, void* stream) {
    if (!d_W || !d_R1 || !d_R2 || !d_X) return BWLA_ERR_NULL;
    if (k > 0 && (!d_A || !d_Bt)) return BWLA_ERR_NULL;
    if (!aligned16(d_W) || !aligned16(d_A) || !aligned16(d_Bt) || !aligned16(d_R1) || !aligned16(d_R2) ||
        !aligned16(d_X) || !aligned16(d_ybar))
        return BWLA_ERR_ALIGN;
    Ctx x;
    const bwla_status_t s = open_ctx(x, n, m, n1, n2, k, d_ws, ws_bytes, stream);
    if (s != BWLA_OK) return s;
    rotated(x, d_W, d_A, d_Bt, d_R1, d_R2);
    QRows r = row_steps(0, nullptr, nullptr, nullptr);
    r.X = d_X; r.ybar = d_ybar;
    rows(x, r);
    return finish(x);
}

// the steps of centered rows that the caller holds
static hipError_t rows_of(const double* d_X, int64_t n, int64_t m, unsigned steps, double s2_min, const double* d_c,
                          const double* d_s2, double* part, void* stream) {
    QRows r{};
    r.Y = d_X; r.m = (int)m; r.steps = steps; r.c = const_cast<double*>(d_c); r.s2 = const_cast<double*>(d_s2);
    r.s2_min = s2_min; r.part = part;
    return bwla_q_launch_rows(r, (int)n, static_cast<hipStream_t>(stream));
}

static bwla_status_t check_rows(const double* d_X, int64_t n, int64_t m, const double* d_c, const double* d_s2) {
    if (!d_X || !d_c || !d_s2) return BWLA_ERR_NULL;
    if (n <= 0 || m <= 0) return BWLA_ERR_SHAPE;
    if (n > 65535 || m > 65536) return BWLA_ERR_UNSUPPORTED;
    if (!aligned16(d_X) || !aligned16(d_c) || !aligned16(d_s2)) return BWLA_ERR_ALIGN;
    return BWLA_OK;
}

bwla_status_t bwla_q_init_theta(const double* d_X, int64_t n, int64_t m, double s2_min, double* d_c, double* d_s2,
                                void* stream) {
    const bwla_status_t s = check_rows(d_X, n, m, d_c, d_s2);
    if (s != BWLA_OK) return s;
    return rows_of(d_X, n, m, QROWS_INIT, s2_min, d_c, d_s2, nullptr, stream) == hipSuccess ? BWLA_OK : BWLA_ERR_HIP;
}

bwla_status_t bwla_q_em_step(const double* d_X, int64_t n, int64_t m, double s2_min, double* d_c, double* d_s2,
                             void* stream) {
    const bwla_status_t s = check_rows(d_X, n, m, d_c, d_s2);
    if (s != BWLA_OK) return s;
    return rows_of(d_X, n, m, QROWS_EM, s2_min, d_c, d_s2, nullptr, stream) == hipSuccess ? BWLA_OK : BWLA_ERR_HIP;
}

bwla_status_t bwla_q_gmm_nll(const double* d_X, int64_t n, int64_t m, const double* d_c, const double* d_s2,
                             double* d_out, void* d_ws, size_t ws_bytes, void* stream) {
    const bwla_status_t s = check_rows(d_X, n, m, d_c, d_s2);
    if (s != BWLA_OK) return s;
    if (!d_out || !d_ws) return BWLA_ERR_NULL;
    if (!aligned16(d_ws)) return BWLA_ERR_ALIGN;
    if (ws_bytes < (size_t)n * sizeof(double)) return BWLA_ERR_BUFSIZE;
    double* part = static_cast<double*>(d_ws);
    if (rows_of(d_X, n, m, QROWS_NLL, 0.0, d_c, d_s2, part, stream) != hipSuccess) return BWLA_ERR_HIP;
    QRowsFinish f{};
    f.part = part; f.nll = d_out; f.scale = 1.0 / ((double)n * (double)m); f.n = (int)n;
    return bwla_q_launch_rows_finish(f, static_cast<hipStream_t>(stream)) == hipSuccess ? BWLA_OK : BWLA_ERR_HIP;
}

bwla_status_t bwla_q_procrustes(int32_t which, const double* d_Wres, const double* d_R1, const double* d_R2,
                                const double* d_c, const double* d_s2, int64_t n, int64_t m, int32_t n1, int32_t n2,
                                double* d_Rnew, void* d_ws, size_t ws_bytes, void* stream) {
    if (!d_Wres || !d_R1 || !d_R2 || !d_c || !d_s2 || !d_Rnew) return BWLA_ERR_NULL;
    if (which != 1 && which != 2) return BWLA_ERR_SHAPE;
    if (!aligned16(d_Wres) || !aligned16(d_R1) || !aligned16(d_R2) || !aligned16(d_c) || !aligned16(d_s2) ||
        !aligned16(d_Rnew))
        return BWLA_ERR_ALIGN;
    Ctx x;
    const bwla_status_t s = open_ctx(x, n, m, n1, n2, 0, d_ws, ws_bytes, stream);
    if (s != BWLA_OK) return s;
    procrustes(x, which, d_Wres, d_R1, d_R2, d_c, d_s2, d_Rnew);
    return finish(x);
}

bwla_status_t bwla_q_svd_square(const double* d_G, int32_t nn, double* d_sig, double* d_Ut, double* d_Vt, void* d_ws,
                                size_t ws_bytes, void* stream) {
    if (!d_G || !d_ws) return BWLA_ERR_NULL;
    if (nn <= 0) return BWLA_ERR_SHAPE;
    if (nn > 256) return BWLA_ERR_UNSUPPORTED;
    if (!aligned16(d_G) || !aligned16(d_sig) || !aligned16(d_Ut) || !aligned16(d_Vt) || !aligned16(d_ws))
        return BWLA_ERR_ALIGN;
    if (ws_bytes < (size_t)2 * nn * nn * sizeof(double)) return BWLA_ERR_BUFSIZE;
    QJacobi j{};
    j.G = d_G; j.n = nn; j.pw = 0.0; j.sig = d_sig; j.Ws = d_Ut; j.Vs = d_Vt; j.work = static_cast<double*>(d_ws);
    return bwla_q_launch_jacobi(j, static_cast<hipStream_t>(stream)) == hipSuccess ? BWLA_OK : BWLA_ERR_HIP;
}

bwla_status_t bwla_q_truncate_rank(const double* d_Y, int64_t n, int64_t m, int32_t k, int32_t iters, double tol,
                                   double* d_A, double* d_Bt, double* d_sig, void* d_ws, size_t ws_bytes,
                                   void* stream) {
    if (!d_Y || !d_A || !d_Bt) return BWLA_ERR_NULL;
    if (k <= 0 || iters < 0) return BWLA_ERR_SHAPE;
    if (!aligned16(d_Y) || !aligned16(d_A) || !aligned16(d_Bt) || !aligned16(d_sig)) return BWLA_ERR_ALIGN;
    Ctx x;
    const bwla_status_t s = open_ctx(x, n, m, 1, 1, k, d_ws, ws_bytes, stream);   // no factors
    if (s != BWLA_OK) return s;
    truncate(x, d_Y, iters, tol, d_A, d_Bt, x.d(x.P.lam));
    if (d_sig) x.ck(bwla_q_launch_pow_vec(x.d(x.P.lam), 0.5, k, d_sig, x.st));
    return finish(x);
}

bwla_status_t bwla_q_psp_step(const double* d_W, double* d_A, double* d_Bt, int32_t k, const double* d_R1,
                              const double* d_R2, const double* d_c, const double* d_s2, int64_t n, int64_t m,
                              int32_t n1, int32_t n2, double mu, int32_t iters, double tol, void* d_ws, size_t ws_bytes,
                              void* stream) {
    if (!d_W || !d_A || !d_Bt || !d_R1 || !d_R2 || !d_c || !d_s2) return BWLA_ERR_NULL;
    if (k <= 0 || iters < 0) return BWLA_ERR_SHAPE;
    if (!aligned16(d_W) || !aligned16(d_A) || !aligned16(d_Bt) || !aligned16(d_R1) || !aligned16(d_R2) ||
        !aligned16(d_c) || !aligned16(d_s2))
        return BWLA_ERR_ALIGN;
    Ctx x;
    const bwla_status_t s = open_ctx(x, n, m, n1, n2, k, d_ws, ws_bytes, stream);
    if (s != BWLA_OK) return s;
    rotated(x, d_W, d_A, d_Bt, d_R1, d_R2);
    rows(x, row_steps(QROWS_GRAD, d_c, d_s2, x.d(x.P.big[3])));
    QRowsFinish f{};
    f.s2 = d_s2; f.fac = x.d(x.P.scal); f.mu = mu; f.scale = 1.0 / ((double)n * (double)m); f.n = (int)n;
    x.ck(bwla_q_launch_rows_finish(f, x.st));
    psp(x, d_A, d_Bt, d_R1, d_R2, false, false, iters, tol, x.d(x.P.lam));
    return finish(x);
}

bwla_status_t bwla_quantize_layer(const float* d_W, int64_t n, int64_t m, int32_t n1, int32_t n2, int32_t k,
                                  int32_t t_outer, double mu, double s2_min, int32_t svd_iters, double svd_tol,
                                  int32_t init_identity, float* d_R1, float* d_R2, float* d_W_rot, float* d_U,
                                  float* d_V, double* d_c, double* d_s2, double* d_hist, void* d_ws, size_t ws_bytes,
                                  void* stream) {
    if (!d_W || !d_R1 || !d_R2 || !d_W_rot) return BWLA_ERR_NULL;
    if (k > 0 && (!d_U || !d_V)) return BWLA_ERR_NULL;
    if (t_outer < 0 || svd_iters < 0 || !(s2_min > 0.0)) return BWLA_ERR_SHAPE;
    if (!aligned16(d_W) || !aligned16(d_R1) || !aligned16(d_R2) || !aligned16(d_W_rot) || !aligned16(d_U) ||
        !aligned16(d_V) || !aligned16(d_c) || !aligned16(d_s2) || !aligned16(d_hist))
        return BWLA_ERR_ALIGN;
    Ctx x;
    const bwla_status_t s = open_ctx(x, n, m, n1, n2, k, d_ws, ws_bytes, stream);
    if (s != BWLA_OK) return s;
    const QPlan& P = x.P;
    const size_t nm = (size_t)P.n * P.m;
    double *W = x.d(P.big[0]), *half = x.d(P.big[2]), *Y = x.d(P.big[3]), *T = x.d(P.big[4]);
    double *R1 = x.d(P.R1), *R2 = x.d(P.R2), *A = x.d(P.A), *Bt = x.d(P.Bt);
    double* c = d_c ? d_c : x.d(P.c);
    double* s2 = d_s2 ? d_s2 : x.d(P.s2);
    double* lam = x.d(P.lam);
    // The steps between two rotations run in one launch over the rows.  Behind it: L_GMM before its EM update to
    // d_hist[at], behind it to the next entry (and the one after, when there is no proximal step between), the step's factor
    auto row_work = [&](unsigned steps, double* out, int at, bool again, bool factor, float* f32, const double* of = nullptr) {
        QRows r = row_steps(steps | (d_hist && at >= 0 ? (unsigned)QROWS_NLL : 0u) |
                            (d_hist && (steps & QROWS_EM) ? (unsigned)QROWS_NLL_EM : 0u), c, s2, out);
        r.Y = of; r.s2_min = s2_min; r.f32 = f32;
        rows(x, r);
        if (!(r.steps & (QROWS_NLL | QROWS_NLL_EM)) && !factor) return;
        QRowsFinish f{};
        if (r.steps & QROWS_NLL) { f.part = x.d(P.rowpart); f.nll = d_hist + at; }
        if (r.steps & QROWS_NLL_EM) {
            f.part_em = x.d(P.rowpart2); f.nll_em = d_hist + at + 1;
            if (again) f.nll_again = d_hist + at + 2;
        }
        if (factor) { f.s2 = s2; f.fac = x.d(P.scal); f.mu = mu; }
        f.scale = 1.0 / ((double)P.n * P.m); f.n = P.n;
        x.ck(bwla_q_launch_rows_finish(f, x.st));
    };
    x.ck(bwla_q_launch_convert_f32_f64(d_W, W, nm, x.st));
    if (init_identity) {
        x.ck(bwla_q_launch_fill_identity(R1, n1, x.st));
        x.ck(bwla_q_launch_fill_identity(R2, n2, x.st));
    } else {
        x.ck(bwla_q_launch_convert_f32_f64(d_R1, R1, (size_t)n1 * n1, x.st));
        x.ck(bwla_q_launch_convert_f32_f64(d_R2, R2, (size_t)n2 * n2, x.st));
    }
    if (k > 0 && t_outer == 0) x.ck(bwla_q_launch_fill_value(lam, k, 0.0, x.st));       // M = 0, whatever A and Bt hold
    // From here on, at the top of a round, big[2] and big[3] belong to the current (M, R1, R2): half = (W - M) R2,
    // Y = (W - M) R.  What a step reads is made once and not again by the step behind it: the update of R1 takes half
    // and Y, and R2's half again, as R2 is still the old one (every step on its own rotated all rows anew: 7 rotations a
    // round, now 3.5, some 200 us each half on 11008 x 4096).
    // At the start M is 0, and with factors that start at the identity W is its own rotation.
    const double* Wres = W;
    const double *half_now = half, *Y_now = Y;
    if (init_identity) half_now = Y_now = W;
    else rotate_rows(x, W, R1, R2, false, half, Y);
    for (int t = 0; t < t_outer; ++t) {
        const unsigned em = QROWS_EM | (t == 0 ? (unsigned)QROWS_INIT : 0u);
        if (k > 0) {
            row_work(em | QROWS_GRAD, Y, 3 * t, false, true, nullptr, Y_now);
            psp(x, A, Bt, R1, R2, init_identity && t == 0, t == 0, svd_iters, svd_tol, lam);
            Wres = rotated(x, W, A, Bt, R1, R2);
            row_work(QROWS_TARGETS, T, 3 * t + 2, false, false, nullptr);
        } else {
            row_work(em | QROWS_TARGETS, T, 3 * t, true, false, nullptr, Y_now);
        }
        if (k > 0) half_now = half;
        procrustes_held(x, 1, half_now, Wres, R1, R1);
        rotate_left(x, R1, half_now, false, Y);
        half_now = half;
        Y_now = Y;
        row_work(QROWS_TARGETS, T, -1, false, false, nullptr);
        procrustes_held(x, 2, nullptr, Wres, R1, R2);
        if (k > 0 || t + 1 == t_outer) {
            // half = R1^T (W - M) of the update above: one product makes Y.  The next round's update of R1
            // needs (W - M) R2 there, which the proximal step makes when there is one
            gemm(x, qgemm_plain(half, R2, Y, P.n * P.n1, P.n2, P.n2));
        } else {
            rotate_rows(x, Wres, R1, R2, false, half, Y);
        }
    }
    // Y = (W - M)(R1 (x) R2) at the final factors, and L_GMM of it
    row_work(t_outer == 0 ? (unsigned)QROWS_INIT : 0u, nullptr, 3 * t_outer, false, false, d_W_rot, Y_now);
    x.ck(bwla_q_launch_convert_f64_f32(R1, d_R1, (size_t)n1 * n1, x.st));
    x.ck(bwla_q_launch_convert_f64_f32(R2, d_R2, (size_t)n2 * n2, x.st));
    if (k > 0) {
        // A = U_k S_k, Bt = V_k, lam = S_k^2: balanced factors V = U_k S_k^(1/2), U = V_k S_k^(1/2)
        x.ck(bwla_q_launch_scale_cols_f32(A, lam, -0.25, P.n, k, d_V, x.st));
        x.ck(bwla_q_launch_scale_cols_f32(Bt, lam, 0.25, P.m, k, d_U, x.st));
    }
    return finish(x);
}

}  // extern "C"
