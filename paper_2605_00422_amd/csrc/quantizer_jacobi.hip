// One-sided Jacobi SVD of a small square matrix in one workgroup (Hestenes' method): the orthogonal
// Procrustes updates of the OKT factors (paper App. A.2.2, "Alternating Procrustes Updates":
// R = U V^T from the SVD of an n1 x n1 or n2 x n2 matrix) and the small eigenproblems of the
// subspace iteration behind the truncated SVD of the proximal step (Sec. 3.2; App. A.2.3).
//
// The columns of G are kept as contiguous rows of a work array (column j = row j, in LDS padded to an
// even length so that a lane moves two elements at a time), V likewise.
// A sweep visits every pair of columns once, in the round-robin order of a tournament: n / 2
// disjoint pairs per round, n - 1 rounds.  A pair belongs to a group of lanes that holds both columns
// in registers (up to four elements per lane), takes their inner product, and applies the plane
// rotation that makes the two columns orthogonal to them and to the matching columns of V.  Up to
// n = 64 a group is one row of 16 lanes -- four pairs per wavefront, all pairs of a round at once,
// the inner product summed on DPP row operations alone, and the tournament is one of blocks of four
// columns whose sixteen pairs a wavefront takes in registers; larger matrices give a pair two rows (one
// lane exchange more) or a whole wavefront (row sums on DPP, the four rows added through lane reads).  Sweeps end when one has
// found nothing but pairs so nearly orthogonal that it leaves them so to 1e-15, or after 60.  At the end the column
// norms are the singular values, the normalized columns U, and V holds the right singular vectors.
// Up to n = 96 both arrays (2 n^2 doubles, at most 144 KiB) live in LDS, where a round costs an LDS
// round trip instead of an L2 one; larger matrices work in the caller's scratch (L2-resident).
// For a symmetric positive semidefinite matrix (the Gram matrices of the subspace iteration) V is not
// kept at all -- the sweeps work on a Cholesky factor, below -- so that matrices up to 136 wide fit LDS; there a
// pair takes two rows of lanes up to n = 128.
#include "bwla_internal.h"
#include "quantizer_internal.h"

namespace {

constexpr int JMAX = 256, JLDS = BWLA_Q_JACOBI_LDS, JLDS_SYM = BWLA_Q_JACOBI_SYM_LDS;
// threads of the workgroup: a row of 16 lanes per pair serves 32 pairs (n <= 64) with 512 threads
constexpr int jacobi_threads(int gw) { return gw == 16 ? 512 : 1024; }

template <int CTRL>
__device__ __forceinline__ double jdpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// sum over a row of 16 lanes, the same value in each of them
__device__ __forceinline__ double jrow_sum(double v) {
    v += jdpp<0xB1>(v);      // quad_perm [1,0,3,2]
    v += jdpp<0x4E>(v);      // quad_perm [2,3,0,1]
    v += jdpp<0x141>(v);     // row_half_mirror
    v += jdpp<0x140>(v);     // row_mirror
    return v;
}
__device__ __forceinline__ double jread(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
template <int GW>
__device__ __forceinline__ double jgroup_sum(double v) {
    v = jrow_sum(v);
    if (GW == 32) v += __shfl_xor(v, 16, 64);          // the other row of the pair's two
    if (GW == 64) v = (jread(v, 0) + jread(v, 16)) + (jread(v, 32) + jread(v, 48));
    return v;
}

// the value of the lane 16 (by32: 32) away under exclusive or: rows of lanes change places, by way of the LDS crossbar: a step is
// bound by the issue of some 110 vector instructions, and a swap of registers takes three for each of these
__device__ __forceinline__ double jrow_xor(double v, bool by32, int lane) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    if (by32) {
        const int from = (lane ^ 32) * 4;
        return __hiloint2double(__builtin_amdgcn_ds_bpermute(from, hi), __builtin_amdgcn_ds_bpermute(from, lo));
    }
    return __hiloint2double(__builtin_amdgcn_ds_swizzle(hi, 0x401f), __builtin_amdgcn_ds_swizzle(lo, 0x401f));
}

// 1 / x to a rounding or two: the hardware's estimate (2^-20 or better) and two Newton steps.  x normal, below 2^1021.
__device__ __forceinline__ double jrcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(fma(-x, y, 1.0), y, y);
    return y;
}

// Tangent t, cosine of the plane rotation that makes columns with squared norms al, be and inner product
// ga orthogonal; the sine is cs * t.  t = sign(d) g / (|d| + sqrt(d^2 + g^2)) with d = be - al, g = 2 ga, both
// scaled by the power of two of al + be, so that neither square overflows and one that underflows does not count.  The
// denominator is worked out in fp32: a tangent right to 2^-22 leaves that part of the inner product to the next sweep,
// which has the square of it to find anyway, and a sweep of steps is a chain of dependent instructions.  The cosine, which
// the columns' lengths hang on, is the hardware's estimate brought to full precision by Newton steps.  Geometric means of the largest
// errors over 136 matrices, 16 to 96 wide, normal, graded, of condition 1e14 and symmetric, the angle so / all of it in fp64: singular
// values 3.59e-15 / 3.61e-15 of the largest, U S V^T - G 1.80e-15 / 1.82e-15, V^T V - I 1.20e-14 / 1.22e-14; 64 x 64 with V 406 / 424 us.
__device__ __forceinline__ void jrotation(double al, double be, double ga, double& tt, double& cs) {
    const int e = __builtin_amdgcn_frexp_exp(al + be);
    const double d = ldexp(be - al, -e), g = ldexp(ga, 1 - e);
    const float df = fabsf((float)d), gf = (float)g;
    const float den = df + __builtin_amdgcn_sqrtf(fmaf(gf, gf, df * df));
    tt = g * copysign((double)__builtin_amdgcn_rcpf(den), d);
    const double w = fma(tt, tt, 1.0);                      // in [1, 2] (and some 2^-20)
    double y = __builtin_amdgcn_rsq(w);
#pragma unroll
    for (int i = 0; i < 2; ++i) {                           // y += y (1 - w y^2) / 2: full precision from 2^-20
        const double e = fma(-w * y, y, 1.0);
        y = fma(0.5 * y, e, y);
    }
    cs = y;
}

// Whether a rotation (tangent t; gg, nn the squares of the columns' inner product and of the product of their norms before it)
// leaves work to a further sweep.  A rotation changes the cosine between one of its columns and a third by t times that of the
// other, so a sweep that finds none of either beyond 3e-9 leaves none beyond 64 x 1e-17, and needs no further one to say so.
__device__ __forceinline__ bool jlarge(double t, double gg, double nn) { return fabs(t) > 3.0e-9 || gg > 1.0e-17 * nn; }

// GW: lanes per pair (16 for n <= 64, 32 for n <= 128, else 64); LDS: the work arrays live in dynamic LDS.
// ACCV: the rotations are accumulated into V.  Without it (a symmetric positive semidefinite G, whose
// left and right singular vectors coincide) the right singular vectors are the normalized columns of
// the rotated G themselves -- orthogonal to the tolerance of the sweeps, and as accurate as eigenvectors
// as the accumulated ones (both diagonalize G up to eps ||G||) -- at half the work and half the memory.
// In LDS (FACTOR) G = L L^T is factored first.  A Gram matrix of filtered columns is graded: the squares of their norms
// may be 1e20 apart.  Sweeps on G itself lose everything below eps ||G||; the columns of L^T carry the grading as
// scales of columns, which one-sided rotations keep out of the result's relative accuracy (Demmel and Veselic,
// 1992), and L^-T X orthonormalizes the block to eps times the condition of the columns scaled to length one.  Eigenvectors
// over roots of eigenvalues are right to eps of the largest column only: at 3e5 between the Ritz values the block was
// orthonormal to 1e-4, and the next filter lost it.  Columns of L^T are the less orthogonal to begin with, though, so that
// blocks whose columns are not far apart go by those of L and the eigenvectors over roots of eigenvalues.
// Times at 64 columns, 11008 x 4096: 57 us without sweeps, 420 for the first block with them (260 more by way of L^T), 260 to
// 200 for the later ones (25 more); 7 for one that is orthonormal already.  Sweeps on G itself: 420 and 400, 265 to 150, on plain blocks that are less graded.
template <int GW, bool LDS, bool ACCV>
__global__ __launch_bounds__(jacobi_threads(GW)) void jacobi_kernel(QJacobi a) {
    if (a.skip && *a.skip) return;
    constexpr int JT = jacobi_threads(GW), JW = JT / 64;
    constexpr bool FACTOR = LDS && !ACCV;
    bool rows = a.ortho;                                    // the sweeps rotate the columns of L^T, i.e. the rows of L
    const int n = a.n, t = threadIdx.x, lane = t & 63, w = t >> 6;
    extern __shared__ __align__(16) double jlds[];
    double* Wc = LDS ? jlds : a.work;
    const int ld = LDS ? (n + 1) & ~1 : n;                              // pitch of a column
    constexpr bool BLOCKED = GW == 16;                                  // (always in LDS)
    const int ncol = BLOCKED ? (n + 7) & ~7 : n;                        // columns, padded with zero ones
    double* Vc = Wc + (size_t)ncol * ld;
    __shared__ int rotated;
    __shared__ double sg[JMAX];                             // during the sweeps: squared norms of the columns
    __shared__ int ord[JMAX];
    __shared__ double di[FACTOR ? BWLA_Q_JACOBI_SYM_LDS : 1];           // 1 / L_jj
    __shared__ double iv[FACTOR ? BWLA_Q_JACOBI_SYM_LDS : 1];           // 1 / norms of the columns at the end
    for (int e = t; e < ncol * ld; e += JT) {
        const int j = e / ld, i = e - j * ld;
        Wc[e] = i < n && j < n ? a.G[(size_t)i * n + j] : 0.0;
        if (ACCV) Vc[e] = i == j ? 1.0 : 0.0;
    }
    // L^T for the triangular solve, column r = row r of L, behind Wc where LDS has room for both
    double* Lt = LDS && n <= JLDS ? Wc + (size_t)ncol * ld : a.work;
    const int ldt = n + 1;                                              // (a column of it is written across banks)
    constexpr int U = GW == 16 ? 1 : GW == 32 ? 2 : 3;                  // elements of a column per lane
    if constexpr (FACTOR) {
        if (a.ortho && !a.it) {
            // A block that is orthonormal to 1e-8 as it is: G^(-1/2) = I - (G - I) / 2 to the square of that, and no sweeps
            __syncthreads();
            if (t == 0) rotated = 0;
            __syncthreads();
            for (int e = t; e < n * n; e += JT) {
                const int j = e / n, i = e - j * n;
                if (!(fabs(Wc[(size_t)j * ld + i] - (i == j ? 1.0 : 0.0)) <= 1.0e-8)) rotated = 1;
            }
            __syncthreads();
            if (!rotated) {
                for (int e = t; e < n * n; e += JT) {
                    const int j = e / n, i = e - j * n;
                    a.Vs[e] = (i == j ? 1.5 : 0.0) - 0.5 * Wc[(size_t)j * ld + i];
                }
                return;                                                 // (sig is not asked for)
            }
        }
        // Four columns a step: every wavefront takes them into registers (rows in lanes) and factors them for itself, then each
        // updates its share of the columns right of them, one barrier a step.  A column keeps its entries below the diagonal and is
        // divided by the root of its pivot at the end.  A pivot that rounding has eaten (a Gram matrix singular to working
        // precision) counts as 1e-14 of the diagonal that it came from, and what is below it, which is as much noise as it
        // is, as nothing: without that, noise grows by squares from step to step.  (64 columns without sweeps, whole call: a column a
        // step 72 us, which was the latency of LDS and of the pivot 64 times over; so 57.)
        __syncthreads();
        for (int j = t; j < n; j += JT) sg[j] = 1.0e-14 * Wc[(size_t)j * ld + j];
        __syncthreads();
        if (a.ortho && !a.quick) {
            // columns of B up to 1e6 apart: eigenvectors over roots of eigenvalues leave B Vs^T orthonormal to 1e-10, and the columns
            // of L are the nearer to orthogonal
            double most = 0.0, least = 1.0e300;
            for (int j = lane; j < n; j += 64) {
                most = fmax(most, sg[j]);
                least = fmin(least, sg[j]);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                most = fmax(most, __shfl_xor(most, off, 64));
                least = fmin(least, __shfl_xor(least, off, 64));
            }
            rows = !(most <= 1.0e12 * least);
        }
        double pc[4][U], ps[4][U];                                      // a step's columns, and over their pivots
        // the entry of `row`, the same row in all lanes, of a column in registers
        auto entry = [&](const double (&c)[U], int row) {
            double v = c[0];
#pragma unroll
            for (int u = 1; u < U; ++u) v = row >= 64 * u ? c[u] : v;
            return jread(v, row & 63);
        };
        auto put_back = [&](int j0) {                                   // (of the step before: others may still have been reading)
#pragma unroll
            for (int c = 1; c < 4; ++c)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = lane + 64 * u;
                    if (j0 + c < n && i >= j0 + c && i < n) Wc[(size_t)(j0 + c) * ld + i] = pc[c][u];
                }
        };
        for (int j0 = 0; j0 < n; j0 += 4) {
            if (w == 0 && j0 > 0) put_back(j0 - 4);
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = lane + 64 * u;
                    pc[c][u] = j0 + c < n && i < n ? Wc[(size_t)(j0 + c) * ld + i] : 0.0;
                }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int j = j0 + c < n ? j0 + c : n - 1;
                const double piv = entry(pc[c], j), inv = j0 + c < n && piv > sg[j] && piv > 1.0e-300 ? jrcp(piv) : 0.0;
#pragma unroll
                for (int u = 0; u < U; ++u) ps[c][u] = pc[c][u] * inv;
#pragma unroll
                for (int d = c + 1; d < 4; ++d) {
                    const double f = entry(pc[c], j0 + d < n ? j0 + d : n - 1);
#pragma unroll
                    for (int u = 0; u < U; ++u) pc[d][u] = fma(-f, ps[c][u], pc[d][u]);
                }
            }
            for (int k0 = j0 + 4 + w; k0 < n; k0 += 4 * JW) {           // (four at a time so that their LDS reads overlap)
                double v[4][U];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int k = k0 + x * JW < n ? k0 + x * JW : n - 1;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = lane + 64 * u;
                        v[x][u] = Wc[(size_t)k * ld + (i < n ? i : 0)];
                    }
                }
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int k = k0 + x * JW < n ? k0 + x * JW : n - 1;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const double f = entry(pc[c], k);
#pragma unroll
                        for (int u = 0; u < U; ++u) v[x][u] = fma(-f, ps[c][u], v[x][u]);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = lane + 64 * u;
                        if (k0 + x * JW < n && i >= k && i < n) Wc[(size_t)k * ld + i] = v[x][u];
                    }
                }
            }
            __syncthreads();
        }
        if (w == 0) put_back((n - 1) & ~3);
        __syncthreads();
        for (int j = w; j < n; j += JW) {
            double* cj = Wc + (size_t)j * ld;
            const double piv = cj[j], floor = sg[j];
            const bool sound = piv > floor && piv > 1.0e-300;
            const double root = sqrt(sound ? piv : floor), inv = sound ? 1.0 / root : 0.0;
            for (int i = lane; i < n; i += 64) {
                const double l = i < j ? 0.0 : i == j ? root : cj[i] * inv;
                if (rows) Lt[(size_t)i * ldt + j] = l;
                else cj[i] = l;
            }
            if (lane == 0) di[j] = root > 0.0 ? 1.0 / root : 0.0;
        }
        __syncthreads();
        if (rows)
            for (int j = w; j < n; j += JW)
                for (int i = lane; i < n; i += 64) Wc[(size_t)j * ld + i] = a.quick ? (i == j ? 1.0 : 0.0) : Lt[(size_t)j * ldt + i];
        if (a.quick && w == 0) {
            // the next filter is (S / power)^2, power some size of the columns; or S / power, once, where pivots 1e5 apart say that
            // S^2 would leave nothing of the small directions
            double top = 0.0, most = 0.0, least = 1.0e300;
            for (int j = lane; j < n; j += 64) {
                top = fmax(top, sg[j]);
                most = fmax(most, di[j]);
                least = fmin(least, di[j]);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                top = fmax(top, __shfl_xor(top, off, 64));
                most = fmax(most, __shfl_xor(most, off, 64));
                least = fmin(least, __shfl_xor(least, off, 64));
            }
            top = top > 0.0 ? sqrt(1.0e14 * top) * a.scale : 1.0;
            const bool once = !(most <= 1.0e5 * least);
            if (lane < 3) {
                a.it->first[lane] = lane ? 0.0 : 1.0 / top;
                a.it->second[lane] = once ? (lane == 1 ? 1.0 : 0.0) : lane ? 0.0 : 1.0 / top;
            }
            if (lane == 0) {
                a.it->power = once ? -top : top;
                a.it->wide = 0;
            }
        }
    }
    const int np = (n + 1) & ~1;
    constexpr int GROUPS = JT / GW;
    const int gid = t / GW, sl = t % GW;
    // element pair u of a lane: in LDS two neighbours (16-byte accesses: 16 lanes cover all banks once;
    // single doubles had the wavefront's four columns meet in the same banks), else GW apart
    auto idx0 = [&](int u) { return LDS ? 2 * (sl + GW * u) : sl + 2 * GW * u; };
    constexpr int D = LDS ? 1 : GW;
    auto load = [&](const double* c, int u, bool live, double& e0, double& e1) {
        const int i = idx0(u);
        if (LDS) {
            double2 v = make_double2(0.0, 0.0);
            if (live && i < n) v = *reinterpret_cast<const double2*>(c + i);
            e0 = v.x; e1 = v.y;
        } else {
            e0 = live && i < n ? c[i] : 0.0;
            e1 = live && i + D < n ? c[i + D] : 0.0;
        }
    };
    auto store = [&](double* c, int u, double e0, double e1) {
        const int i = idx0(u);
        if (LDS) {
            if (i < n) *reinterpret_cast<double2*>(c + i) = make_double2(e0, e1);   // (the padding stays zero)
        } else {
            if (i < n) c[i] = e0;
            if (i + D < n) c[i + D] = e1;
        }
    };
    // one pair of columns through memory, by the GW lanes of a group (all lanes of the workgroup call it)
    auto pair = [&](int p, int q, bool live) {
        double* xp = Wc + (size_t)p * ld;
        double* yp = Wc + (size_t)q * ld;
        double x[4], y[4];
        double al = sg[p], be = sg[q < ncol ? q : 0];
        double ga = 0.0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            load(xp, u, live, x[2 * u], x[2 * u + 1]);
            load(yp, u, live, y[2 * u], y[2 * u + 1]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) ga += x[u] * y[u];
        ga = jgroup_sum<GW>(ga);
        if (ga * ga > al * be) {                            // carried norms that cancellation has spoilt
            al = be = 0.0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                al += x[u] * x[u];
                be += y[u] * y[u];
            }
            al = jgroup_sum<GW>(al);
            be = jgroup_sum<GW>(be);
        }
        // (|ga| > 1e-15 sqrt(al be), without the root)
        if (live && al > 0.0 && be > 0.0 && ga * ga > 1.0e-30 * (al * be)) {
            double tt, cs;
            jrotation(al, be, ga, tt, cs);
            const double sn = cs * tt;
            double* vp = Vc + (size_t)p * ld;
            double* vq = Vc + (size_t)q * ld;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                store(xp, u, cs * x[2 * u] - sn * y[2 * u], cs * x[2 * u + 1] - sn * y[2 * u + 1]);
                store(yp, u, sn * x[2 * u] + cs * y[2 * u], sn * x[2 * u + 1] + cs * y[2 * u + 1]);
                if (ACCV) {
                    double a0, a1, b0, b1;
                    load(vp, u, true, a0, a1);
                    load(vq, u, true, b0, b1);
                    store(vp, u, cs * a0 - sn * b0, cs * a1 - sn * b1);
                    store(vq, u, sn * a0 + cs * b0, sn * a1 + cs * b1);
                }
            }
            if (sl == 0) {
                const double c2 = cs * cs, g2 = 2.0 * tt * ga, t2 = tt * tt;
                sg[p] = c2 * (al - g2 + t2 * be);
                sg[q] = c2 * (be + g2 + t2 * al);
                if (jlarge(tt, ga * ga, al * be)) rotated = 1;
            }
        } else if (live && sl == 0 && (al < 0.0 || be < 0.0)) {
            rotated = 1;
        }
    };
    // position i of a tournament of m (even): 0 stays, the others move on by one per round
    auto at = [](int i, int round, int m) {
        const int v = i - 1 - round;
        return i == 0 ? 0 : 1 + (v < 0 ? v + m - 1 : v);
    };
    __syncthreads();
    for (int sweep = 0; sweep < 60 && !a.quick; ++sweep) {
        if (t == 0) rotated = 0;
        // Squared norms: taken anew at the start of a sweep, carried along by the rotations within it (their
        // error is then that of a sweep's rotations, and a sweep that rotates nothing, the one that ends the
        // loop, has tested every pair on exact ones).  A rotation so needs one inner product instead of three.
        // Against an 80-bit SVD (16 to 86 columns: normal, graded over twelve decades, of half rank, of condition
        // 1e14, Gram matrices of that condition) the largest errors, relative to the largest singular value, are with
        // carried norms / norms summed for every pair: singular values 1.7e-14 / 1.7e-14, V^T V - I
        // 5.5e-14 / 5.5e-14, U S V^T - G 6.0e-15 / 6.1e-15; 64 x 64 with V, times of one card, 484 / 516 us.
        for (int base = 0; base < ncol; base += GROUPS) {
            const int j = base + gid;
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                double e0, e1;
                load(Wc + (size_t)(j < n ? j : 0) * ld, u, j < n, e0, e1);
                s += e0 * e0;
                s += e1 * e1;
            }
            s = jgroup_sum<GW>(s);
            if (j < ncol && sl == 0) sg[j] = s;
        }
        __syncthreads();
        if constexpr (BLOCKED) {
            // Blocks of four columns.  Within the blocks: three rounds through LDS, column i with i ^ r.
            for (int r = 1; r < 4; ++r) {
                const int p = 4 * (gid >> 1) + ((gid & 1) ? (r == 1 ? 2 : 1) : 0);
                const bool live = p < ncol;
                pair(live ? p : 0, live ? p ^ r : 0, live);
                __syncthreads();
            }
            // Between blocks: a tournament of the blocks, a wavefront per pair of them.  It keeps the eight
            // columns in registers over all sixteen pairs -- four rounds, between which the rows of lanes pass
            // the second block's columns round (g ^ 1, g ^ 3, g ^ 2) -- so that LDS and the barrier are met
            // once in four rounds (64 x 64 with V, whole call: 593 -> 408 us; Gram matrices of 64 columns, on average, 395 -> 280).
            const int nb = ncol >> 2, g4 = lane >> 4;
            for (int round = 0; round < nb - 1; ++round) {
                if (w < nb / 2) {
                    const int cx = 4 * at(w, round, nb) + g4, by = 4 * at(nb - 1 - w, round, nb);
                    double x[4], y[4], vx[4], vy[4];
                    double nx = sg[cx], ny = sg[by + g4];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        load(Wc + (size_t)cx * ld, u, true, x[2 * u], x[2 * u + 1]);
                        load(Wc + (size_t)(by + g4) * ld, u, true, y[2 * u], y[2 * u + 1]);
                        if (ACCV) {
                            load(Vc + (size_t)cx * ld, u, true, vx[2 * u], vx[2 * u + 1]);
                            load(Vc + (size_t)(by + g4) * ld, u, true, vy[2 * u], vy[2 * u + 1]);
                        }
                    }
                    bool any = false;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (k > 0) {
                            const bool by32 = k == 2;
                            ny = jrow_xor(ny, by32, lane);
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                y[u] = jrow_xor(y[u], by32, lane);
                                if (ACCV) vy[u] = jrow_xor(vy[u], by32, lane);
                            }
                        }
                        const double ga = jrow_sum((x[0] * y[0] + x[1] * y[1]) + (x[2] * y[2] + x[3] * y[3]));
                        const double gg = ga * ga;
                        double nn = nx * ny;
                        if (!(gg <= nn) || nx < 0.0) {                  // carried norms that cancellation has spoilt
                            nx = jrow_sum((x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]));
                            ny = jrow_sum((y[0] * y[0] + y[1] * y[1]) + (y[2] * y[2] + y[3] * y[3]));
                            nn = nx * ny;
                        }
                        if (gg > 1.0e-30 * nn) {                        // (never for a zero column)
                            double tt, cs;
                            jrotation(nx, ny, ga, tt, cs);
                            const double sn = cs * tt, moves = tt * ga;
                            any |= jlarge(tt, gg, nn);
                            // (of the exact angle; off it by the tangent's 2^-22 of what moves, until norms are taken anew)
                            nx -= moves;
                            ny += moves;
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const double xu = x[u], yu = y[u];
                                x[u] = cs * xu - sn * yu;
                                y[u] = sn * xu + cs * yu;
                                if (ACCV) {
                                    const double vu = vx[u], wu = vy[u];
                                    vx[u] = cs * vu - sn * wu;
                                    vy[u] = sn * vu + cs * wu;
                                }
                            }
                        }
                    }
                    const int cy = by + (g4 ^ 2);                       // whose column the last exchange left here
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        store(Wc + (size_t)cx * ld, u, x[2 * u], x[2 * u + 1]);
                        store(Wc + (size_t)cy * ld, u, y[2 * u], y[2 * u + 1]);
                        if (ACCV) {
                            store(Vc + (size_t)cx * ld, u, vx[2 * u], vx[2 * u + 1]);
                            store(Vc + (size_t)cy * ld, u, vy[2 * u], vy[2 * u + 1]);
                        }
                    }
                    if (sl == 0) {
                        sg[cx] = nx;
                        sg[cy] = ny;
                        if (any) rotated = 1;
                    }
                }
                __syncthreads();
            }
        } else {
            for (int round = 0; round < np - 1; ++round) {
                for (int base = 0; base < np / 2; base += GROUPS) {    // the same trip count in every lane
                    const int pr = base + gid;
                    int p = 0, q = 0;
                    bool live = pr < np / 2;
                    if (live) {
                        p = at(pr, round, np);
                        q = at(np - 1 - pr, round, np);
                        live = p < n && q < n;                          // else the bye of an odd n
                        if (p > q) { const int s = p; p = q; q = s; }
                    }
                    pair(p, q, live);
                }
                __syncthreads();
            }
        }
        if (!rotated) break;
        __syncthreads();
    }
    for (int j = w; j < n; j += JW) {
        double s = 0.0;
        for (int e = lane; e < n; e += 64) s += Wc[(size_t)j * ld + e] * Wc[(size_t)j * ld + e];
        s = jgroup_sum<64>(s);
        if (lane == 0) sg[j] = FACTOR ? s : sqrt(s);
    }
    __syncthreads();
    for (int j = t; j < n; j += JT) {
        if (FACTOR) iv[j] = sg[j] > 0.0 ? 1.0 / sqrt(sg[j]) : 0.0;
        int rank = 0;
        for (int i = 0; i < n; ++i) rank += (sg[i] > sg[j] || (sg[i] == sg[j] && i < j)) ? 1 : 0;
        ord[rank] = j;
    }
    __syncthreads();
    if (FACTOR && rows) {
        // L^T M = X, eight right sides a wavefront, their rows in lanes, from the last row up
        for (int j0 = 8 * w; j0 < n; j0 += 8 * JW) {
            double x[8][U];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int j = ord[j0 + q < n ? j0 + q : n - 1];
                const double inv = iv[j];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = lane + 64 * u;
                    x[q][u] = i < n ? inv * Wc[(size_t)j * ld + i] : 0.0;
                }
            }
            double row[U], d = di[n - 1];
            auto fetch = [&](int r, double (&to)[U]) {
#pragma unroll
                for (int u = 0; u < U; ++u) to[u] = lane + 64 * u < r ? Lt[(size_t)r * ldt + lane + 64 * u] : 0.0;
            };
            fetch(n - 1, row);
            for (int r = n - 1; r >= 0; --r) {
                double next[U], dn = 0.0;
                if (r > 0) {
                    fetch(r - 1, next);
                    dn = di[r - 1];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    double v = x[q][0];
#pragma unroll
                    for (int u = 1; u < U; ++u) v = r >= 64 * u ? x[q][u] : v;
                    const double m = jread(v, r & 63) * d;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const double kept = fma(-row[u], m, x[q][u]);
                        x[q][u] = lane + 64 * u == r ? m : kept;
                    }
                }
                if (r > 0) {
#pragma unroll
                    for (int u = 0; u < U; ++u) row[u] = next[u];
                    d = dn;
                }
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = lane + 64 * u;
                    if (j0 + q < n && i < n) a.Vs[(size_t)(j0 + q) * n + i] = x[q][u];
                }
        }
    } else {
        for (int jj = w; jj < n; jj += JW) {
            const int j = ord[jj];
            const double s = sg[j];
            double scale = 0.0;
            if (s > 0.0) {
                if (FACTOR) scale = a.ortho ? iv[j] * iv[j] : iv[j];
                else scale = (a.pw == 0.0 ? 1.0 : pow(s, a.pw)) / (ACCV ? 1.0 : s);
            }
            for (int e = lane; e < n; e += 64) {
                if (a.Ws) a.Ws[(size_t)jj * n + e] = Wc[(size_t)j * ld + e];
                if (a.Vs) a.Vs[(size_t)jj * n + e] = scale * (ACCV ? Vc[(size_t)j * ld + e] : Wc[(size_t)j * ld + e]);
            }
        }
    }
    if (a.sig)
        for (int jj = t; jj < n; jj += JT) a.sig[jj] = sg[ord[jj]];
    if (a.it && !a.quick && w == 0) {
        // Ritz values of S out of the eigenvalues sg of the filtered block's Gram matrix
        const double theta = a.it->theta, power = a.it->power, before = a.it->moved;
        auto ritz = [&](int jj) {
            const double r = sqrt(sg[ord[jj]]);
            if (a.degree == 1) return r * a.scale;
            if (power < 0.0) return -power * r;
            if (power > 0.0) return power * sqrt(r);
            return 0.5 * theta * (sqrt(0.5 * (r + 1.0)) + 1.0);         // r = 2 x^2 - 1, x = 2 l / theta - 1
        };
        double moved = 0.0;
        for (int jj = lane; jj < n; jj += 64) {
            const double l = ritz(jj), l2 = l * l;
            if (jj < a.lead) moved = fmax(moved, fabs(l2 - a.prev[jj]) / fmax(l2, 1.0e-300));
            a.prev[jj] = l2;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) moved = fmax(moved, __shfl_xor(moved, off, 64));
        if (lane == 0) {
            const double top = ritz(0), next = ritz(n - 1);
            // Values of a filtered block are those of the block before it, to the square of an angle.  So the movement is the error e
            // that the block two calls back had, and this one's is two quotients of movements smaller.  Plain iterations that
            // stop with a movement of at most tol return the block behind it, one product on: with a quotient f = (theta / l_k)^2 a
            // product their e lies between f^2 tol and f tol, by where the last movement has fallen.  Where this one's is not above
            // the smaller of them it is as near as any of theirs.  (The first call has no values; a quotient takes two movements, and
            // counts as no smaller than the filter can make it, T_2(2 l_k / theta - 1)^-2: the first blocks' need not be of a kind.)
            const double gap = next / ritz(a.lead < n ? a.lead - 1 : n - 1), gap2 = gap * gap;
            const double xk = 2.0 / gap - 1.0, tk = 2.0 * xk * xk - 1.0, rate = fmax(moved / before, 1.0 / (tk * tk));
            const bool still = a.call >= 3 && moved <= a.tol;
            const bool there = a.call >= 4 && rate <= 0.5 && moved * rate * rate <= gap2 * gap2 * a.tol;
            if (still || there) *a.done = a.call;
            // A product leaves eps top of the largest direction in every column, T_2 so eps (2 top / theta)^2 of it, which
            // orthonormalizing takes out as long as that is small against one.  With values further apart (wide) what the first
            // of the two products has left is taken out before the second, which is eps (2 top / theta) then.  Where theta is all
            // rounding, a block of lower rank, it is multiplied by S^2, deflated likewise: nothing is asked of theta.
            // (Singular values k to 3000 apart had gone by S^2, whose products are not worth more than plain ones, and 1e4 apart
            // and more lost the small ones in it: one of 1e4 over a bulk of 1, rank 8 of 400 x 300, 2 % behind the rank, 66 products in
            // place of 200, energy lost beyond the best's 4.5e-3, now 6e-16 and plain
            // ones 1.8e-14.)
            const bool cheb = next > 0.0 && next >= 1.0e-13 * top;
            const double inv = cheb ? 1.0 / next : top > 0.0 ? 1.0 / top : 0.0;
            a.it->theta = next;
            a.it->power = cheb ? 0.0 : top;
            a.it->wide = next >= 1.0e-6 * top ? 0 : 1;
            a.it->moved = moved;
            a.it->first[0] = cheb ? 2.0 * inv : inv;
            a.it->first[1] = cheb ? -1.0 : 0.0;
            a.it->first[2] = 0.0;
            a.it->second[0] = cheb ? 4.0 * inv : inv;
            a.it->second[1] = cheb ? -2.0 : 0.0;
            a.it->second[2] = cheb ? -1.0 : 0.0;
        }
    }
}

// A workgroup a column of U: its products with the columns of Q in front, rows shared by the wavefronts and columns in lanes, then
// the rows again less those.  Returns at once but for wide blocks.
constexpr int DT = 512, DU = (BWLA_Q_JACOBI_SYM_LDS + 63) / 64;
__global__ __launch_bounds__(DT) void deflate_kernel(const double* Q, double* U, int m, int p, const QRitz* it, const double* prev,
                                                     const int* skip) {
    if (*skip || !it->wide) return;
    __shared__ double part[DT / 64][64 * DU];
    const int j = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double mine = prev[j];
    double e[DU];
    bool front[DU], any = false;
#pragma unroll
    for (int u = 0; u < DU; ++u) {
        const int i = lane + 64 * u;
        front[u] = i < j && prev[i < j ? i : j] > 1.0e4 * mine;
        any |= front[u];
        e[u] = 0.0;
    }
    if (__ballot(any) == 0) return;                         // (the same in every wavefront)
    for (int r = w; r < m; r += DT / 64) {
        const double v = U[(size_t)r * p + j];
#pragma unroll
        for (int u = 0; u < DU; ++u)
            if (front[u]) e[u] = fma(Q[(size_t)r * p + lane + 64 * u], v, e[u]);
    }
#pragma unroll
    for (int u = 0; u < DU; ++u) part[w][lane + 64 * u] = e[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < DU; ++u) {
        e[u] = 0.0;
        for (int i = 0; i < DT / 64; ++i) e[u] += part[i][lane + 64 * u];
    }
    for (int r = w; r < m; r += DT / 64) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < DU; ++u)
            if (front[u]) s = fma(Q[(size_t)r * p + lane + 64 * u], e[u], s);
        s = jgroup_sum<64>(s);
        if (lane == 0) U[(size_t)r * p + j] -= s;
    }
}

}  // namespace

hipError_t bwla_q_launch_jacobi(const QJacobi& j, hipStream_t st) {
    if (j.n < 1 || j.n > JMAX) return hipErrorInvalidValue;
    const bool in_lds = j.n <= (j.sym ? JLDS_SYM : JLDS);
    const size_t cols = j.n <= 64 ? (j.n + 7) & ~7 : j.n, one = cols * ((j.n + 1) & ~1);
    const size_t second = j.n > JLDS ? 0 : j.sym ? (size_t)j.n * (j.n + 1) : one;           // L^T, or V
    const size_t lds = in_lds ? (one + second) * sizeof(double) : 0;
    auto launch = [&](auto kern, int threads) {
        if (lds > 48 * 1024) {
            const hipError_t e = bwla_ensure_lds((const void*)kern, lds + 8192);             // (and what it holds statically)
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3(1), dim3(threads), lds, st, j);
        return hipGetLastError();
    };
    if (j.sym) {
        if (j.n <= 64) return launch(jacobi_kernel<16, true, false>, jacobi_threads(16));
        if (j.n <= 128) return launch(jacobi_kernel<32, true, false>, jacobi_threads(32));
        if (in_lds) return launch(jacobi_kernel<64, true, false>, jacobi_threads(64));
        return launch(jacobi_kernel<64, false, false>, jacobi_threads(64));
    }
    if (j.n <= 64) return launch(jacobi_kernel<16, true, true>, jacobi_threads(16));
    if (in_lds) return launch(jacobi_kernel<64, true, true>, jacobi_threads(64));
    return launch(jacobi_kernel<64, false, true>, jacobi_threads(64));
}

hipError_t bwla_q_launch_deflate(const double* Q, double* U, int m, int p, const QRitz* it, const double* prev, const int* skip,
                                 hipStream_t st) {
    if (p < 1 || p > BWLA_Q_JACOBI_SYM_LDS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(deflate_kernel, dim3(p), dim3(DT), 0, st, Q, U, m, p, it, prev, skip);
    return hipGetLastError();
}
