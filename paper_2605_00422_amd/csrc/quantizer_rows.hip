// Row-wise steps of the offline quantizer (paper App. A.1 Algorithm 2; App. A.2.2 for the mixture,
// its EM updates and the MM targets; App. A.2.3 for the gradient behind the proximal step), fp64.
// One workgroup per weight row, and one kernel for all of them: a launch runs the steps that follow one another
// on the same row -- center, start or update the mixture, its likelihood before and after, then the targets or the
// gradient -- with the row in registers, so that a row is read once and written once however many steps there are.
// Sums are taken per thread in a fixed order, then over the wavefront by butterflies and over the wavefronts in
// wavefront order, so that a result does not depend on the launch.
#include "bwla_internal.h"
#include "quantizer_internal.h"

namespace {

constexpr int RT = 256;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
// sum over the workgroup of T threads, returned to every thread; `sh` holds T / 64 doubles
template <int T = RT>
__device__ __forceinline__ double block_sum(double v, double* sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < T / 64; i += 4) s += (sh[i] + sh[i + 1]) + (sh[i + 2] + sh[i + 3]);
    return s;
}

__global__ void convert_f32_f64_kernel(const float* src, double* dst, size_t count) {
    for (size_t e = (size_t)blockIdx.x * RT + threadIdx.x; e < count; e += (size_t)gridDim.x * RT) dst[e] = (double)src[e];
}
__global__ void convert_f64_f32_kernel(const double* src, float* dst, size_t count) {
    for (size_t e = (size_t)blockIdx.x * RT + threadIdx.x; e < count; e += (size_t)gridDim.x * RT) dst[e] = (float)src[e];
}

// e = exp(-y) and rest = 1 - exp(-y), y = 2 |c x| / s^2, both right to some roundings of their own size; with them
// 2 r^+ - 1 = tanh(c x / s^2) = rest / (1 + e): the two densities' ratio is exp(2 c x / s^2) (App. A.2.2, E step).  The likelihood
// takes e and everything else the quotient, so one exponential an entry and state of the mixture serves all steps.
// exp(-y) = 2^-k (1 + p) with k = y / ln 2 to the nearest integer and p = exp(k ln 2 - y) - 1 by its Taylor series to the thirteenth
// power (what follows is 1.2e-17 of p); rest from p, as 1 - e would be off by a rounding of one: with c = 1e-8 s that was 5e-11 of the
// next c.  (Launches at 11008 x 4096, 154, 128, 174 and 320 us with a call of exp and 1 - e: 162, 135,
// 178 and 335.)
__device__ __forceinline__ void mix_exp(double x, double c, double inv, double& e, double& rest) {
    double y = 2.0 * fabs(c * x * inv);
    y = y > 800.0 ? 800.0 : y;                              // (exp(-800) is 0; a NaN stays)
    const double k = rint(y * 1.4426950408889634);
    const double r = fma(k, 2.3190468138462996e-17, fma(k, 0.69314718055994531, -y));    // ln 2 in two parts
    constexpr double inverse_factorial[12] = {1.0 / 6227020800, 1.0 / 479001600, 1.0 / 39916800, 1.0 / 3628800, 1.0 / 362880, 1.0 / 40320,
                                              1.0 / 5040,       1.0 / 720,       1.0 / 120,      1.0 / 24,      1.0 / 6,      1.0 / 2};
    double q = inverse_factorial[0];
#pragma unroll
    for (int i = 1; i < 12; ++i) q = fma(q, r, inverse_factorial[i]);
    const double p = fma(q * r, r, r), s = ldexp(1.0, -(int)k);
    e = fma(s, p, s);
    rest = fma(-s, p, 1.0 - s);
}
__device__ __forceinline__ double mix_resp(double e, double rest, double x, double c) {
    const double d = 1.0 + e;                               // in [1, 2]
    double y = __builtin_amdgcn_rcp(d);                     // 2^-20 or better, and two Newton steps
    y = fma(fma(-d, y, 1.0), y, y);
    y = fma(fma(-d, y, 1.0), y, y);
    double t = rest * y;
    t = fma(fma(-t, d, rest), y, t);
    return c * x < 0.0 ? -t : t;
}

// A row of T threads with E entries each in registers (thread t holds entries t, t + T, ...), or, with E = 0, a row of any
// length that is read again by every step and whose responsibilities are computed again.  What bounds it at 11008 x 4096:
// the first launch of a round (start, two likelihoods, update, gradient) the vector units, two exponentials an entry and
// some sums; the others memory (720 MB at 4.7 TB/s).  304, 162, 136 and 177 us a round; with a launch a step
// (13, responsibilities by tanh kept in LDS between two sums) 2310, and 85 for the result in fp32.
template <int T, int E>
__global__ __launch_bounds__(T) void rows_kernel(QRows g) {
    __shared__ double sh[T / 64];
    const int m = g.m, t = threadIdx.x;
    const size_t row = blockIdx.x;
    const double* y = g.Y + row * m;
    double x[E ? E : 1], k[E ? E : 1];                      // the centered row; what a step keeps of it
    double mean = 0.0;
    // f(x_j, its slot, j) for this thread's entries
    auto each = [&](auto f) {
        if constexpr (E > 0) {
#pragma unroll
            for (int u = 0; u < E; ++u)
                if (t + u * T < m) f(x[u], u, t + u * T);
        } else {
            int u = 0;
            for (int j = t; j < m; j += T, ++u) f(y[j] - mean, u, j);
        }
    };
    auto sum = [&](auto f) {
        double s = 0.0;
        each([&](double v, int u, int j) { s += f(v, u, j); });
        return block_sum<T>(s, sh);
    };
    if constexpr (E > 0) {
#pragma unroll
        for (int u = 0; u < E; ++u) x[u] = t + u * T < m ? y[t + u * T] : 0.0;
    }
    if (g.f32) each([&](double v, int, int j) { g.f32[row * m + j] = (float)v; });
    if (g.steps & QROWS_CENTER) {                           // the row mean taken out (Sec. 3.1, "Transformation Objectives")
        mean = sum([](double v, int, int) { return v; }) / m;
        if constexpr (E > 0) {
#pragma unroll
            for (int u = 0; u < E; ++u) x[u] -= mean;
        }
        if (g.ybar && t == 0) g.ybar[row] = mean;
        if (g.X) each([&](double v, int, int j) { g.X[row * m + j] = v; });
    }
    if (!(g.steps & ~QROWS_CENTER)) return;
    double c = 0.0, v = 1.0;
    if (g.steps & QROWS_INIT) {                             // Algorithm 2's empirical start: c = mean |x|, s^2 = mean (|x| - c)^2, floored
        c = sum([](double w, int, int) { return fabs(w); }) / m;
        v = fmax(sum([&](double w, int, int) { const double d = fabs(w) - c; return d * d; }) / m, g.s2_min);
    } else {
        c = g.c[row];
        v = g.s2[row];
    }
    double inv = 1.0 / v;
    auto resp = [&](double w, int u) {
        if constexpr (E > 0) return k[u];
        double e, rest;
        mix_exp(w, c, inv, e, rest);
        return mix_resp(e, rest, w, c);
    };
    // the responsibilities of the state (c, v) into k, and its likelihood: minus the row's sum of
    // log[ 1/2 phi(x; c, s^2) + 1/2 phi(x; -c, s^2) ] to part[row]
    auto state = [&](bool nll, double* part) {
        // sum of max(lp, lm) + log1p(exp(-|lp - lm|)) + log(1/2): the logarithms of up to sixteen factors 1 + e are taken
        // as one of their product.  What is carried is the product less one, q <- q + e + q e: a sum of terms that are
        // not negative, so that an e below the rounding of 1 + e counts as it does in log1p(e).
        double q = 0.0, s = 0.0, d2 = 0.0;
        int count = 0;
        const double ac = fabs(c);
        each([&](double w, int u, int) {
            double e, rest;
            mix_exp(w, c, inv, e, rest);
            if (E > 0) k[E > 0 ? u : 0] = mix_resp(e, rest, w, c);
            if (nll) {
                const double d = fabs(w) - ac;
                d2 = fma(d, d, d2);
                q = fma(q, e, q + e);
                ++count;
                if (E == 0 && (u & 15) == 15) {
                    s -= log1p(q);
                    q = 0.0;
                }
            }
        });
        if (nll) {
            s -= log1p(q);
            s += 0.5 * inv * d2 + count * (0.5 * log(2.0 * 3.14159265358979323846 * v) + log(2.0));
            const double tot = block_sum<T>(s, sh);
            if (t == 0) part[row] = tot;
        }
    };
    if ((E > 0 && (g.steps & (QROWS_EM | QROWS_GRAD | QROWS_TARGETS))) || (g.steps & QROWS_NLL))
        state(g.steps & QROWS_NLL, g.part);
    if (g.steps & QROWS_EM) {
        // one EM update (App. A.2.2): c from the responsibilities at the old parameters, then s^2 with the new c
        const double c1 = sum([&](double w, int u, int) { return resp(w, u) * w; }) / m;
        const double v1 = sum([&](double w, int u, int) {
            const double r = 0.5 * (1.0 + resp(w, u)), dp = w - c1, dm = w + c1;
            return r * dp * dp + (1.0 - r) * dm * dm;
        }) / m;
        c = c1;
        v = fmax(v1, g.s2_min);
        inv = 1.0 / v;
        if (g.steps & (QROWS_NLL_EM | QROWS_GRAD | QROWS_TARGETS))
            if (E > 0 || (g.steps & QROWS_NLL_EM)) state(g.steps & QROWS_NLL_EM, g.part_em);
    }
    if ((g.steps & (QROWS_INIT | QROWS_EM)) && t == 0) {
        g.c[row] = c;
        g.s2[row] = v;
    }
    if (g.steps & (QROWS_GRAD | QROWS_TARGETS)) {
        // gradient: H[(x - m) lambda] with m = (2 r - 1) c, lambda = 1 / s^2: minus the gradient of L_GMM in the centered
        // coordinates, times -n m (App. A.2.2 for d L / d x_ij = (x_ij - m_ij) / (n m s_i^2); App. A.2.3 for the adjoint's H).
        // targets, on the uncentered rows (App. A.2.2, "MM Surrogate"): H m + ybar 1 (the concave part of the centered
        // objective majorized by its tangent), times lambda, the weight of the row in the Procrustes matrices
        const bool grad = g.steps & QROWS_GRAD;
        auto value = [&](double w, int u) {
            const double r = c * resp(w, u);
            return grad ? (w - r) * inv : r;
        };
        const double bar = sum([&](double w, int u, int) {
            const double o = value(w, u);
            if (E > 0) k[E > 0 ? u : 0] = o;
            return o;
        }) / m;
        double* out = g.out + row * m;
        each([&](double w, int u, int j) {
            const double o = E > 0 ? k[E > 0 ? u : 0] : value(w, u);
            out[j] = grad ? o - bar : inv * (o - bar + mean);
        });
    }
}

// what a launch over rows leaves to one workgroup each: the scaled sums of its two likelihoods, and (block 2) the factor
// that turns (x - m) lambda into minus the gradient over mu, fac[0] = mu > 0 ? 1 / (n m mu) : min_i s2_i, with zeros behind it
__global__ __launch_bounds__(1024) void rows_finish_kernel(QRowsFinish f) {
    __shared__ double sh[16];
    const int t = threadIdx.x;
    if (blockIdx.x < 2) {
        const double* part = blockIdx.x == 0 ? f.part : f.part_em;
        if (!part) return;
        double s = 0.0;
        for (int i = t; i < f.n; i += 1024) s += part[i];
        const double tot = block_sum<1024>(s, sh) * f.scale;
        if (t == 0) {
            if (blockIdx.x == 0) f.nll[0] = tot;
            else {
                f.nll_em[0] = tot;
                if (f.nll_again) f.nll_again[0] = tot;
            }
        }
        return;
    }
    if (!f.fac) return;
    double v = 1.0e300;
    for (int i = t; i < f.n; i += 1024) v = fmin(v, f.s2[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
    if ((t & 63) == 0) sh[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
        for (int i = 1; i < 16; ++i) v = fmin(v, sh[i]);
        f.fac[0] = f.mu > 0.0 ? f.scale / f.mu : v;
        f.fac[1] = f.fac[2] = 0.0;
    }
}

__device__ __forceinline__ uint32_t hash32(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
    return x;
}
__global__ void fill_hash_kernel(double* Q, size_t count, uint32_t seed) {
    for (size_t e = (size_t)blockIdx.x * RT + threadIdx.x; e < count; e += (size_t)gridDim.x * RT) {
        const uint32_t h = hash32((uint32_t)e * 0x9e3779b9u + hash32(seed + (uint32_t)(e >> 32)));
        Q[e] = (double)h * (1.0 / 2147483648.0) - 1.0;
    }
}
__global__ void fill_identity_kernel(double* R, int n) {
    for (int e = blockIdx.x * RT + threadIdx.x; e < n * n; e += gridDim.x * RT) R[e] = (e / n == e % n) ? 1.0 : 0.0;
}
// X = C / ||C||_F, one workgroup (the start of the Newton-Schulz iteration for the polar factor:
// every singular value of X is at most 1); a zero matrix stays zero
__global__ __launch_bounds__(RT) void scale_inv_frob_kernel(const double* C, int count, double* X) {
    __shared__ double sh[4];
    double s = 0.0;
    for (int e = threadIdx.x; e < count; e += RT) s += C[e] * C[e];
    const double tot = block_sum(s, sh);
    const double inv = tot > 0.0 ? 1.0 / sqrt(tot) : 0.0;
    for (int e = threadIdx.x; e < count; e += RT) X[e] = C[e] * inv;
}
// out[0] = 1 / sqrt(largest absolute column sum of G): for G = X^T X that sum bounds sigma_max(X)^2
__global__ __launch_bounds__(RT) void gram_inv_norm_kernel(const double* G, int nn, double* out) {
    __shared__ double sh[RT];
    double worst = 0.0;
    for (int j = threadIdx.x; j < nn; j += RT) {
        double s = 0.0;
        for (int i = 0; i < nn; ++i) s += fabs(G[(size_t)i * nn + j]);
        worst = s > worst ? s : worst;
    }
    sh[threadIdx.x] = worst;
    __syncthreads();
    if (threadIdx.x == 0) {
        double w = 0.0;
        for (int i = 0; i < RT; ++i) w = sh[i] > w ? sh[i] : w;
        out[0] = w > 0.0 ? 1.0 / sqrt(w) : 0.0;
    }
}
__global__ void scale_by_kernel(double* X, size_t count, const double* s) {
    const double f = s[0];
    for (size_t e = (size_t)blockIdx.x * RT + threadIdx.x; e < count; e += (size_t)gridDim.x * RT) X[e] *= f;
}
// *done = 1 once max |G - I| <= tol (G nn x nn, one workgroup); never cleared here
__global__ __launch_bounds__(RT) void near_identity_kernel(const double* G, int nn, double tol, int* done) {
    __shared__ double sh[4];
    double worst = 0.0;
    for (int e = threadIdx.x; e < nn * nn; e += RT) {
        const double d = fabs(G[e] - (e / nn == e % nn ? 1.0 : 0.0));
        worst = d > worst || d != d ? d : worst;            // (a NaN stays)
    }
    // (the largest by way of the sum helper's layout: per wavefront, then over the four)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(worst, off, 64);
        worst = o > worst || o != o ? o : worst;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = worst;
    __syncthreads();
    if (threadIdx.x == 0) {
        double w = sh[0];
        for (int i = 1; i < 4; ++i) w = sh[i] > w || sh[i] != sh[i] ? sh[i] : w;
        if (w <= tol) *done = 1;
    }
}
__global__ void set_int_kernel(int* p, int v) { *p = v; }
__global__ void fill_value_kernel(double* p, size_t count, double v) {
    for (size_t e = (size_t)blockIdx.x * RT + threadIdx.x; e < count; e += (size_t)gridDim.x * RT) p[e] = v;
}
__global__ void pow_vec_kernel(const double* src, double pw, int count, double* dst) {
    for (int e = blockIdx.x * RT + threadIdx.x; e < count; e += gridDim.x * RT) dst[e] = src[e] > 0.0 ? pow(src[e], pw) : 0.0;
}

__global__ void scale_cols_f32_kernel(const double* src, const double* lam, double pw, int n, int k, float* dst) {
    for (size_t e = (size_t)blockIdx.x * RT + threadIdx.x; e < (size_t)n * k; e += (size_t)gridDim.x * RT) {
        const double l = lam[e % k];
        dst[e] = (float)(l > 0.0 ? src[e] * pow(l, pw) : 0.0);
    }
}

inline int flat_blocks(size_t count) {
    const size_t b = (count + RT - 1) / RT;
    return (int)(b < 4096 ? (b ? b : 1) : 4096);
}

}  // namespace

hipError_t bwla_q_launch_convert_f32_f64(const float* src, double* dst, size_t count, hipStream_t st) {
    hipLaunchKernelGGL(convert_f32_f64_kernel, dim3(flat_blocks(count)), dim3(RT), 0, st, src, dst, count);
    return hipGetLastError();
}
hipError_t bwla_q_launch_convert_f64_f32(const double* src, float* dst, size_t count, hipStream_t st) {
    hipLaunchKernelGGL(convert_f64_f32_kernel, dim3(flat_blocks(count)), dim3(RT), 0, st, src, dst, count);
    return hipGetLastError();
}
hipError_t bwla_q_launch_rows(const QRows& g, int n, hipStream_t st) {
    // the fewest threads whose registers hold the row
    const auto launch = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3(n), dim3(threads), 0, st, g);
        return hipGetLastError();
    };
    if (g.m <= 1024) return launch(rows_kernel<256, 4>, 256);
    if (g.m <= 4096) return launch(rows_kernel<256, 16>, 256);
    if (g.m <= 8192) return launch(rows_kernel<512, 16>, 512);
    if (g.m <= 16384) return launch(rows_kernel<1024, 16>, 1024);
    return launch(rows_kernel<256, 0>, 256);
}
hipError_t bwla_q_launch_rows_finish(const QRowsFinish& f, hipStream_t st) {
    hipLaunchKernelGGL(rows_finish_kernel, dim3(f.fac ? 3 : f.part_em ? 2 : 1), dim3(1024), 0, st, f);
    return hipGetLastError();
}
hipError_t bwla_q_launch_fill_hash(double* Q, size_t count, uint32_t seed, hipStream_t st) {
    hipLaunchKernelGGL(fill_hash_kernel, dim3(flat_blocks(count)), dim3(RT), 0, st, Q, count, seed);
    return hipGetLastError();
}
hipError_t bwla_q_launch_fill_identity(double* R, int n, hipStream_t st) {
    hipLaunchKernelGGL(fill_identity_kernel, dim3(flat_blocks((size_t)n * n)), dim3(RT), 0, st, R, n);
    return hipGetLastError();
}
hipError_t bwla_q_launch_scale_inv_frob(const double* C, int count, double* X, hipStream_t st) {
    hipLaunchKernelGGL(scale_inv_frob_kernel, dim3(1), dim3(RT), 0, st, C, count, X);
    return hipGetLastError();
}
hipError_t bwla_q_launch_gram_inv_norm(const double* G, int nn, double* out, hipStream_t st) {
    hipLaunchKernelGGL(gram_inv_norm_kernel, dim3(1), dim3(RT), 0, st, G, nn, out);
    return hipGetLastError();
}
hipError_t bwla_q_launch_scale_by(double* X, size_t count, const double* s, hipStream_t st) {
    hipLaunchKernelGGL(scale_by_kernel, dim3(flat_blocks(count)), dim3(RT), 0, st, X, count, s);
    return hipGetLastError();
}
hipError_t bwla_q_launch_near_identity(const double* G, int nn, double tol, int* done, hipStream_t st) {
    hipLaunchKernelGGL(near_identity_kernel, dim3(1), dim3(RT), 0, st, G, nn, tol, done);
    return hipGetLastError();
}
hipError_t bwla_q_launch_set_int(int* p, int v, hipStream_t st) {
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, st, p, v);
    return hipGetLastError();
}
hipError_t bwla_q_launch_fill_value(double* p, size_t count, double v, hipStream_t st) {
    hipLaunchKernelGGL(fill_value_kernel, dim3(flat_blocks(count)), dim3(RT), 0, st, p, count, v);
    return hipGetLastError();
}
hipError_t bwla_q_launch_pow_vec(const double* src, double pw, int count, double* dst, hipStream_t st) {
    hipLaunchKernelGGL(pow_vec_kernel, dim3(flat_blocks((size_t)count)), dim3(RT), 0, st, src, pw, count, dst);
    return hipGetLastError();
}
hipError_t bwla_q_launch_scale_cols_f32(const double* src, const double* lam, double pw, int n, int k, float* dst,
                                        hipStream_t st) {
    hipLaunchKernelGGL(scale_cols_f32_kernel, dim3(flat_blocks((size_t)n * k)), dim3(RT), 0, st, src, lam, pw, n, k, dst);
    return hipGetLastError();
}
