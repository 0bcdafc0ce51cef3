// Lowest eigenpair of a symmetric tridiagonal matrix on the device: multisection (kTriThreads
// points per round) for the eigenvalue, a twisted factorization for its vector.  Shared by the
// single and the batched Lanczos.
#pragma once

#include <hip/hip_runtime.h>

namespace qsd {

constexpr int kTriThreads = 256;

struct TridiagLds {
    double a[1024], b[1024];     // the matrix, then the pivots of the two factorizations
    double b2[1024];             // squared off-diagonals over the squared norm
    double dp[1024], dm[1024];
    double red[3][kTriThreads / 64];
    double lo, hi;
    int first[kTriThreads / 64];
    double best[2][kTriThreads / 64];
    int best_at[kTriThreads / 64];
    int twist;
};

// Whether T - x I has a leading principal minor that is not positive (then T has an eigenvalue at
// or below x), by the three-term recurrence of the minors p_i, scaled by a power of two every
// eight steps: one dependent multiply-add per step, where the recurrence of their ratios
// (Sturm counts) divides.  a and x are over the norm, so eight steps stay far inside the range.
__device__ __forceinline__ bool minor_not_positive(const double *a, const double *b2, int m, double x) {
    double p0 = 1.0, p1 = a[0] - x;
    bool neg = !(p1 > 0.0);
    for (int i0 = 1; i0 < m; i0 += 8) {
        auto step = [&](int i) {
            const double p2 = fma(a[i] - x, p1, -b2[i - 1] * p0);
            neg |= !(p2 > 0.0);
            p0 = p1;
            p1 = p2;
        };
        if (i0 + 8 <= m) {
#pragma unroll
            for (int k = 0; k < 8; ++k) step(i0 + k);
        } else {
            for (int i = i0; i < m; ++i) step(i);
        }
        if (neg) return true;  // (a wave ends with its last lane)
        const int s = max(__builtin_amdgcn_frexp_exp(p0), __builtin_amdgcn_frexp_exp(p1));
        p0 = __builtin_ldexp(p0, -s);
        p1 = __builtin_ldexp(p1, -s);
    }
    return neg;
}

// Lowest eigenpair of T_m (alpha[0..m), beta[0..m-1)), m <= 1024, computed by one block of
// kTriThreads threads.  tri[0] = theta, tri[1] = beta[m-1] * |s[m-1]|, tri[3 + i] = s[i].
//
// The vector comes from the two triangular factorizations of T - theta I, from the top and from the
// bottom, joined where their pivots leave the smallest remainder (Dhillon and Parlett's twisted
// factorization): its small last components, which the residual estimate needs, are products
// of pivot ratios and keep their relative accuracy.  The two chains of divisions run in two
// lanes; inverse iteration took five times as many in one.
__device__ void tridiag_lowest(const double *__restrict__ alpha, const double *__restrict__ beta, int m,
                               double *__restrict__ tri, TridiagLds &L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Gershgorin bounds and the norm
    double lo = INFINITY, hi = -INFINITY;
    for (int i = tid; i < m; i += kTriThreads) {
        const double ai = alpha[i], bi = beta[i], bl = i > 0 ? fabs(beta[i - 1]) : 0.0;
        const double r = bl + (i + 1 < m ? fabs(bi) : 0.0);
        L.a[i] = ai;
        L.b[i] = bi;
        lo = fmin(lo, ai - r);
        hi = fmax(hi, ai + r);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, d, 64));
        hi = fmax(hi, __shfl_xor(hi, d, 64));
    }
    if (lane == 0) {
        L.red[0][wave] = lo;
        L.red[1][wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kTriThreads / 64; ++w) {
        lo = fmin(lo, L.red[0][w]);
        hi = fmax(hi, L.red[1][w]);
    }
    const double norm = fmax(fmax(fabs(lo), fabs(hi)), 1e-300);
    const double pad = 2.2e-16 * norm * 4 + 1e-300;
    // scaled by a power of two (exact) so that all entries are at most 1 in modulus
    const int sc = __builtin_amdgcn_frexp_exp(norm);
    for (int i = tid; i < m; i += kTriThreads) {
        L.dp[i] = __builtin_ldexp(L.a[i], -sc);
        const double bs = __builtin_ldexp(L.b[i], -sc);
        L.b2[i] = bs * bs;
    }
    if (tid == 0) {
        L.lo = lo - pad;
        L.hi = hi + pad;
    }
    __syncthreads();
    // multisection: each round splits [lo, hi] into kTriThreads + 1 pieces
    for (int round = 0; round < 12; ++round) {
        lo = L.lo;
        hi = L.hi;
        if (!(hi - lo > 4.4e-16 * fmax(fabs(lo), fabs(hi)) + 1e-300)) break;
        const double step = (hi - lo) / (double)(kTriThreads + 1);
        const double x = lo + step * (double)(tid + 1);
        const unsigned long long w = __ballot(minor_not_positive(L.dp, L.b2, m, __builtin_ldexp(x, -sc)));
        if (lane == 0) L.first[wave] = w ? (int)__builtin_ctzll(w) + 64 * wave : kTriThreads;
        __syncthreads();
        if (tid == 0) {
            int f = kTriThreads;  // the first point with an eigenvalue at or below it
#pragma unroll
            for (int k = kTriThreads / 64 - 1; k >= 0; --k) f = L.first[k] < kTriThreads ? L.first[k] : f;
            L.lo = f > 0 ? lo + step * (double)f : lo;
            L.hi = f < kTriThreads ? lo + step * (double)(f + 1) : hi;
        }
        __syncthreads();
    }
    const double theta = 0.5 * (L.lo + L.hi);
    __syncthreads();  // dp is read as the scaled diagonal above
    // pivots from the top (dp) and from the bottom (dm); a vanishing one is replaced
    const double tiny = 1e-300 + 2.2e-16 * norm * 1e-3;
    if (tid == 0) {
        double d = L.a[0] - theta;
        for (int i = 0;; ++i) {
            if (fabs(d) < tiny) d = d < 0.0 ? -tiny : tiny;
            L.dp[i] = d;
            if (i + 1 >= m) break;
            d = (L.a[i + 1] - theta) - L.b[i] * (L.b[i] / d);
        }
    }
    if (tid == 64) {
        double d = L.a[m - 1] - theta;
        for (int i = m - 1;; --i) {
            if (fabs(d) < tiny) d = d < 0.0 ? -tiny : tiny;
            L.dm[i] = d;
            if (i == 0) break;
            d = (L.a[i - 1] - theta) - L.b[i - 1] * (L.b[i - 1] / d);
        }
    }
    __syncthreads();
    // the twist: smallest |gamma_i| = |dp_i + dm_i - (a_i - theta)|
    double best = INFINITY;
    int at = m;
    for (int i = tid; i < m; i += kTriThreads) {
        const double g = fabs(L.dp[i] + L.dm[i] - (L.a[i] - theta));
        if (g < best) {
            best = g;
            at = i;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const double o = __shfl_xor(best, d, 64);
        const int oi = __shfl_xor(at, d, 64);
        if (o < best || (o == best && oi < at)) {
            best = o;
            at = oi;
        }
    }
    if (lane == 0) {
        L.best[0][wave] = best;
        L.best_at[wave] = at;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kTriThreads / 64; ++w)
            if (L.best[0][w] < best || (L.best[0][w] == best && L.best_at[w] < at)) {
                best = L.best[0][w];
                at = L.best_at[w];
            }
        L.twist = at < m ? at : 0;
    }
    __syncthreads();
    // ratios of neighbouring components, then the products away from the twist (two chains)
    const int r = L.twist;
    for (int i = tid; i < m; i += kTriThreads) {
        if (i < r) L.dp[i] = -L.b[i] / L.dp[i];            // s_i / s_{i+1}
        if (i > r) L.dm[i] = -L.b[i - 1] / L.dm[i];        // s_i / s_{i-1}
    }
    __syncthreads();
    if (tid == 0) {
        double s = 1.0;
        L.a[r] = 1.0;
        for (int i = r - 1; i >= 0; --i) {
            s *= L.dp[i];
            L.a[i] = s;
        }
    }
    if (tid == 64) {
        double s = 1.0;
        for (int i = r + 1; i < m; ++i) {
            s *= L.dm[i];
            L.a[i] = s;
        }
    }
    __syncthreads();
    // (the largest component is at most a moderate multiple of the twist's: no overflow)
    double n2 = 0.0;
    for (int i = tid; i < m; i += kTriThreads) n2 += L.a[i] * L.a[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n2 += __shfl_xor(n2, d, 64);
    if (lane == 0) L.red[2][wave] = n2;
    __syncthreads();
    n2 = 0.0;
#pragma unroll
    for (int w = 0; w < kTriThreads / 64; ++w) n2 += L.red[2][w];
    const double inv = 1.0 / sqrt(n2);
    // the sign of the first component that inverse iteration from all ones gives is that of the
    // sum of the components
    double sum = 0.0;
    for (int i = tid; i < m; i += kTriThreads) sum += L.a[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) L.best[1][wave] = sum;
    __syncthreads();
    sum = 0.0;
#pragma unroll
    for (int w = 0; w < kTriThreads / 64; ++w) sum += L.best[1][w];
    const double f = sum < 0.0 ? -inv : inv;
    for (int i = tid; i < m; i += kTriThreads) tri[3 + i] = L.a[i] * f;
    if (tid == 0) {
        tri[0] = theta;
        tri[1] = fabs(beta[m - 1] * (L.a[m - 1] * f));
    }
}

}  // namespace qsd
