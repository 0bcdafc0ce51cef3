// Ground-state Lanczos on the device (FP64 basis and recurrence, full reorthogonalization).
//
// The paper hands its SpMV operator to external eigensolvers; this solver keeps the whole
// iteration on the GPU.  The iteration number comes with the launches; for graph replay it lives in
// device memory and every buffer has a fixed address, so that one iteration, a fixed kernel
// sequence, can be captured once and replayed:
//   w = H x                       (SpMV, FP64 or FP32 elements with FP64 accumulation)
//   h = V^T w; w -= V h  (twice)  (classical Gram-Schmidt applied twice against v_0..v_k)
//   alpha_k = sum of the two h_k; beta_k = ||w||; v_{k+1} = x = w / beta_k
// The tridiagonal eigenproblem is solved on the device every few iterations (multisection on the
// leading minors for the lowest eigenvalue, a twisted factorization for its vector); only theta and
// the Ritz residual estimate beta_k |s_k| are copied to the host.
#include <chrono>
#include <cmath>
#include <vector>

#include "common.h"
#include "hits.h"
#include "product.h"
#include "tridiag.h"

namespace qsd {
namespace {

constexpr int kRed = 256;       // threads of reduction kernels
constexpr int kListIters = 24;  // iterations from which a solve makes its own element list
constexpr int kPartRows = 256;  // rows per partial sum of the projections, at most kMaxParts of them
constexpr int kMaxParts = 512;  // (fixed by N alone => deterministic sums)
constexpr int kInlineParts = 16;   // partial sums per projection that the update kernel adds itself
constexpr int kFuseWaves = 8;      // waves of the fused update and projection
constexpr int kFuseMax = 32 * kFuseWaves;  // basis vectors it takes
constexpr int kNextRows = 4;       // rows per thread of the normalization
constexpr int kNormParts = 4096;   // partial squared norms that the normalization adds itself

struct LzState {
    int64_t N = 0;           // rows
    int64_t NR = 0;          // doubles per vector: N (real) or 2N (complex, interleaved)
    bool cplx = false;
    int m = 0;               // max iterations
    int parts = 0;           // partial sums per projection
    int64_t sqn = 0;         // partial squared norms (256-row tiles)
    uint8_t *mem = nullptr;  // every array below lies in it
    double *V = nullptr;     // [m+1][N]
    double *x = nullptr;     // [N] current basis vector (graph replay, which needs a fixed address)
    double *w = nullptr;     // [N]
    float *x32 = nullptr;    // [N]
    float *w32 = nullptr;    // [N]
    double *part = nullptr;  // [(m+1) * parts] (two planes for complex)
    double *part2 = nullptr; // [(m+1) * parts2], the second projection's
    int parts2 = 0;          // partial sums per second projection
    int fused = 0;           // vectors from which the first update and the second projection are one kernel
    double *sq = nullptr;    // [max(sqn, kMaxParts)]
    double *hv = nullptr;    // [m+1]
    double *alpha = nullptr; // [m]
    double *beta = nullptr;  // [m]
    int *kdev = nullptr;     // iteration number (graph replay)
    double *tri = nullptr;   // [m + 4]: theta, resid, breakdown flag, s[0..m)
    int64_t *spike = nullptr;
    void free_all() { dev_free(mem); }
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// Sum of v over the workgroup (kRed threads), by a fixed tree, in every thread.
__device__ __forceinline__ double block_sum(double v, double *ws) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < kRed / 64; ++q) t += ws[q];
    __syncthreads();
    return t;
}

// Sums of 16 values over a wave: on return the lane holds the sum of value (lane >> 2).  Each of
// the first four steps halves the values a lane carries (15 exchanges and additions, then 2),
// where 16 separate trees take 96 of each: 6.8 us of a 4096-row launch were mostly these.
template <int Q>
__device__ __forceinline__ double wave_sum_q(double (&a)[Q], int lane) {
    if constexpr (Q == 1) {
        a[0] += __shfl_xor(a[0], 2, 64);
        a[0] += __shfl_xor(a[0], 1, 64);
        return a[0];
    } else {
        const bool up = (lane & (2 * Q)) != 0;  // Q = 16 splits by lane bit 5, .., Q = 2 by bit 2
        double b[Q / 2];
#pragma unroll
        for (int q = 0; q < Q / 2; ++q) {
            const double keep = up ? a[q + Q / 2] : a[q], send = up ? a[q] : a[q + Q / 2];
            b[q] = keep + __shfl_xor(send, 2 * Q, 64);
        }
        return wave_sum_q(b, lane);
    }
}

// The iteration number: the launch's, or the device counter's under graph replay.
__device__ __forceinline__ int iter_of(const int *kdev, int k) { return kdev ? *kdev : k; }

// Whether an iteration over cnt vectors takes the fused update and projection, which starts at
// `fused` vectors: a captured graph holds both forms, and each looks at the device's counter.
__device__ __forceinline__ bool is_fused(int cnt, int fused) { return cnt >= fused && cnt <= kFuseMax; }
constexpr int kNever = 1 << 30;

// part[j][b] = sum over the rows of chunk b of V[j][i] * w[i], j = 0..k; complex (Hermitian)
// vectors: the real and imaginary parts of sum conj(V[j][i]) w[i] in two planes.
// blockIdx.x selects kGemvJ basis vectors: each thread reads w[i] once and kGemvJ basis values,
// so the basis streams at full occupancy; block sums by a fixed tree (deterministic).  Row
// chunks ascend with blockIdx.y; the update kernel walks the rows downwards, so each pass over the
// basis starts with what the pass before read last (a basis of up to 256 MB is served from the
// memory-side cache).
constexpr int kGemvJ = 16;

template <bool C>
__global__ __launch_bounds__(kRed) void k_gemv_t(const double *__restrict__ V, const double *__restrict__ w, int64_t N,
                                                 const int *__restrict__ kdev, int karg, int fused, int64_t plane,
                                                 double *__restrict__ part) {
    constexpr int P = C ? 2 : 1;
    __shared__ double red[P * kGemvJ][kRed / 64];
    const int cnt = iter_of(kdev, karg) + 1;
    const int j0 = blockIdx.x * kGemvJ;
    if (j0 >= cnt || is_fused(cnt, fused)) return;
    const int nj = min(kGemvJ, cnt - j0);
    const int64_t chunk = (N + gridDim.y - 1) / gridDim.y;
    const int64_t a = (int64_t)blockIdx.y * chunk;
    const int64_t b = min(N, a + chunk);
    double acc[P][kGemvJ];
#pragma unroll
    for (int q = 0; q < kGemvJ; ++q) acc[0][q] = acc[P - 1][q] = 0.0;
    for (int64_t i = a + threadIdx.x; i < b; i += kRed) {
        if constexpr (C) {
            const double2 *v0 = (const double2 *)V + (int64_t)j0 * N;
            const double2 wi = ((const double2 *)w)[i];
#pragma unroll
            for (int q = 0; q < kGemvJ; ++q)
                if (q < nj) {
                    const double2 v = v0[(int64_t)q * N + i];
                    acc[0][q] += v.x * wi.x + v.y * wi.y;
                    acc[1][q] += v.x * wi.y - v.y * wi.x;
                }
        } else {
            // (past the last vector the loads repeat it and the sums are dropped: no branch keeps
            // them apart)
            const double *v0 = V + (int64_t)j0 * N + i;
            const double wi = w[i];
#pragma unroll
            for (int q = 0; q < kGemvJ; ++q) acc[0][q] += v0[(int64_t)min(q, nj - 1) * N] * wi;
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert(kGemvJ == 16, "wave_sum_q leaves value lane >> 2 in a lane");
#pragma unroll
    for (int c = 0; c < P; ++c) {
        const double s = wave_sum_q(acc[c], lane);
        if ((lane & 3) == 0) red[P * (lane >> 2) + c][wave] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < P * nj) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kRed / 64; ++q) t += red[threadIdx.x][q];
        const int jj = threadIdx.x / P;
        part[(threadIdx.x % P) * plane + (int64_t)(j0 + jj) * gridDim.y + blockIdx.y] = t;
    }
}

// hv[j] = sum_b part[j][b] (one block per j and plane, fixed tree; planes interleaved in hv).
template <bool C>
__global__ __launch_bounds__(kRed) void k_reduce_parts(const double *__restrict__ part, int nparts,
                                                       const int *__restrict__ kdev, int karg, int64_t plane,
                                                       double *__restrict__ hv) {
    __shared__ double ws[kRed / 64];
    const int j = blockIdx.x, im = blockIdx.y;
    if (j > iter_of(kdev, karg)) return;
    double s = 0.0;
    const double *pp = part + im * plane + (int64_t)j * nparts;
    for (int p = threadIdx.x; p < nparts; p += kRed) s += pp[p];
    s = block_sum(s, ws);
    if (threadIdx.x == 0) hv[(C ? 2 : 1) * j + im] = s;
}

// w[i] -= sum_{j<=k} V[j][i] h[j], and alpha[k] += Re h[k] (one block).  h is hv, or with
// nparts > 0 the sum of the few partial sums, which saves the reduction's launch.  With `sq` each
// block also leaves its rows' squared norm there.  Rows descend with blockIdx.x.
template <bool C>
__global__ __launch_bounds__(kRed) void k_update(const double *__restrict__ V, const double *__restrict__ hv,
                                                 const double *__restrict__ part, int nparts, int64_t plane, int64_t N,
                                                 const int *__restrict__ kdev, int karg, int fused,
                                                 double *__restrict__ w, double *__restrict__ alpha,
                                                 double *__restrict__ sq) {
    constexpr int P = C ? 2 : 1;
    __shared__ double sh[P * 512];
    __shared__ double ws[kRed / 64];
    const int k = iter_of(kdev, karg), cnt = k + 1;
    if (is_fused(cnt, fused)) return;
    const int64_t i = (int64_t)(gridDim.x - 1 - blockIdx.x) * kRed + threadIdx.x;
    double ar = 0.0, ai = 0.0;
    for (int j0 = 0; j0 < cnt; j0 += 512) {
        const int nj = min(512, cnt - j0);
        __syncthreads();
        for (int q = threadIdx.x; q < P * nj; q += kRed) {
            double h;
            if (nparts > 0) {
                const double *pp = part + (q % P) * plane + (int64_t)(j0 + q / P) * nparts;
                h = 0.0;
#pragma unroll 8
                for (int p = 0; p < nparts; ++p) h += pp[p];
            } else {
                h = hv[P * j0 + q];
            }
            sh[q] = h;
            if (blockIdx.x == 0 && P * j0 + q == P * k) alpha[k] += h;
        }
        __syncthreads();
        if (i < N) {
            if constexpr (C) {
                for (int q = 0; q < nj; ++q) {
                    const double2 v = ((const double2 *)V)[(int64_t)(j0 + q) * N + i];
                    const double hr = sh[2 * q], hi = sh[2 * q + 1];
                    ar += v.x * hr - v.y * hi;
                    ai += v.x * hi + v.y * hr;
                }
            } else {
                const double *v0 = V + (int64_t)j0 * N + i;
#pragma unroll 8
                for (int q = 0; q < nj; ++q) ar += v0[(int64_t)q * N] * sh[q];
            }
        }
    }
    double n2 = 0.0;
    if (i < N) {
        if constexpr (C) {
            double2 t = ((double2 *)w)[i];
            t.x -= ar;
            t.y -= ai;
            ((double2 *)w)[i] = t;
            n2 = t.x * t.x + t.y * t.y;
        } else {
            const double t = w[i] - ar;
            w[i] = t;
            n2 = t * t;
        }
    }
    if (sq) {
        n2 = block_sum(n2, ws);
        if (threadIdx.x == 0) sq[blockIdx.x] = n2;
    }
}

// The first update and the second projection in one pass over the basis: w -= V h, then
// out[j][b] = sum over the rows of block b of V[j][i] w[i].  A wave holds the values of its lanes'
// rows for Q of the vectors (wave, wave + 8, ..) in registers between the two, and the next tile's
// are on their way meanwhile.  Past the last vector the loads repeat it: the weight is 0 and the sum
// is dropped.  Bound by the basis reads as the separate kernels are, of which it saves one in four:
// 700 000 rows, 50 vectors 45 us where the two take 96 (5.9 TB/s); 100 iterations 24.1 -> 19.9 ms.
template <int Q>
__global__ __launch_bounds__(64 * kFuseWaves) void k_update_project(const double *__restrict__ V,
                                                                    const double *__restrict__ hv,
                                                                    const double *__restrict__ part, int nparts,
                                                                    int64_t N, const int *__restrict__ kdev, int karg,
                                                                    int from, double *__restrict__ w,
                                                                    double *__restrict__ alpha,
                                                                    double *__restrict__ out) {
    constexpr int G = kFuseWaves;
    __shared__ double sh[G * Q];
    __shared__ double red[2][G][64];
    const int k = iter_of(kdev, karg), cnt = k + 1;
    if (cnt < from || cnt > G * Q) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int j = threadIdx.x; j < G * Q; j += 64 * G) {
        double h = 0.0;
        if (j < cnt) {
            if (nparts > 0) {
                const double *pp = part + (int64_t)j * nparts;
                for (int p = 0; p < nparts; ++p) h += pp[p];
            } else {
                h = hv[j];
            }
            if (blockIdx.x == 0 && j == k) alpha[k] += h;
        }
        sh[j] = h;
    }
    __syncthreads();
    double v[Q], acc[Q], wi = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = acc[q] = 0.0;
    auto load = [&](int64_t t, double(&b)[Q], double &wb) {
        const int64_t i = min(t * 64 + lane, N - 1);
#pragma unroll
        for (int q = 0; q < Q; ++q) b[q] = V[(int64_t)min(q * G + wave, k) * N + i];
        wb = wave == 0 ? w[i] : 0.0;
    };
    int64_t t = (N + 63) / 64 - 1 - blockIdx.x;
    if (t >= 0) load(t, v, wi);
    for (int buf = 0; t >= 0; t -= gridDim.x, buf ^= 1) {
        double nv[Q], nw;
        load(max(t - (int64_t)gridDim.x, (int64_t)0), nv, nw);
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) s += v[q] * sh[q * G + wave];
        red[buf][wave][lane] = wave == 0 ? wi - s : s;
        __syncthreads();
        double u = red[buf][0][lane];
#pragma unroll
        for (int g = 1; g < G; ++g) u -= red[buf][g][lane];
        const int64_t i = t * 64 + lane;
        if (i >= N) u = 0.0;
        if (wave == 0 && i < N) w[i] = u;
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] += v[q] * u;
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = nv[q];
        wi = nw;
    }
#pragma unroll
    for (int q0 = 0; q0 < Q; q0 += 16) {
        double a[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) a[q] = q0 + q < Q ? acc[q0 + q] : 0.0;
        const double d = wave_sum_q(a, lane);
        const int j = (q0 + (lane >> 2)) * G + wave;
        if ((lane & 3) == 0 && j < cnt) out[(int64_t)j * gridDim.x + blockIdx.x] = d;
    }
}

// y[i] = sum_{j<cnt} V[j][i] s[j]
__global__ __launch_bounds__(kRed) void k_gemv_n(const double *__restrict__ V, const double *__restrict__ s, int cnt,
                                                 int64_t N, double *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * kRed + threadIdx.x;
    if (i >= N) return;
    double acc = 0.0;
    for (int j = 0; j < cnt; ++j) acc += V[(int64_t)j * N + i] * s[j];
    y[i] = acc;
}

__global__ __launch_bounds__(kRed) void k_sq_part(const double *__restrict__ w, int64_t N, double *__restrict__ part) {
    __shared__ double ws[kRed / 64];
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kRed + threadIdx.x; i < N; i += (int64_t)gridDim.x * kRed) s += w[i] * w[i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < kRed / 64; ++q) t += ws[q];
        part[blockIdx.x] = t;
    }
}

// One value from n partial sums (more than the normalization adds itself).
__global__ __launch_bounds__(kRed) void k_sum(double *__restrict__ part, int64_t n) {
    __shared__ double ws[kRed / 64];
    double s = 0.0;
    for (int64_t p = threadIdx.x; p < n; p += kRed) s += part[p];
    s = block_sum(s, ws);
    if (threadIdx.x == 0) part[0] = s;
}

// beta[k] = sqrt(sum of the nsq partial squared norms), V[k+1] = w / beta[k] (also x when given).
// Breakdown (w vanished relative to the recurrence: an invariant subspace) records the
// number of valid iterations in tri[2] once; later iterations then carry zeros.
__global__ __launch_bounds__(kRed) void k_next(double *__restrict__ V, double *__restrict__ x,
                                               const double *__restrict__ w, int64_t N, const int *__restrict__ kdev,
                                               int karg, const double *__restrict__ sq, int nsq,
                                               const double *__restrict__ alpha, double *__restrict__ beta, int m,
                                               double *__restrict__ tri) {
    __shared__ double ws[kRed / 64];
    const int k = iter_of(kdev, karg);
    double s = 0.0;
    for (int p = threadIdx.x; p < nsq; p += kRed) s += sq[p];
    const double b = sqrt(block_sum(s, ws));  // the same sum in every block
    const double scale = fabs(alpha[k]) + (k > 0 ? beta[k - 1] : 0.0);
    const bool brk0 = !(b > 1e-12 * scale) || !(b > 1e-300);
    const bool brk = tri[2] != 0.0 || brk0;  // (block 0 may set it meanwhile: then brk0 holds here too)
    const double inv = brk ? 0.0 : 1.0 / b;
    const int64_t i0 = (int64_t)blockIdx.x * (kRed * kNextRows) + threadIdx.x;
#pragma unroll
    for (int q = 0; q < kNextRows; ++q) {
        const int64_t i = i0 + q * kRed;
        if (i < N) {
            const double v = w[i] * inv;
            if (x) x[i] = v;
            if (k + 1 <= m) V[(int64_t)(k + 1) * N + i] = v;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const bool first = brk && tri[2] == 0.0;
        if (first) tri[2] = (double)(k + 1);
        beta[k] = first ? 0.0 : b;
    }
}

__global__ void k_bump(int *kdev) { *kdev += 1; }

__global__ void k_f64_to_f32(const double *__restrict__ a, float *__restrict__ b, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        b[i] = (float)a[i];
}
__global__ void k_f32_to_f64(const float *__restrict__ a, double *__restrict__ b, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        b[i] = (double)a[i];
}

// Lowest eigenpair of T_m for one Lanczos run (one block).
__global__ __launch_bounds__(kTriThreads) void k_tridiag(const double *__restrict__ alpha,
                                                        const double *__restrict__ beta, int m,
                                                        double *__restrict__ tri) {
    __shared__ TridiagLds L;
    tridiag_lowest(alpha, beta, m, tri, L);
}

// argmin of d (lowest index among ties); one block
__global__ __launch_bounds__(kRed) void k_argmin(const double *__restrict__ d, int64_t N, int64_t *__restrict__ out) {
    __shared__ double bv[kRed];
    __shared__ int64_t bi[kRed];
    double v = INFINITY;
    int64_t idx = N;
    for (int64_t i = threadIdx.x; i < N; i += kRed)
        if (d[i] < v) {
            v = d[i];
            idx = i;
        }
    bv[threadIdx.x] = v;
    bi[threadIdx.x] = idx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int t = 1; t < kRed; ++t)
            if (bv[t] < v || (bv[t] == v && bi[t] < idx)) {
                v = bv[t];
                idx = bi[t];
            }
        *out = idx;
    }
}

__global__ void k_init_v0(double *__restrict__ x, int64_t N, int mode, uint64_t seed, const int64_t *__restrict__ spike,
                          int stride = 1) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        double v;
        if (mode == QSD_V0_UNIFORM) {
            v = 1.0;
        } else if (mode == QSD_V0_MIN_DIAG) {
            v = (i == stride * *spike) ? 1.0 : 0.0;
        } else {
            // splitmix64 of (seed, i): uniform in [-1, 1)
            uint64_t z = seed + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            z ^= z >> 31;
            v = (double)(z >> 11) * 0x1.0p-52 - 1.0;
        }
        x[i] = v;
    }
}

// x /= sqrt(sum part) (summed per block in fixed order; kRed threads); also stored in `copy`
__global__ __launch_bounds__(kRed) void k_scale(double *__restrict__ x, int64_t N, const double *__restrict__ part,
                                                int nparts, double *__restrict__ copy) {
    __shared__ double ws[kRed / 64];
    double s = 0.0;
    for (int p = threadIdx.x; p < nparts; p += kRed) s += part[p];
    const double inv = 1.0 / sqrt(block_sum(s, ws));
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
    {
        const double v = x[i] * inv;
        x[i] = v;
        if (copy) copy[i] = v;
    }
}

// r = Hy - theta y -> partial sums of r^2 and of y^2
__global__ __launch_bounds__(kRed) void k_resid_part(const double *__restrict__ hy, const double *__restrict__ y,
                                                     double theta, int64_t N, double *__restrict__ part) {
    __shared__ double ws[kRed / 64];
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kRed + threadIdx.x; i < N; i += (int64_t)gridDim.x * kRed) {
        const double r = hy[i] - theta * y[i];
        s += r * r;
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < kRed / 64; ++q) t += ws[q];
        part[blockIdx.x] = t;
    }
}

inline unsigned gridN(int64_t n) { return (unsigned)((n + kRed - 1) / kRed); }

// The current basis vector: under graph replay at the fixed address, else in the basis.
const double *current(const LzState &S, int k) { return k < 0 ? S.x : S.V + (int64_t)k * S.NR; }

template <bool C>
void enqueue_blas(LzState &S, int k, hipStream_t st) {
    const int64_t N = S.N;
    const int *kdev = k < 0 ? S.kdev : nullptr;
    const int cnt = k < 0 ? S.m + 1 : k + 1;  // basis vectors the launch has to cover
    const dim3 gt((cnt + kGemvJ - 1) / kGemvJ, S.parts);
    const int64_t plane = (int64_t)(S.m + 1) * S.parts, plane2 = (int64_t)(S.m + 1) * S.parts2;
    const bool own = S.parts <= kInlineParts;  // (and parts2)
    const int P = C ? 2 : 1;
    auto reduce = [&](const double *part, int parts, int64_t pl) {
        if (!own) k_reduce_parts<C><<<dim3(cnt, P), kRed, 0, st>>>(part, parts, kdev, k, pl, S.hv);
    };
    k_gemv_t<C><<<gt, kRed, 0, st>>>(S.V, S.w, N, kdev, k, kNever, plane, S.part);
    reduce(S.part, S.parts, plane);
    // w -= V h and the second projection: in one kernel or in two
    const int from = C ? kNever : S.fused;
    if (cnt >= from && (kdev || cnt <= kFuseMax)) {
        auto fused = [&](auto q) {
            k_update_project<decltype(q)::value><<<S.parts2, 64 * kFuseWaves, 0, st>>>(
                S.V, S.hv, S.part, own ? S.parts : 0, N, kdev, k, from, S.w, S.alpha, S.part2);
        };
        const int Q = (std::min(cnt, kFuseMax) + kFuseWaves - 1) / kFuseWaves;
        using std::integral_constant;
        if (Q <= 4) fused(integral_constant<int, 4>{});
        else if (Q <= 6) fused(integral_constant<int, 6>{});
        else if (Q <= 8) fused(integral_constant<int, 8>{});
        else if (Q <= 10) fused(integral_constant<int, 10>{});
        else if (Q <= 12) fused(integral_constant<int, 12>{});
        else if (Q <= 14) fused(integral_constant<int, 14>{});
        else if (Q <= 16) fused(integral_constant<int, 16>{});
        else if (Q <= 20) fused(integral_constant<int, 20>{});
        else if (Q <= 24) fused(integral_constant<int, 24>{});
        else if (Q <= 28) fused(integral_constant<int, 28>{});
        else fused(integral_constant<int, 32>{});
    }
    if (kdev || cnt < from || cnt > kFuseMax) {
        k_update<C><<<(unsigned)S.sqn, kRed, 0, st>>>(S.V, S.hv, S.part, own ? S.parts : 0, plane, N, kdev, k, from, S.w,
                                                      S.alpha, nullptr);
        k_gemv_t<C><<<dim3(gt.x, S.parts2), kRed, 0, st>>>(S.V, S.w, N, kdev, k, from, plane2, S.part2);
    }
    reduce(S.part2, S.parts2, plane2);
    k_update<C><<<(unsigned)S.sqn, kRed, 0, st>>>(S.V, S.hv, S.part2, own ? S.parts2 : 0, plane2, N, kdev, k, kNever, S.w,
                                                  S.alpha, S.sq);
    int nsq = (int)S.sqn;
    if (S.sqn > kNormParts) {
        k_sum<<<1, kRed, 0, st>>>(S.sq, S.sqn);
        nsq = 1;
    }
    k_next<<<(unsigned)((S.NR + kRed * kNextRows - 1) / (kRed * kNextRows)), kRed, 0, st>>>(S.V, k < 0 ? S.x : nullptr, S.w, S.NR, kdev, k, S.sq, nsq, S.alpha, S.beta,
                                         S.m, S.tri);
    if (k < 0) k_bump<<<1, 1, 0, st>>>(S.kdev);
}

// Iteration k, or with k < 0 the iteration that the device counter says (graph capture).
int enqueue_iteration(const SpmvOp &op, LzState &S, bool f32, int k, hipStream_t st) {
    const double *x = current(S, k);
    if (f32) {
        k_f64_to_f32<<<1024, kRed, 0, st>>>(x, S.x32, S.NR);
        QSD_TRY(op.matvec(1, S.x32, 1, S.w32, 1, S.cplx ? QSD_C64 : QSD_F32, st));
        k_f32_to_f64<<<1024, kRed, 0, st>>>(S.w32, S.w, S.NR);
    } else {
        QSD_TRY(op.matvec(1, x, 1, S.w, 1, S.cplx ? QSD_C128 : QSD_F64, st));
    }
    if (S.cplx)
        enqueue_blas<true>(S, k, st);
    else
        enqueue_blas<false>(S, k, st);
    QSD_CHECK_HIP(hipGetLastError());
    return QSD_OK;
}

// alpha, beta, the head of tri and the iteration counter at the start of a run
__global__ void k_clear(double *__restrict__ alpha, double *__restrict__ beta, int m, double *__restrict__ tri,
                        int *__restrict__ kdev) {
    for (int i = threadIdx.x; i < m; i += blockDim.x) alpha[i] = beta[i] = 0.0;
    if (threadIdx.x < 4) tri[threadIdx.x] = 0.0;
    if (threadIdx.x == 0) *kdev = 0;
}

}  // namespace
}  // namespace qsd

using namespace qsd;

extern "C" void qsd_lanczos_default_opts(qsd_lanczos_opts *o) {
    if (!o) return;
    o->max_iter = 300;
    o->tol = 1e-10;
    o->v0_mode = QSD_V0_UNIFORM;
    o->seed = 0;
    o->spmv_dtype = QSD_F64;
    o->check_every = 5;
    o->want_vector = 0;
    o->use_graph = 0;
    o->alloc = nullptr;
}

namespace {

int lanczos_impl(SpmvOp op, const qsd_lanczos_opts *opts, double *eval_out, void *d_evec,
                 qsd_lanczos_info *info, void *stream) {
    auto t_start = std::chrono::steady_clock::now();
    if (!eval_out) return fail(QSD_ERR_INVALID_ARG, "NULL argument");
    qsd_lanczos_opts o;
    qsd_lanczos_default_opts(&o);
    if (opts) o = *opts;
    const bool cplx = op.is_complex();
    if (o.max_iter < 1 || o.max_iter > 1000) return fail(QSD_ERR_INVALID_ARG, "max_iter must be in [1, 1000]");
    if (!(o.tol > 0)) return fail(QSD_ERR_INVALID_ARG, "tol must be > 0");
    if (o.spmv_dtype != QSD_F64 && o.spmv_dtype != QSD_F32) return fail(QSD_ERR_DTYPE, "spmv_dtype must be F64 or F32");
    const int32_t mv64 = cplx ? QSD_C128 : QSD_F64, mv32 = cplx ? QSD_C64 : QSD_F32;
    if (!op.takes(o.spmv_dtype == QSD_F32 ? mv32 : mv64))
        return fail(QSD_ERR_DTYPE, "spmv_dtype must be the stored matrix's dtype");
    if (o.v0_mode < QSD_V0_UNIFORM || o.v0_mode > QSD_V0_USER) return fail(QSD_ERR_INVALID_ARG, "bad v0_mode");
    if ((o.v0_mode == QSD_V0_USER || o.want_vector) && !d_evec)
        return fail(QSD_ERR_INVALID_ARG, "d_evec is required for QSD_V0_USER / want_vector");
    if (o.check_every < 1) o.check_every = 1;
    hipStream_t st = (hipStream_t)stream;
    // basis and work vectors from the caller's allocator or the operator's (the scope outlives S)
    AllocScope scope(o.alloc ? o.alloc : op.allocator(), stream);
    const int64_t N = op.N();
    const int64_t NR = cplx ? 2 * N : N;  // doubles per vector
    LzState S;
    S.N = N;
    S.NR = NR;
    S.cplx = cplx;
    S.m = (int)std::min<int64_t>(o.max_iter, N);
    const bool f32 = o.spmv_dtype == QSD_F32;
    int rc = QSD_OK;
    S.parts = (int)std::min<int64_t>(kMaxParts, std::max<int64_t>(1, (N + kPartRows - 1) / kPartRows));
    S.parts2 = S.parts <= kInlineParts ? S.parts : (int)std::min<int64_t>(kMaxParts, (N + 63) / 64);
    // Where the fused kernel gains: 700 000 rows 16 vectors 23 us against 23 for the two, 32 vectors 26
    // against 38; shorter passes are latencies, of which it has more (4096 rows, 35 iterations 1296 us
    // against 1225; 30 000 rows, 30 iterations 1476 against 1436; 100 000 rows, 50 iterations 2969
    // against 3192).
    S.fused = (int)std::min<int64_t>(kNever, std::max<int64_t>(17, (2000000 + N - 1) / N));
    S.sqn = (N + kRed - 1) / kRed;
    {
        // one allocation, carved (256-byte aligned)
        size_t off = 0;
        auto take = [&](size_t bytes) {
            const size_t at = off;
            off += (bytes + 255) / 256 * 256;
            return at;
        };
        const int P = cplx ? 2 : 1;
        const size_t oV = take((size_t)(S.m + 1) * NR * 8), ox = take(NR * 8), ow = take(NR * 8);
        const size_t ox32 = take(f32 ? NR * 4 : 0), ow32 = take(f32 ? NR * 4 : 0);
        const size_t op_ = take((size_t)(S.m + 1) * S.parts * P * 8);
        const size_t op2 = take((size_t)(S.m + 1) * S.parts2 * P * 8);
        const size_t os = take(std::max<size_t>(S.sqn, kMaxParts) * 8), oh = take((size_t)(S.m + 1) * P * 8);
        const size_t oa = take((size_t)S.m * 8), ob = take((size_t)S.m * 8), ok = take(8), ot = take((size_t)(S.m + 4) * 8);
        const size_t osp = take(8);
        rc = dev_alloc(&S.mem, off);
        S.V = (double *)(S.mem + oV);
        S.x = (double *)(S.mem + ox);
        S.w = (double *)(S.mem + ow);
        S.x32 = (float *)(S.mem + ox32);
        S.w32 = (float *)(S.mem + ow32);
        S.part = (double *)(S.mem + op_);
        S.part2 = (double *)(S.mem + op2);
        S.sq = (double *)(S.mem + os);
        S.hv = (double *)(S.mem + oh);
        S.alpha = (double *)(S.mem + oa);
        S.beta = (double *)(S.mem + ob);
        S.kdev = (int *)(S.mem + ok);
        S.tri = (double *)(S.mem + ot);
        S.spike = (int64_t *)(S.mem + osp);
    }
    // a sparse operator is applied from the list of its elements: the operator's own, or one made
    // for this solve (its cost is that of about three SpMVs)
    qsd_hits *made = nullptr;
    if (rc == QSD_OK && op.h && !prod_usable(op.h) && !(op.h->schedule & QSD_SCHED_HASH_LOOKUP)) {
        if (!op.h->hits && S.m >= kListIters) rc = hits_build(op.h, &made, st);
        op.hits = op.h->hits ? op.h->hits : made;
    }
    if (rc != QSD_OK) {
        S.free_all();
        return rc;
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipGraphExec_t gexec = nullptr;
    hipGraph_t graph = nullptr;
    double theta = 0.0, ritz = INFINITY, expl = NAN;
    int iters = 0;
    bool converged = false;
    float mv_ms = 0.0f;
    do {
        // start vector
        if (o.v0_mode == QSD_V0_USER) {
            if (hipMemcpyAsync(S.x, d_evec, NR * 8, hipMemcpyDeviceToDevice, st) != hipSuccess) {
                rc = fail(QSD_ERR_HIP, "copy failed");
                break;
            }
        } else {
            if (o.v0_mode == QSD_V0_MIN_DIAG) k_argmin<<<1, kRed, 0, st>>>(op.diag(), N, S.spike);
            k_init_v0<<<1024, kRed, 0, st>>>(S.x, NR, o.v0_mode, o.seed, S.spike, cplx ? 2 : 1);
        }
        k_sq_part<<<kMaxParts, kRed, 0, st>>>(S.x, NR, S.sq);
        k_scale<<<1024, kRed, 0, st>>>(S.x, NR, S.sq, kMaxParts, S.V);
        k_clear<<<1, 256, 0, st>>>(S.alpha, S.beta, S.m, S.tri, S.kdev);
        if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
            rc = fail(QSD_ERR_HIP, "event create failed");
            break;
        }
        if (o.use_graph) {
            if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess) {
                rc = fail(QSD_ERR_HIP, "stream capture failed");
                break;
            }
            int erc = enqueue_iteration(op, S, f32, -1, st);
            hipError_t ce = hipStreamEndCapture(st, &graph);
            if (erc != QSD_OK || ce != hipSuccess) {
                rc = erc != QSD_OK ? erc : fail(QSD_ERR_HIP, "end capture failed");
                break;
            }
            if (hipGraphInstantiate(&gexec, graph, nullptr, nullptr, 0) != hipSuccess) {
                rc = fail(QSD_ERR_HIP, "graph instantiate failed");
                break;
            }
        }
        std::vector<double> tri(3);
        int done = 0;
        while (done < S.m) {
            const int nstep = std::min(o.check_every, S.m - done);
            for (int s = 0; s < nstep && rc == QSD_OK; ++s) {
                if (gexec) {
                    if (hipGraphLaunch(gexec, st) != hipSuccess) rc = fail(QSD_ERR_HIP, "graph launch failed");
                } else {
                    rc = enqueue_iteration(op, S, f32, done + s, st);
                }
            }
            if (rc != QSD_OK) break;
            done += nstep;
            k_tridiag<<<1, kRed, 0, st>>>(S.alpha, S.beta, done, S.tri);
            if (hipMemcpyAsync(tri.data(), S.tri, 3 * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess) {
                rc = fail(QSD_ERR_HIP, "Lanczos iteration failed: %s", hipGetErrorString(hipGetLastError()));
                break;
            }
            iters = done;
            if (tri[2] != 0.0) {
                // invariant subspace after tri[2] iterations: T of that size is exact
                iters = (int)tri[2];
                k_tridiag<<<1, kRed, 0, st>>>(S.alpha, S.beta, iters, S.tri);
                if (hipMemcpyAsync(tri.data(), S.tri, 2 * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
                    hipStreamSynchronize(st) != hipSuccess) {
                    rc = fail(QSD_ERR_HIP, "tridiagonal solve failed");
                    break;
                }
                theta = tri[0];
                ritz = 0.0;
                converged = true;
                break;
            }
            theta = tri[0];
            ritz = tri[1];
            if (ritz <= o.tol * std::fabs(theta)) {
                converged = true;
                break;
            }
        }
        if (rc != QSD_OK) break;
        // matvec timing: one extra timed SpMV (the Lanczos loop itself is not instrumented)
        hipEventRecord(e0, st);
        if (f32)
            rc = op.matvec(1, S.x32, 1, S.w32, 1, mv32, st);
        else
            rc = op.matvec(1, gexec ? S.x : S.V, 1, S.w, 1, mv64, st);
        hipEventRecord(e1, st);
        if (rc != QSD_OK) break;
        hipEventSynchronize(e1);
        hipEventElapsedTime(&mv_ms, e0, e1);
        if (o.want_vector) {
            double *y = (double *)d_evec;
            k_gemv_n<<<gridN(NR), kRed, 0, st>>>(S.V, S.tri + 3, iters, NR, y);
            k_sq_part<<<kMaxParts, kRed, 0, st>>>(y, NR, S.sq);
            k_scale<<<1024, kRed, 0, st>>>(y, NR, S.sq, kMaxParts, nullptr);
            if (op.takes(mv64)) {
                if ((rc = op.matvec(1, y, 1, S.w, 1, mv64, st)) != QSD_OK) break;
            } else {  // a stored FP32 matrix: the residual of the FP32 operator
                k_f64_to_f32<<<1024, kRed, 0, st>>>(y, S.x32, NR);
                if ((rc = op.matvec(1, S.x32, 1, S.w32, 1, mv32, st)) != QSD_OK) break;
                k_f32_to_f64<<<1024, kRed, 0, st>>>(S.w32, S.w, NR);
            }
            k_resid_part<<<kMaxParts, kRed, 0, st>>>(S.w, y, theta, NR, S.sq);
            std::vector<double> parts(kMaxParts);
            if (hipMemcpyAsync(parts.data(), S.sq, kMaxParts * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess) {
                rc = fail(QSD_ERR_HIP, "residual failed");
                break;
            }
            double t = 0.0;
            for (double p : parts) t += p;
            expl = std::sqrt(t) / std::max(1e-300, std::fabs(theta));
        }
    } while (0);
    if (gexec) hipGraphExecDestroy(gexec);
    if (graph) hipGraphDestroy(graph);
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
    hits_free(made);
    S.free_all();
    if (rc != QSD_OK) return rc;
    *eval_out = theta;
    if (info) {
        info->iterations = iters;
        info->converged = converged ? 1 : 0;
        info->ritz_residual = ritz;
        info->explicit_residual = expl;
        info->matvec_ms = mv_ms;
        info->total_ms =
            std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    }
    if (!converged) return fail(QSD_ERR_NOT_CONVERGED, "Lanczos did not converge in %d iterations", iters);
    return QSD_OK;
}

}  // namespace

extern "C" int qsd_lanczos(const qsd_ham *h, const qsd_lanczos_opts *opts, double *eval_out, void *d_evec,
                           qsd_lanczos_info *info, void *stream) {
    clear_error();
    if (!h) return fail(QSD_ERR_INVALID_ARG, "NULL argument");
    SpmvOp op;
    op.h = h;
    return lanczos_impl(op, opts, eval_out, d_evec, info, stream);
}

extern "C" int qsd_csr_lanczos(const qsd_csr *c, const qsd_lanczos_opts *opts, double *eval_out, void *d_evec,
                               qsd_lanczos_info *info, void *stream) {
    clear_error();
    if (!c) return fail(QSD_ERR_INVALID_ARG, "NULL argument");
    SpmvOp op;
    op.c = c;
    return lanczos_impl(op, opts, eval_out, d_evec, info, stream);
}
