// Element lists of sparse operators and the SpMV that runs from them (see hits.h).
#include "hits.h"

#include <algorithm>
#include <type_traits>

#include "matvec.h"

namespace qsd {
namespace {

// Whether a list pays is asked of a sample first where the count of all rows, which takes as long as an
// SpMV by the row engine, is dear: many rows, or many groups, which a lane walks one after the other
// however few rows there are (10 000 rows of a molecular product, 18 280 groups: 2.2 ms, 1.5% of a solve
// of 30 iterations, which lost that much; the sample takes 67 us).
constexpr int kSampleRows = 256, kSampleThreads = 512;
constexpr int64_t kSampleTiles = 512, kSampleGroups = 1024;
// What one row counts at most (a sample around a reference string has a few rows with hundreds), and the
// elements per row beyond which the rest is not counted: one is the limit, and some room for chance.
constexpr uint32_t kSampleMost = 8;
constexpr double kSampleMean = 1.5;
// Elements from which a row gets a wave of its own.  A lane walks its elements in a chain of
// dependent reads, about a microsecond each: 156 rows of 18 to 39 elements (700 000 heavy-hex
// strings) kept the launch going for 34 us, and 150 rows of 48 to 117 (3M strings, 8 vectors) for
// 180; sharing such a row among the lanes of whichever wave held it took 41 and 121.
constexpr uint32_t kLongRow = 8;

inline unsigned tiles_of(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Off-diagonal elements of kSampleRows rows spread over the subspace: a workgroup per row, a thread per
// group (a term with the row's ladder and projector bits in a group whose column is present).
template <int Wp>
__global__ __launch_bounds__(kSampleThreads) void k_hit_sample(SubView s, HamView h,
                                                               unsigned long long *__restrict__ total) {
    __shared__ uint32_t sum;
    if (threadIdx.x == 0) sum = 0u;
    __syncthreads();
    const int64_t r = (int64_t)blockIdx.x * s.N / kSampleRows;
    uint64_t key[Wp];
#pragma unroll
    for (int w = 0; w < Wp; ++w) key[w] = s.keys[(int64_t)w * s.N + r];
    const uint64_t hrow = s.hkey[r];
    uint32_t n = 0;
    for (int64_t g = threadIdx.x; g < h.G; g += kSampleThreads) {
        uint64_t col[Wp];
#pragma unroll
        for (int w = 0; w < Wp; ++w) col[w] = key[w] ^ h.g_mask[g * Wp + w];
        if (probe<Wp>(s, hrow ^ h.g_hash[g], col) < 0) continue;
        const uint32_t t0 = h.g_term0[g], t1 = t0 + h.g_nterm[g];
        bool any = false;
        for (uint32_t t = t0; t < t1 && !any; ++t) any = term_pass<Wp>(key, h.t_cws + (int64_t)t * 3 * Wp);
        n += any;
    }
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
    if ((threadIdx.x & 63) == 0 && n) atomicAdd(&sum, n);
    __syncthreads();
    if (threadIdx.x == 0 && sum) atomicAdd(total, (unsigned long long)min(sum, kSampleMost));
}

// Off-diagonal elements of all rows: their number per row (1 << 32 | count for a row that has some),
// the row bits, the total, and the rows with many.
template <int Wp>
__global__ __launch_bounds__(kBlock) void k_hit_count(SubView s, HamView h, int64_t *__restrict__ cnt,
                                                      uint64_t *__restrict__ bits,
                                                      unsigned long long *__restrict__ total) {
    __shared__ ChunkLds<Wp> lds;
    uint64_t key[Wp], hrow;
    uint32_t prow;
    bool valid;
    const int64_t row0 = (int64_t)blockIdx.x * kBlock;
    const int64_t r = load_row<Wp>(s, row0, key, hrow, prow, valid);
    uint32_t n = 0;
    row_engine<Wp>(s, h, key, hrow, prow, valid, lds, sink<double>([&](int64_t, double, double, int) { ++n; }), nullptr,
                   false, true);
    if (!valid) n = 0;
    if (valid) cnt[r] = n ? (int64_t)((1ull << 32) | n) : 0;
    const uint64_t w = __ballot(n != 0u);
    const int64_t word = (row0 >> 6) + (threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0 && word * 64 < s.N) bits[word] = w;
    unsigned long long t = n;
    for (int d = 32; d >= 1; d >>= 1) t += __shfl_xor(t, d, 64);
    const uint64_t lng = __ballot(n > kLongRow);
    if ((threadIdx.x & 63) == 0 && t) atomicAdd(total, t);
    if ((threadIdx.x & 63) == 0 && lng) atomicAdd(total + 1, (unsigned long long)__popcll(lng));
}

// rows[i], ptr[i] of the rows with elements, from the scanned counts (rows << 32 | elements).
__global__ __launch_bounds__(kBlock) void k_hit_rows(const int64_t *__restrict__ scan, int64_t N,
                                                     uint32_t *__restrict__ rows, uint32_t *__restrict__ ptr,
                                                     uint32_t *__restrict__ lng, unsigned long long *__restrict__ nlng) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r > N) return;
    const uint64_t a = (uint64_t)scan[r];
    if (r == N) {
        ptr[a >> 32] = (uint32_t)a;
    } else if ((uint64_t)scan[r + 1] != a) {
        rows[a >> 32] = (uint32_t)r;
        ptr[a >> 32] = (uint32_t)a;
        if ((uint32_t)scan[r + 1] - (uint32_t)a > kLongRow) lng[atomicAdd(nlng, 1ull)] = (uint32_t)(a >> 32);
    }
}

template <int Wp>
__global__ __launch_bounds__(kBlock) void k_hit_fill(SubView s, HamView h, const uint32_t *__restrict__ rows, int64_t M,
                                                     const uint32_t *__restrict__ ptr, qsd_hit *__restrict__ rec) {
    __shared__ ChunkLds<Wp> lds;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool valid = i < M;
    const int64_t r = rows[valid ? i : M - 1];
    uint64_t key[Wp];
#pragma unroll
    for (int w = 0; w < Wp; ++w) key[w] = s.keys[(int64_t)w * s.N + r];
    const uint64_t hrow = s.hkey[r];
    const uint32_t prow = s.pfilt ? s.pkey[r] : 0u;
    uint32_t o = valid ? ptr[i] : 0u;
    row_engine<Wp>(s, h, key, hrow, prow, valid, lds, range_sink<double>([&](int64_t j, uint32_t t0, uint32_t len) {
        rec[o++] = qsd_hit{(uint32_t)j, t0, len, 0u};
    }), nullptr, false, true);
}

// The first `nl` workgroups take the listed rows (chains of dependent reads, so they start first,
// the longest rows before the rest), the others write y = d x, element by element in storage order
// (coalesced whatever the number of vectors), for the rows without elements.  The listed rows' sums
// are formed as in every other path (d x first, then the elements in group order), so the results are
// bitwise the same.  Bound by the stream of x, d and y: the list is a few per cent of the rows on the
// workloads this serves.  3M rows of 200 qubits, 8 vectors: 119 us, 106 at the rate of a copy; with
// the row engine 1651.
constexpr int kDiagItems = 4;

template <int Wp, int NV, class ET, bool CPLX>
__global__ __launch_bounds__(kBlock) void k_hits_matvec(SubView s, HamView h, qsd_hits p, const ET *__restrict__ dre,
                                                        const ET *__restrict__ dim, const ET *__restrict__ x,
                                                        int64_t ldx, ET *__restrict__ y, int64_t ldy, int nvec,
                                                        unsigned nl) {
    const unsigned block = blockIdx.y * gridDim.x + blockIdx.x;
    if (block >= nl) {
        const int64_t n = s.N * nvec, e0 = (int64_t)(block - nl) * (kBlock * kDiagItems) + threadIdx.x;
#pragma unroll
        for (int k = 0; k < kDiagItems; ++k) {
            const int64_t e = e0 + k * kBlock;
            if (e >= n) continue;
            const int64_t r = nvec == NV ? e / NV : e / nvec;
            const int64_t v = e - r * nvec;
            if ((p.rowbits[r >> 6] >> (r & 63)) & 1ull) continue;
            double re, im;
            if (CPLX) {
                diag_term<true>((double)dre[r], (double)dim[r], (double)x[2 * (r * ldx + v)],
                                (double)x[2 * (r * ldx + v) + 1], re, im);
                y[2 * (r * ldy + v)] = (ET)re;
                y[2 * (r * ldy + v) + 1] = (ET)im;
            } else {
                diag_term<false>((double)dre[r], 0.0, (double)x[r * ldx + v], 0.0, re, im);
                y[r * ldy + v] = (ET)re;
            }
        }
        return;
    }
    const int lane = threadIdx.x & 63;
    auto load_x = [&](int64_t j, int64_t u, double &xr, double &xi) {
        if (CPLX) {
            xr = (double)x[2 * (j * ldx + u)];
            xi = (double)x[2 * (j * ldx + u) + 1];
        } else {
            xr = (double)x[j * ldx + u];
            xi = 0.0;
        }
    };
    // a row with many elements has a wave of its own, another NV lanes, a vector each (x and y are
    // read and written in whole lines)
    const unsigned nw = (unsigned)((p.L + kBlock / 64 - 1) / (kBlock / 64));
    const bool own = block < nw;
    int64_t i, ic;  // position in the list, and one that is always valid
    if (own) {
        i = (int64_t)block * (kBlock / 64) + (threadIdx.x >> 6);
        if (i >= p.L) return;  // whole waves
        i = ic = p.lng[i];
    } else {
        i = ((int64_t)(block - nw) * kBlock + threadIdx.x) / NV;
        ic = i < p.M ? i : p.M - 1;
    }
    const int v = lane % NV, vc = v < nvec ? v : 0;
    const int64_t r = p.rows[ic];
    uint64_t key[Wp];
#pragma unroll
    for (int w = 0; w < Wp; ++w) key[w] = s.keys[(int64_t)w * s.N + r];
    double are, aim = 0.0, x0r, x0i;
    load_x(r, vc, x0r, x0i);
    diag_term<CPLX>((double)dre[r], CPLX ? (double)dim[r] : 0.0, x0r, x0i, are, aim);
    auto add = [&](ET vre, ET vim, double xr, double xi) {
        if (CPLX) {
            are += (double)vre * xr - (double)vim * xi;
            aim += (double)vre * xi + (double)vim * xr;
        } else {
            are += (double)vre * xr;
        }
    };
    uint32_t e = p.ptr[ic];
    const uint32_t end = p.ptr[ic + 1];
    if (!own) {
        if (i >= p.M || v >= nvec || end - e > kLongRow) return;
        // two elements at a time, their records and x before either is evaluated
        for (; e < end; e += 2u) {
            qsd_hit q[2];
            double xr[2], xi[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) q[k] = p.rec[min(e + k, end - 1u)];
#pragma unroll
            for (int k = 0; k < 2; ++k) load_x(q[k].col, vc, xr[k], xi[k]);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (e + k >= end) continue;
                ET vre, vim;
                (void)range_value<Wp, ET>(h, key, q[k].t0, q[k].len, vre, vim);
                add(vre, vim, xr[k], xi[k]);
            }
        }
    } else {
        // 64 elements are evaluated, a lane each; then 64 / NV at a time have their x fetched and
        // every group of NV lanes adds the products in order
        for (; e < end; e += 64u) {
            const uint32_t n = min(64u, end - e);
            const qsd_hit q = p.rec[min(e + (uint32_t)lane, end - 1u)];
            ET vre, vim;
            (void)range_value<Wp, ET>(h, key, q.t0, q.len, vre, vim);
            // (one step's x in registers: eight steps' cost the streaming workgroups their occupancy)
#pragma unroll 1
            for (uint32_t c = 0; c < n; c += 64u / NV) {
                double xr, xi;
                load_x((uint32_t)__shfl((int)q.col, (int)min(c + (uint32_t)lane / NV, n - 1u), 64), vc, xr, xi);
                const uint32_t m = min(64u / NV, n - c);
                for (uint32_t k = 0; k < m; ++k) {
                    const ET a = (ET)__shfl(vre, (int)(c + k), 64);
                    const ET ai = CPLX ? (ET)__shfl(vim, (int)(c + k), 64) : (ET)0;
                    const double br = __shfl(xr, (int)k * NV + v, 64);
                    const double bi = CPLX ? __shfl(xi, (int)k * NV + v, 64) : 0.0;
                    add(a, ai, br, bi);
                }
            }
        }
        if (lane >= NV || v >= nvec) return;
    }
    if (CPLX) {
        y[2 * (r * ldy + v)] = (ET)are;
        y[2 * (r * ldy + v) + 1] = (ET)aim;
    } else {
        y[r * ldy + v] = (ET)are;
    }
}

__global__ void k_hit_zero(unsigned long long *p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

// f(integral_constant of the operator's key width)
template <class F>
void with_width(const qsd_ham *h, F f) {
    using std::integral_constant;
    switch (h->Wp) {
        case 1: f(integral_constant<int, 1>{}); break;
        case 2: f(integral_constant<int, 2>{}); break;
        case 4: f(integral_constant<int, 4>{}); break;
        case 8: f(integral_constant<int, 8>{}); break;
        case 16: f(integral_constant<int, 16>{}); break;
    }
}

// `small` takes three totals (elements, rows with many, those listed so far), `scratch` the rows' counts.
int build(const qsd_ham *h, qsd_hits *p, int64_t *&small, int64_t *&scratch, hipStream_t st) {
    const int64_t N = h->N, tiles = tiles_of(N);
    unsigned long long t[2] = {0, 0};
    QSD_TRY(dev_alloc(&small, 4));
    auto *total = (unsigned long long *)small;
    const SubView s = sub_view(h->s);
    const HamView v = ham_view(h, false);
    k_hit_zero<<<1, 64, 0, st>>>(total, 4);
    if (tiles > kSampleTiles || h->G > kSampleGroups) {
        with_width(h, [&](auto wp) {
            k_hit_sample<decltype(wp)::value><<<kSampleRows, kSampleThreads, 0, st>>>(s, v, total + 3);
        });
        QSD_CHECK_HIP(hipMemcpyAsync(t, total + 3, 8, hipMemcpyDeviceToHost, st));
        QSD_CHECK_HIP(hipStreamSynchronize(st));
        if ((double)t[0] > kSampleMean * kSampleRows) return QSD_OK;
    }
    QSD_TRY(dev_alloc(&scratch, N + 1));
    int64_t *cnt = scratch;
    QSD_TRY(dev_alloc(&p->rowbits, (size_t)((N + 63) / 64)));
    with_width(h, [&](auto wp) {
        k_hit_count<decltype(wp)::value><<<(unsigned)tiles, kBlock, 0, st>>>(s, v, cnt, p->rowbits, total);
    });
    int64_t sum = 0;
    QSD_TRY(exclusive_scan_i64(cnt, cnt, N + 1, st));  // (cnt[N] is read, and moves nothing)
    QSD_CHECK_HIP(hipMemcpyAsync(t, total, sizeof(t), hipMemcpyDeviceToHost, st));
    QSD_CHECK_HIP(hipMemcpyAsync(&sum, cnt + N, 8, hipMemcpyDeviceToHost, st));
    QSD_CHECK_HIP(hipStreamSynchronize(st));
    if (t[0] > (unsigned long long)N) return QSD_OK;
    p->H = (int64_t)t[0];
    p->M = sum >> 32;
    p->L = (int64_t)t[1];
    auto up = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
    const size_t at1 = up(p->H * sizeof(qsd_hit)), at2 = at1 + up(p->M * 4), at3 = at2 + up((p->M + 1) * 4);
    QSD_TRY(dev_alloc(&p->mem, at3 + p->L * 4));
    p->rec = (qsd_hit *)p->mem;
    p->rows = (uint32_t *)(p->mem + at1);
    p->ptr = (uint32_t *)(p->mem + at2);
    p->lng = (uint32_t *)(p->mem + at3);
    k_hit_rows<<<tiles_of(N + 1), kBlock, 0, st>>>(cnt, N, p->rows, p->ptr, p->lng, total + 2);
    if (p->M > 0)
        with_width(h, [&](auto wp) {
            k_hit_fill<decltype(wp)::value><<<tiles_of(p->M), kBlock, 0, st>>>(s, v, p->rows, p->M, p->ptr, p->rec);
        });
    QSD_CHECK_HIP(hipGetLastError());
    return QSD_OK;
}

template <int Wp, int NV, class ET, bool CPLX>
void launch(const qsd_ham *h, const qsd_hits *p, const void *x, int64_t ldx, void *y, int64_t ldy, int nvec,
            hipStream_t st) {
    constexpr bool f32 = std::is_same<ET, float>::value;
    const ET *dre = f32 ? (const ET *)h->diag32 : (const ET *)h->diag;
    const ET *dim = CPLX ? (f32 ? (const ET *)h->diag32_im : (const ET *)h->diag_im) : nullptr;
    const unsigned nd = (unsigned)((h->N * nvec + kBlock * kDiagItems - 1) / (kBlock * kDiagItems));
    const unsigned nl = (unsigned)((p->L + kBlock / 64 - 1) / (kBlock / 64)) + tiles_of(p->M * NV);
    const dim3 grid = folded_grid((int64_t)nl + nd, kBlock);
    k_hits_matvec<Wp, NV, ET, CPLX><<<grid, kBlock, 0, st>>>(sub_view(h->s), ham_view(h, f32), *p, dre, dim,
                                                               (const ET *)x, ldx, (ET *)y, ldy, nvec, nl);
}

template <int Wp, class ET, bool CPLX>
void by_width(const qsd_ham *h, const qsd_hits *p, const void *x, int64_t ldx, void *y, int64_t ldy, int nvec,
              hipStream_t st) {
    if (nvec <= 1)
        launch<Wp, 1, ET, CPLX>(h, p, x, ldx, y, ldy, nvec, st);
    else if (nvec <= 2)
        launch<Wp, 2, ET, CPLX>(h, p, x, ldx, y, ldy, nvec, st);
    else if (nvec <= 4 || CPLX)
        launch<Wp, 4, ET, CPLX>(h, p, x, ldx, y, ldy, nvec, st);
    else if (nvec <= 8)
        launch<Wp, CPLX ? 4 : 8, ET, CPLX>(h, p, x, ldx, y, ldy, nvec, st);
    else
        launch<Wp, CPLX ? 4 : 16, ET, CPLX>(h, p, x, ldx, y, ldy, nvec, st);
}

template <class ET, bool CPLX>
void by_key(const qsd_ham *h, const qsd_hits *p, const void *x, int64_t ldx, void *y, int64_t ldy, int nvec,
            hipStream_t st) {
    with_width(h, [&](auto wp) { by_width<decltype(wp)::value, ET, CPLX>(h, p, x, ldx, y, ldy, nvec, st); });
}

}  // namespace

void hits_free(qsd_hits *&p) {
    if (!p) return;
    dev_free(p->rowbits);
    dev_free(p->mem);
    delete p;
    p = nullptr;
}

int hits_build(const qsd_ham *h, qsd_hits **out, hipStream_t st) {
    *out = nullptr;
    if (h->N == 0 || h->G == 0) return QSD_OK;
    auto *p = new (std::nothrow) qsd_hits();
    if (!p) return fail(QSD_ERR_OUT_OF_MEMORY, "host allocation failed");
    int64_t *small = nullptr, *scratch = nullptr;
    int rc = build(h, p, small, scratch, st);
    dev_free(small);
    dev_free(scratch);
    if (rc == QSD_ERR_OUT_OF_MEMORY) {  // every caller has a path without the list
        clear_error();
        hits_free(p);
        return QSD_OK;
    }
    if (rc != QSD_OK || !p->mem)
        hits_free(p);
    else
        *out = p;
    return rc;
}

int hits_matvec(const qsd_ham *h, const qsd_hits *p, int nvec, const void *x, int64_t ldx, void *y, int64_t ldy,
                int32_t dtype, hipStream_t st) {
    const bool cplx = dtype == QSD_C128 || dtype == QSD_C64;
    const int chunk = cplx ? 4 : 16;
    const size_t esz = dtype == QSD_F64 ? 8 : dtype == QSD_F32 ? 4 : dtype == QSD_C128 ? 16 : 8;
    for (int v0 = 0; v0 < nvec; v0 += chunk) {
        const int nv = std::min(chunk, nvec - v0);
        const void *xv = (const char *)x + v0 * esz;
        void *yv = (char *)y + v0 * esz;
        switch (dtype) {
            case QSD_F64: by_key<double, false>(h, p, xv, ldx, yv, ldy, nv, st); break;
            case QSD_F32: by_key<float, false>(h, p, xv, ldx, yv, ldy, nv, st); break;
            case QSD_C128: by_key<double, true>(h, p, xv, ldx, yv, ldy, nv, st); break;
            case QSD_C64: by_key<float, true>(h, p, xv, ldx, yv, ldy, nv, st); break;
        }
    }
    QSD_CHECK_HIP(hipGetLastError());
    return QSD_OK;
}

}  // namespace qsd
