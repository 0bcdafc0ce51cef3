// Factored SpMV on alpha x beta product subspaces: the plan (lists built on the device from the
// operator's classification, factor.h) and the kernel.  See product.h for the form.
#include "product.h"

#include <algorithm>
#include <cstring>
#include <numeric>
#include <type_traits>

#include "device.h"
#include "factor.h"
#include "matvec.h"

namespace qsd {
namespace {

constexpr uint32_t kLdsBytes = 64u * 1024u;  // a workgroup's x row and tables (two or more workgroups per CU)
// Threads and low parts per workgroup.  1500 x 1500 strings in FP64: 256 1054 us, 384 1167 (four
// tiles with a short last one), 512 950, 768 979; 600 x 600: 98, 88, 88, 89.
constexpr uint32_t kMaxThreads = 512;
// Waves per SIMD that the registers must allow.  600 x 600: 88 us without it, 72 with 7; 8 costs
// scalar spills (300 x 301: 24.6 -> 26.4).  Four vectors spill at 7 (400 x 400 in FP32 46 us, at 5 44).
constexpr int waves_for(int V) { return V >= 4 ? 5 : 7; }
// Bytes of the lists: 24 MB for 1500 x 1500 strings of a 16-orbital molecule, 134 for all 4368 x 4368.
// Few low parts with many high ones of long class B tails can ask for gigabytes, in which case the plan
// may be at most as large as the subspace's own keys, hashes and table (128 bytes a row).
constexpr uint64_t kMaxLists = 1ull << 30, kMaxListsPerRow = 128;

// What the list kernels read of the operator.
struct GroupList {
    const uint32_t *flip;  // [n] the part's flip mask
    const uint32_t *t0;    // [n] first term
    const uint32_t *nt;    // [n] terms
    uint32_t n, n1;                     // groups, and those of segment 1
};
struct FlipList {
    const uint32_t *flip;  // [n]
    const uint32_t *care;  // [n] bits that select the flip's key
    const uint32_t *key0;  // [n + 1] keys of the flip
    const uint32_t *want;  // [keys]
    const uint32_t *sign;  // [keys]
    uint32_t n;
};
struct BuildView {
    const uint64_t *keys;    // [N] rows
    const uint32_t *pfilt;
    const uint16_t *prank;
    const uint4 *cw;         // [T] care, want, sign
    const double2 *coef;     // [T]
    const float2 *coef32;    // [T]
    const uint32_t *tinfo;   // [T] kind | key << 8
    uint32_t na, nb;
    int split;
};

__device__ __forceinline__ uint32_t below(uint64_t m, int lane) {
    return (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
}

// Position of a lane's flip in its part's list of keys: the flip's key that matches the part
// (at most one does), or -1.
__device__ __forceinline__ int flip_key(const FlipList &f, uint32_t i, uint32_t part, uint32_t &sgn) {
    const uint32_t c = part & f.care[i];
    for (uint32_t k = f.key0[i]; k < f.key0[i + 1]; ++k)
        if (c == f.want[k]) {
            sgn = (uint32_t)__popc(part & f.sign[k]) & 1u;
            return (int)k;
        }
    return -1;
}

// The lists of one part, one workgroup per part: 64 groups (flips) at a time, the entries that exist
// keep their order through a ballot; each wave takes a run of the groups and of the flips.  WRITE = false
// only counts: entries per wave (which tell a wave where to write), lengths and their maxima.
// Latency-bound (a chain of reads per 64 groups): 300 x 300 strings of a 16-orbital molecule, 1940
// groups and 120 flips a part: 372 us with a wave per part and a launch each for low and high ones, 117 so.
constexpr uint32_t kListWaves = 8;

template <bool HIGH, bool WRITE>
__device__ __forceinline__ void prod_lists(const BuildView &v, const GroupList &g, const FlipList &f, const qsd_prod &p,
                                           uint32_t i, uint32_t *__restrict__ cnt, uint32_t *__restrict__ mx,
                                           uint32_t (*__restrict__ sums)[3]) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, n = HIGH ? v.nb : v.na;
    const uint32_t lowmask = (1u << v.split) - 1u;
    const uint32_t part = HIGH ? (uint32_t)(v.keys[(int64_t)i * v.na] >> v.split) : (uint32_t)v.keys[i] & lowmask;
    const uint32_t *filt = v.pfilt + (HIGH ? kPartWords / 2 : 0);
    const uint32_t at = !HIGH && WRITE ? p.place[i] : i;  // a low part's position
    cnt += (HIGH ? (int64_t)v.na + i : (int64_t)i) * kListWaves * 3;
    uint32_t n1 = 0, n2 = 0, n3 = 0;
    if (WRITE)
        for (uint32_t w = 0; w < wave; ++w) {
            n1 += cnt[3 * w];
            n2 += cnt[3 * w + 1];
            n3 += cnt[3 * w + 2];
        }
    auto run = [&](uint32_t len) { return ((len + 63u) / 64u + kListWaves - 1u) / kListWaves * 64u; };
    const uint32_t gr = run(g.n), fr = run(f.n);
    for (uint32_t g0 = wave * gr; g0 < min(wave * gr + gr, g.n); g0 += 64u) {
        const uint32_t q = g0 + lane;
        bool on = false;
        uint32_t col = 0, key = 0, sgn = 0, nt = 0;
        double val = 0.0;
        float val32 = 0.0f;
        // segment 1's slot in the lists is known only after the ballot: its tail terms are
        // written in a second walk below
        if (q < g.n) {
            const uint32_t to = part ^ g.flip[q];
            if ((filt[to >> 5] >> (to & 31u)) & 1u) {
                col = part_rank(v.pfilt, v.prank, HIGH ? 1 : 0, to);
                key = HIGH ? 2u * (p.nWb - 1u) : 2u * (p.nUa - 1u);  // the table row of zeros
                for (uint32_t t = g.t0[q]; t < g.t0[q] + g.nt[q]; ++t) {
                    const uint4 m = v.cw[t];
                    const uint32_t care = HIGH ? m.x >> v.split : m.x & lowmask;
                    const uint32_t want = HIGH ? m.y >> v.split : m.y & lowmask;
                    if ((part & care) != want) continue;
                    const uint32_t s = (uint32_t)__popc(part & (HIGH ? m.z >> v.split : m.z & lowmask)) & 1u;
                    const uint32_t info = v.tinfo[t];
                    if ((info & 255u) == kOwn) {
                        on = true;
                        ++nt;
                        val += s ? -v.coef[t].x : v.coef[t].x;
                        val32 += s ? -v.coef32[t].x : v.coef32[t].x;
                    } else {
                        if ((info & 255u) == kFirst) on = true;
                        key = 2u * (info >> 8) + s;
                    }
                }
            }
        }
        const uint64_t b1 = __ballot(on && q < g.n1), b2 = __ballot(on && q >= g.n1);
        if (WRITE && on) {
            if (q < g.n1) {
                const uint32_t k = n1 + below(b1, (int)lane);
                if (HIGH) {
                    uint32_t *e = p.b1_ent + 2 * ((int64_t)i * p.nB1 + k);
                    e[0] = col;
                    e[1] = key | nt << 24;
                    const int64_t o = ((int64_t)i * p.nB1 + k) * p.tail_len;
                    uint32_t at = 0;
                    for (uint32_t t = g.t0[q]; t < g.t0[q] + g.nt[q]; ++t) {
                        const uint4 m = v.cw[t];
                        if ((part & (m.x >> v.split)) != (m.y >> v.split) || (v.tinfo[t] & 255u) != kOwn) continue;
                        const bool s = (__popc(part & (m.z >> v.split)) & 1) != 0;
                        p.d.tail[o + at] = s ? -v.coef[t].x : v.coef[t].x;
                        p.f.tail[o + at] = s ? -v.coef32[t].x : v.coef32[t].x;
                        ++at;
                    }
                } else {
                    const int64_t o = (int64_t)k * v.na + at;
                    p.a1_ent[o] = col | key << 16;
                    p.d.a1[o] = val;
                    p.f.a1[o] = val32;
                }
            } else {
                const uint32_t k = n2 + below(b2, (int)lane);
                const int64_t o = HIGH ? (int64_t)i * p.nB2 + k : prod_at(k, v.na, at);
                if (HIGH)
                    p.b2_col[o] = col;
                else
                    p.a2_col[o] = (uint16_t)col;
                (HIGH ? p.d.b2 : p.d.a2)[o] = val;
                (HIGH ? p.f.b2 : p.f.a2)[o] = val32;
            }
        }
        n1 += (uint32_t)__popcll(b1);
        n2 += (uint32_t)__popcll(b2);
    }
    for (uint32_t f0 = wave * fr; f0 < min(wave * fr + fr, f.n); f0 += 64u) {
        const uint32_t q = f0 + lane;
        uint32_t col = 0, sgn = 0;
        int key = -1;
        if (q < f.n) {
            const uint32_t to = part ^ f.flip[q];
            if ((filt[to >> 5] >> (to & 31u)) & 1u) {
                col = part_rank(v.pfilt, v.prank, HIGH ? 1 : 0, to);
                key = flip_key(f, q, part, sgn);
            }
        }
        const uint64_t b3 = __ballot(key >= 0);
        if (WRITE && key >= 0) {
            const uint32_t k = n3 + below(b3, (int)lane);
            if (HIGH) {
                uint32_t *e = p.bab_ent + 2 * ((int64_t)i * p.nBAB + k);
                e[0] = col;
                e[1] = 2u * (uint32_t)key + sgn;
            } else {
                p.ab_ent[prod_at(k, v.na, at)] = col | (2u * (uint32_t)key + sgn) << 16;
            }
        }
        n3 += (uint32_t)__popcll(b3);
    }
    if (!WRITE) {
        if (lane == 0) {
            cnt[3 * wave] = sums[wave][0] = n1;
            cnt[3 * wave + 1] = sums[wave][1] = n2;
            cnt[3 * wave + 2] = sums[wave][2] = n3;
        }
        __syncthreads();
        if (threadIdx.x < 3u) {
            uint32_t t = 0;
            for (uint32_t w = 0; w < kListWaves; ++w) t += sums[w][threadIdx.x];
            (HIGH ? p.blen : p.alen)[threadIdx.x * (int64_t)n + i] = t;
            atomicMax(&mx[(HIGH ? 4u : 0u) + threadIdx.x], t);
        }
        if (HIGH && threadIdx.x == 0) {
            p.blen[3 * (int64_t)n + i] = part;
            atomicMax(&mx[7], (uint32_t)__popc(part & p.rmask));
        }
    } else if (!HIGH) {
        // the lengths by position, and the rest of A2 and AB: entries that add 0 * 0 (the zeros after x's
        // row and after the coefficients), so that a wave's lanes walk them without a test
        uint32_t t[3] = {0u, 0u, 0u};
        for (uint32_t w = 0; w < kListWaves; ++w)
            for (int k = 0; k < 3; ++k) t[k] += cnt[3 * w + k];
        const uint32_t zero = 2u * p.nU;
        for (uint32_t k = t[1] + threadIdx.x; k < p.nA2; k += 64u * kListWaves) {
            const int64_t o = prod_at(k, v.na, at);
            p.a2_col[o] = (uint16_t)v.na;
            p.d.a2[o] = 0.0;
            p.f.a2[o] = 0.0f;
        }
        for (uint32_t k = t[2] + threadIdx.x; k < p.nAB; k += 64u * kListWaves)
            p.ab_ent[prod_at(k, v.na, at)] = v.na | zero << 16;
        if (threadIdx.x < 3u) p.alen[threadIdx.x * (int64_t)n + at] = t[threadIdx.x];
    }
}

template <bool WRITE>
__global__ __launch_bounds__(64 * kListWaves) void k_prod_lists(BuildView v, GroupList ga, FlipList fa, GroupList gb,
                                                                FlipList fb, qsd_prod p, uint32_t *__restrict__ cnt,
                                                                uint32_t *__restrict__ mx) {
    __shared__ uint32_t sums[kListWaves][3];
    if (blockIdx.x < v.na)
        prod_lists<false, WRITE>(v, ga, fa, p, blockIdx.x, cnt, mx, sums);
    else
        prod_lists<true, WRITE>(v, gb, fb, p, blockIdx.x - v.na, cnt, mx, sums);
}

// wtab[w][a] = the key's first term plus its terms that want a low qubit the part has set, in
// increasing qubit order (dep[w][q], 0 where there is none).
template <class ET>
__global__ __launch_bounds__(256) void k_prod_wtab(const uint64_t *__restrict__ keys, uint32_t na, int split,
                                                   const ET *__restrict__ head, const ET *__restrict__ dep,
                                                   ET *__restrict__ wtab) {
    const uint32_t a = blockIdx.x * 256u + threadIdx.x, w = blockIdx.y;
    if (a >= na) return;
    const uint32_t part = (uint32_t)keys[a] & ((1u << split) - 1u);
    ET s = 0;
    s += head[w];
    for (int q = 0; q < split; ++q)
        if ((part >> q) & 1u) s += dep[(int64_t)w * split + q];
    wtab[(int64_t)w * na + a] = s;
}

// ------------------------------------------------------------------------------- SpMV

// Four values of a list at once.
template <class T>
struct alignas(4 * sizeof(T)) Four {
    T v[4];
};

// Where the class B tails lie in a workgroup's LDS: after x with its zero and `aux` table entries, and
// after the sums in rank order.
template <class ET>
__host__ __device__ inline uint32_t tail_at(uint32_t na, uint32_t T, uint32_t aux, int V) {
    const uint32_t a = ((na + 1u) * V + aux) * (uint32_t)sizeof(ET), b = T * V * 8u;
    return ((a > b ? a : b) + 31u) / 32u * 32u;
}

// V values of the interleaved vectors, read or written at once.
template <class ET, int V>
struct alignas(V * sizeof(ET) < 16 ? V * sizeof(ET) : 16) Pack {
    ET v[V];
};

// Whether a workgroup's V vectors can be: all of them are there, and aligned.
template <class ET, int V>
__device__ __forceinline__ bool wide(const ET *x, int64_t ldx, const ET *y, int64_t ldy, int nv) {
    return V > 1 && nv == V &&
           (((uintptr_t)x | (uintptr_t)y | (uintptr_t)(ldx * sizeof(ET)) | (uintptr_t)(ldy * sizeof(ET))) &
            (alignof(Pack<ET, V>) - 1u)) == 0u;
}

// One workgroup: T low parts of the high part b, V of the interleaved vectors.  Class A and AB
// columns lie in whole rows x[b'][:], which are staged in LDS (12 KB for 1500 strings in FP64), so
// the random gathers run at the LDS rate and not at the 0.36 lanes per clock and CU that the texture
// path gives gathers from L2; the high part's own lists are uniform over the workgroup (scalar
// loads), and class B reads x[b'][a] coalesced.
//
// The low parts of a tile sit in lanes by the length of their AB lists, so the lanes of a wave end
// together (in rank order a wave of 1500 strings walks 27 entries for a mean of 19), and A2 and AB
// are padded with entries that add 0 * 0 and read four at a time, so there is no lane test and no
// remainder loop.  Before class B the sums go back to rank order through LDS.  Lists in rank order
// with a remainder loop: 1500 x 1500 1200 -> 950 us, 600 x 600 117 -> 88.  With the class B tails in
// LDS 920 and (88 -> 72 by the registers' bound) 69.
//
// Bound: LDS.  An AB element is two LDS reads (coefficient, x) at random banks, some three and a half
// passes each; 1500 x 1500 has 970 M of them.  Two high parts per workgroup, which share the list
// reads, gained nothing here (1115 us) and loading the next row into registers ahead of its turn 2 %.
//
// With several vectors a lane's values lie ldx apart from the next lane's, so an instruction that
// reads one of them meets 64 lines: WIDE reads all V at once (300 x 300, 8 vectors in FP64 102 -> 68 us,
// 400 x 400, 4 in FP32 80 -> 44; eight vectors per workgroup spill: 80 and 16 vectors 184 for 228).
template <class ET, int V, bool WIDE>
__device__ __forceinline__ void prod_block(const ProdView<ET> &p, const ET *__restrict__ x, int64_t ldx,
                                           ET *__restrict__ y, int64_t ldy, int nv, uint32_t tile, uint32_t b,
                                           char *smem) {
    ET *xs = (ET *)smem;                     // [na + 1][V], the last 0
    ET *aux = xs + (size_t)(p.na + 1u) * V;  // class A table rows, then the AB coefficients
    const uint32_t B = blockDim.x;
    const uint32_t pos = tile * p.T + threadIdx.x;
    const bool valid = threadIdx.x < p.T && pos < p.na;
    const uint32_t at = valid ? pos : p.na - 1u;

    using Vec = Pack<ET, V>;
    auto get = [&](const ET *at) {
        Vec t;
        if constexpr (WIDE) {
            t = *(const Vec *)at;
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) t.v[v] = (V == 1 || v < nv) ? at[v] : (ET)0;
        }
        return t;
    };
    auto stage = [&](uint32_t bc) {
        const ET *xr = x + (int64_t)bc * p.na * ldx;
        for (uint32_t j = threadIdx.x; j < p.na; j += B) *(Vec *)(xs + j * V) = get(xr + (int64_t)j * ldx);
    };
    // a wave's longest list, in steps of four
    auto wave_steps = [](uint32_t n) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) n = max(n, (uint32_t)__shfl_xor((int)n, d, 64));
        return ((uint32_t)__builtin_amdgcn_readfirstlane((int)n) + 3u) / 4u;
    };
    const uint32_t al = p.order[at];  // the lane's low part up to class B
    double acc[V];
    {
        const int64_t row = (int64_t)b * p.na + al;
        const double dr = (double)p.diag[row];
        const Vec t = get(x + row * ldx);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = dr * (double)t.v[v];
    }
    const uint32_t n1 = valid ? p.alen[at] : 0u;
    const uint32_t n2 = wave_steps(valid ? p.alen[p.na + at] : 0u);
    const uint32_t n3 = wave_steps(valid ? p.alen[2 * (int64_t)p.na + at] : 0u);
    // class A: columns of the row's own block
    const uint32_t occ = p.blen[3 * (int64_t)p.nb + b] & p.rmask;
    const uint32_t nocc = (uint32_t)__popc(occ);
    if (threadIdx.x < V) xs[p.na * V + threadIdx.x] = (ET)0;
    // class B terms after the table, in fours (0 past the last), where the sums at the end leave them
    const uint32_t m1 = p.blen[b], m2 = p.blen[p.nb + b], tl = (p.tail_len + 3u) / 4u * 4u;
    ET *tails = (ET *)(smem + tail_at<ET>(p.na, p.T, p.aux, V));
    for (uint32_t k = threadIdx.x; k < m1 * tl; k += B) {
        const uint32_t i = k / tl, t = k - i * tl;
        const int64_t o = (int64_t)b * p.nB1 + i;
        // (read from L2 one by one they were a chain of scalar loads: 1500 x 1500 950 us, 337 x 411 29)
        tails[k] = t < p.b1_ent[2 * o + 1] >> 24 ? p.tail[o * p.tail_len + t] : (ET)0;
    }
    stage(b);
    uint32_t m = occ;
    for (uint32_t r = 0; m; ++r, m &= m - 1u) {
        const ET *d = p.dep + (int64_t)__builtin_ctz(m) * p.nUa;
        for (uint32_t u = threadIdx.x; u < p.nUa; u += B) aux[r * p.nUa + u] = d[u];
    }
    __syncthreads();
#pragma unroll 2
    for (uint32_t k = 0; k < n1; ++k) {
        const uint32_t e = p.a1_ent[(int64_t)k * p.na + at];
        ET val = p.a1[(int64_t)k * p.na + at];
        const uint32_t u = e >> 17, col = e & 0xFFFFu;
        const bool neg = (e >> 16) & 1u;
        for (uint32_t r = 0; r < nocc; ++r) {
            const ET c = aux[r * p.nUa + u];
            val += neg ? -c : c;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] += (double)val * (double)xs[col * V + v];
    }
    {
        const auto *cols = (const Four<uint16_t> *)p.a2_col;
        const auto *vals = (const Four<ET> *)p.a2;
#pragma unroll(V == 1 ? 2 : 1)
        for (uint32_t k = 0; k < n2; ++k) {
            const Four<uint16_t> col = cols[(int64_t)k * p.na + at];
            const Four<ET> val = vals[(int64_t)k * p.na + at];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < V; ++v)
                    acc[v] += (double)val.v[j] * (double)xs[(uint32_t)col.v[j] * V + v];
        }
    }
    // class AB: each flip of the high part brings a row of x and its key's coefficients (both signs:
    // entry 2 u + s is the coefficient with the low part's sign s applied, the last is 0; 0 = the
    // pair of keys has no term)
    const uint32_t nab = p.blen[2 * (int64_t)p.nb + b];
    const auto *ents = (const Four<uint32_t> *)p.ab_ent;
    auto class_ab = [&](auto full) {
        for (uint32_t i = 0; i < nab; ++i) {
            const uint32_t *ent = p.bab_ent + 2 * ((int64_t)b * p.nBAB + i);
            const ET *ct = p.ctab + (int64_t)(ent[1] >> 1) * p.nU;
            __syncthreads();  // the previous row and tables are no longer read
            stage(ent[0]);
            for (uint32_t u = threadIdx.x; u < p.nU; u += B) {
                const ET c = (ent[1] & 1u) ? -ct[u] : ct[u];
                aux[2 * u] = c;
                aux[2 * u + 1] = -c;
            }
            if (threadIdx.x == 0) aux[2 * p.nU] = (ET)0;
            __syncthreads();
#pragma unroll(V == 1 ? 2 : 1)
            for (uint32_t k = 0; k < n3; ++k) {
                const Four<uint32_t> f = ents[(int64_t)k * p.na + at];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const ET c = aux[f.v[j] >> 16];
                    const uint32_t col = f.v[j] & 0xFFFFu;
                    if (decltype(full)::value || c != (ET)0) {
#pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] += (double)c * (double)xs[col * V + v];
                    }
                }
            }
        }
    };
    if (p.full)
        class_ab(std::true_type{});
    else
        class_ab(std::false_type{});
    // back to rank order
    double *ex = (double *)smem;  // [T][V]
    __syncthreads();
    if (valid) {
#pragma unroll
        for (int v = 0; v < V; ++v) ex[(al - tile * p.T) * V + v] = acc[v];
    }
    __syncthreads();
    if (!valid) return;
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = ex[threadIdx.x * V + v];
    // class B: the same low part in other blocks
    const uint32_t a = pos;
    const ET *xa = x + (int64_t)a * ldx;
    const int64_t bstride = (int64_t)p.na * ldx;
    for (uint32_t i = 0; i < m1; ++i) {
        const int64_t o = (int64_t)b * p.nB1 + i;
        const uint32_t bc = p.b1_ent[2 * o], e = p.b1_ent[2 * o + 1];
        const uint32_t w = (e & 0xFFFFFFu) >> 1, nt = e >> 24;
        const ET wv = p.wtab[(int64_t)w * p.na + a];
        const Vec t = get(xa + bc * bstride);
        ET val = (e & 1u) ? -wv : wv;
        for (uint32_t q = 0; q < nt; q += 4u) {
            const Four<ET> c = *(const Four<ET> *)(tails + i * tl + q);
#pragma unroll
            for (int j = 0; j < 4; ++j) val += c.v[j];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] += (double)val * (double)t.v[v];
    }
#pragma unroll 8
    for (uint32_t i = 0; i < m2; ++i) {
        const int64_t o = (int64_t)b * p.nB2 + i;
        const double val = (double)p.b2[o];
        const Vec t = get(xa + p.b2_col[o] * bstride);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] += val * (double)t.v[v];
    }
    ET *yr = y + ((int64_t)b * p.na + a) * ldy;
    if constexpr (WIDE) {
        Vec t;
#pragma unroll
        for (int v = 0; v < V; ++v) t.v[v] = (ET)acc[v];
        *(Vec *)yr = t;
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (V == 1 || v < nv) yr[v] = (ET)acc[v];
    }
}

template <class ET, int V>
__global__ __launch_bounds__(kMaxThreads, waves_for(V)) void k_prod_matvec(ProdView<ET> p, const ET *__restrict__ x,
                                                                    int64_t ldx, ET *__restrict__ y, int64_t ldy,
                                                                    int nvec) {
    extern __shared__ __align__(32) char smem[];
    // workgroups of one XCD take consecutive high parts of one tile of low parts: they share the
    // tile's lists in that XCD's L2
    const uint32_t id = (uint32_t)tile_index(blockIdx.x, gridDim.x, true);
    const uint32_t tile = id / p.nb;
    const int v0 = blockIdx.y * V;
    const int nv = min(V, nvec - v0);
    x += v0;
    y += v0;
    if (wide<ET, V>(x, ldx, y, ldy, nv))
        prod_block<ET, V, (V > 1)>(p, x, ldx, y, ldy, nv, tile, id - tile * p.nb, smem);
    else
        prod_block<ET, V, false>(p, x, ldx, y, ldy, nv, tile, id - tile * p.nb, smem);
}

// Requests of a table: a workgroup finds its request by the requests' first workgroups.
template <class ET, int V>
__global__ __launch_bounds__(kMaxThreads, waves_for(V)) void k_prod_batched(const ProdReq<ET> *__restrict__ reqs, int n,
                                                                           uint32_t blocks) {
    extern __shared__ __align__(32) char smem[];
    const uint32_t block = blockIdx.y * gridDim.x + blockIdx.x;
    if (block >= blocks) return;
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (reqs[mid].first <= block)
            lo = mid;
        else
            hi = mid - 1;
    }
    const ProdReq<ET> &R = reqs[lo];
    if (R.kdev && *R.kdev >= R.m) return;  // at its iteration limit (uniform for the block)
    uint32_t id = block - R.first;
    const uint32_t per = (R.p.na + R.p.T - 1u) / R.p.T * R.p.nb;  // workgroups per vector chunk
    const uint32_t vc = id / per;
    id -= vc * per;
    const uint32_t tile = id / R.p.nb;
    const int v0 = (int)vc * V;
    const int nv = min(V, R.nv - v0);
    if (wide<ET, V>(R.x + v0, R.ld, R.y + v0, R.ld, nv))
        prod_block<ET, V, (V > 1)>(R.p, R.x + v0, R.ld, R.y + v0, R.ld, nv, tile, id - tile * R.p.nb, smem);
    else
        prod_block<ET, V, false>(R.p, R.x + v0, R.ld, R.y + v0, R.ld, nv, tile, id - tile * R.p.nb, smem);
}

uint32_t tiles_of(const qsd_prod *p) { return (p->na + p->T - 1u) / p->T; }

// LDS of a workgroup: x and the zero after it, the class A table rows or the AB coefficients and the
// zero after them (then the sums in rank order), and the class B tails.
uint32_t aux_entries(const qsd_prod *p) { return std::max(p->max_occ * p->nUa, 2u * p->nU + 1u); }

template <class ET>
uint32_t lds_bytes(const qsd_prod *p, int V) {
    return tail_at<ET>(p->na, p->T, aux_entries(p), V) + p->nB1 * ((p->tail_len + 3u) / 4u * 4u) * (uint32_t)sizeof(ET);
}

// ------------------------------------------------------------------------------- plan

std::vector<float> narrowed(const std::vector<double> &v) { return std::vector<float>(v.begin(), v.end()); }

constexpr int kNoPlan = 1;  // the lists do not fit: no error, and no plan

// The lists: counted, sized by one round trip to the host, then written.  `scratch` and `keep`
// hold the host images, which the caller keeps until the stream has passed the copies.
int build_device(qsd_ham *h, qsd_prod *p, const Classified &c, Block &scratch, Block &keep, Block &lists,
                 size_t tables, hipStream_t st) {
    const qsd_subspace *s = h->s;
    // The product map needs none of this memory, so a block that is refused means no plan; only one
    // that is no larger than the operator's tables counts as one of them (where that does not fit,
    // neither do the vectors).
    auto alloc = [&](Block &b) -> int {
        const int rc = dev_alloc(&b.dev, b.size());
        if (rc != QSD_ERR_OUT_OF_MEMORY || b.size() <= tables) return rc;
        clear_error();
        return kNoPlan;
    };
    size_t og[2][3], of[2][5];
    for (int H = 0; H < 2; ++H) {
        og[H][0] = scratch.put(c.gflip[H]);
        og[H][1] = scratch.put(c.gt0[H]);
        og[H][2] = scratch.put(c.gnt[H]);
        of[H][0] = scratch.put(c.fflip[H]);
        of[H][1] = scratch.put(c.fcare[H]);
        of[H][2] = scratch.put(c.fkey0[H]);
        of[H][3] = scratch.put(c.fwant[H]);
        of[H][4] = scratch.put(c.fsign[H]);
    }
    const size_t oi = scratch.put(c.tinfo), om = scratch.put(std::vector<uint32_t>(8, 0u));
    const size_t owh = scratch.put(c.whead), owd = scratch.put(c.wdep);
    const size_t owh32 = scratch.put(narrowed(c.whead)), owd32 = scratch.put(narrowed(c.wdep));
    const size_t on = scratch.room(((size_t)p->na + p->nb) * kListWaves * 3 * 4);
    const size_t od = keep.put(c.dep), od32 = keep.put(narrowed(c.dep));
    const size_t oc = keep.put(c.ctab), oc32 = keep.put(narrowed(c.ctab));
    const size_t oa = keep.room(3 * (size_t)p->na * 4), ob = keep.room(4 * (size_t)p->nb * 4);
    QSD_TRY(alloc(scratch));
    QSD_TRY(scratch.copy(st));
    QSD_TRY(alloc(keep));
    QSD_TRY(keep.copy(st));
    p->d.dep = keep.at<double>(od);
    p->f.dep = keep.at<float>(od32);
    p->d.ctab = keep.at<double>(oc);
    p->f.ctab = keep.at<float>(oc32);
    p->alen = keep.at<uint32_t>(oa);
    p->blen = keep.at<uint32_t>(ob);
    const BuildView v{s->keys, s->pfilt, s->prank, (const uint4 *)h->t_cw32, (const double2 *)h->t_coef,
                      (const float2 *)h->t_coef32, scratch.at<uint32_t>(oi), p->na, p->nb, p->split};
    GroupList g[2];
    FlipList f[2];
    for (int H = 0; H < 2; ++H) {
        g[H] = GroupList{scratch.at<uint32_t>(og[H][0]), scratch.at<uint32_t>(og[H][1]), scratch.at<uint32_t>(og[H][2]),
                         (uint32_t)c.gflip[H].size(), c.n1[H]};
        f[H] = FlipList{scratch.at<uint32_t>(of[H][0]), scratch.at<uint32_t>(of[H][1]), scratch.at<uint32_t>(of[H][2]),
                        scratch.at<uint32_t>(of[H][3]), scratch.at<uint32_t>(of[H][4]), (uint32_t)c.fflip[H].size()};
    }
    uint32_t *mx = scratch.at<uint32_t>(om);
    uint32_t *cnt = scratch.at<uint32_t>(on);
    k_prod_lists<false><<<p->na + p->nb, 64 * kListWaves, 0, st>>>(v, g[0], f[0], g[1], f[1], *p, cnt, mx);
    uint32_t m[8];
    std::vector<uint32_t> n3(p->na);
    QSD_CHECK_HIP(hipMemcpyAsync(m, mx, sizeof(m), hipMemcpyDeviceToHost, st));
    QSD_CHECK_HIP(hipMemcpyAsync(n3.data(), p->alen + 2 * (size_t)p->na, (size_t)p->na * 4, hipMemcpyDeviceToHost, st));
    QSD_CHECK_HIP(hipStreamSynchronize(st));
    p->nA1 = m[0];
    p->nA2 = (m[1] + 3u) / 4u * 4u;
    p->nAB = (m[2] + 3u) / 4u * 4u;
    p->nB1 = m[4];
    p->nB2 = m[5];
    p->nBAB = m[6];
    p->max_occ = m[7];
    if (lds_bytes<double>(p, 1) > kLdsBytes) return kNoPlan;
    // within each tile, the low parts by the length of their AB lists
    const size_t na = p->na, nb = p->nb;
    std::vector<uint32_t> order(na), place(na);
    std::iota(order.begin(), order.end(), 0u);
    for (size_t t = 0; t < na; t += p->T)
        std::stable_sort(order.begin() + t, order.begin() + std::min<size_t>(na, t + p->T),
                         [&](uint32_t i, uint32_t j) { return n3[i] > n3[j]; });
    for (size_t i = 0; i < na; ++i) place[order[i]] = (uint32_t)i;
    const size_t oo = lists.put(std::move(order)), op = lists.put(std::move(place));
    const size_t o1 = lists.room(4 * p->nA1 * na), o2 = lists.room(2 * p->nA2 * na), o3 = lists.room(4 * p->nAB * na);
    const size_t o4 = lists.room(8 * p->nB1 * nb), o5 = lists.room(4 * p->nB2 * nb), o6 = lists.room(8 * p->nBAB * nb);
    size_t ov[2][5];
    for (int k = 0; k < 2; ++k) {
        const size_t e = k ? 4 : 8;
        ov[k][0] = lists.room(e * p->nA1 * na);
        ov[k][1] = lists.room(e * p->nA2 * na);
        ov[k][2] = lists.room(e * p->nWb * na);
        ov[k][3] = lists.room(e * nb * p->nB1 * p->tail_len);
        ov[k][4] = lists.room(e * nb * p->nB2);
    }
    if (lists.size() > std::max(kMaxLists, kMaxListsPerRow * (uint64_t)s->N)) return kNoPlan;
    QSD_TRY(alloc(lists));
    QSD_TRY(lists.copy(st));
    p->order = lists.at<uint32_t>(oo);
    p->place = lists.at<uint32_t>(op);
    p->a1_ent = lists.at<uint32_t>(o1);
    p->a2_col = lists.at<uint16_t>(o2);
    p->ab_ent = lists.at<uint32_t>(o3);
    p->b1_ent = lists.at<uint32_t>(o4);
    p->b2_col = lists.at<uint32_t>(o5);
    p->bab_ent = lists.at<uint32_t>(o6);
    auto values = [&](auto &w, const size_t *o) {
        using T = std::remove_pointer_t<decltype(w.a1)>;
        w.a1 = lists.at<T>(o[0]);
        w.a2 = lists.at<T>(o[1]);
        w.wtab = lists.at<T>(o[2]);
        w.tail = lists.at<T>(o[3]);
        w.b2 = lists.at<T>(o[4]);
    };
    values(p->d, ov[0]);
    values(p->f, ov[1]);
    k_prod_lists<true><<<p->na + p->nb, 64 * kListWaves, 0, st>>>(v, g[0], f[0], g[1], f[1], *p, cnt, nullptr);
    const dim3 gw((p->na + 255u) / 256u, p->nWb);
    k_prod_wtab<double><<<gw, 256, 0, st>>>(s->keys, p->na, p->split, scratch.at<double>(owh), scratch.at<double>(owd),
                                           p->d.wtab);
    k_prod_wtab<float><<<gw, 256, 0, st>>>(s->keys, p->na, p->split, scratch.at<float>(owh32),
                                          scratch.at<float>(owd32), p->f.wtab);
    QSD_CHECK_HIP(hipGetLastError());
    return QSD_OK;
}

}  // namespace

void prod_free(qsd_prod *&p) {
    if (!p) return;
    dev_free(p->mem[0]);
    dev_free(p->mem[1]);
    delete p;
    p = nullptr;
}

int prod_build(qsd_ham *h, size_t tables, hipStream_t st) {
    const qsd_subspace *s = h->s;
    if (!s->prank || h->is_complex || h->G == 0) return QSD_OK;
    // the x row of one block and the tables have to fit a workgroup's LDS
    if ((uint64_t)s->pna * sizeof(double) > kLdsBytes) return QSD_OK;
    const bool kept = h->op->parts && h->op->parts->split == s->split;
    const Classified other = kept ? Classified() : classify(h->op, s->split);
    const Classified &c = kept ? *h->op->parts : other;
    if (!c.ok || (uint64_t)c.nWb * s->pna > kMaxTable) return QSD_OK;
    auto *p = new (std::nothrow) qsd_prod();
    if (!p) return fail(QSD_ERR_OUT_OF_MEMORY, "host allocation failed");
    p->split = s->split;
    p->na = s->pna;
    // tiles of up to kMaxThreads low parts, of one size, in whole waves
    const uint32_t tiles = (p->na + kMaxThreads - 1u) / kMaxThreads;
    p->T = ((p->na + tiles - 1u) / tiles + 63u) / 64u * 64u;
    p->nb = (uint32_t)(s->N / s->pna);
    p->nUa = c.nUa;
    p->nU = (uint32_t)c.fwant[0].size();
    p->nW = (uint32_t)c.fwant[1].size();
    p->nWb = c.nWb;
    p->tail_len = c.tail_len;
    p->rmask = c.rmask;
    p->full = c.full;
    Block scratch, keep, lists;
    int rc = build_device(h, p, c, scratch, keep, lists, tables, st);
    // the host images outlive their copies
    if (hipStreamSynchronize(st) != hipSuccess && rc == QSD_OK)
        rc = fail(QSD_ERR_HIP, "product lists failed: %s", hipGetErrorString(hipGetLastError()));
    dev_free(scratch.dev);
    p->mem[0] = keep.dev;
    p->mem[1] = lists.dev;
    if (rc != QSD_OK) {
        prod_free(p);
        return rc == kNoPlan ? QSD_OK : rc;
    }
    h->prod = p;
    return QSD_OK;
}

bool prod_usable(const qsd_ham *h) {
    return h->prod && h->s->prank && h->s->split == h->prod->split && !(h->schedule & QSD_SCHED_HASH_LOOKUP);
}

template <class ET>
ProdView<ET> prod_view(const qsd_ham *h) {
    const qsd_prod *p = h->prod;
    const ProdVals<ET> *v;
    const ET *diag;
    if constexpr (std::is_same<ET, double>::value) {
        v = &p->d;
        diag = h->diag;
    } else {
        v = &p->f;
        diag = h->diag32;
    }
    return ProdView<ET>{p->na, p->nb, p->T, aux_entries(p), p->nB1, p->nB2, p->nBAB, p->nUa, p->nU, p->tail_len, p->rmask,
                        p->full ? 1u : 0u,
                        p->a1_ent, p->a2_col, p->ab_ent, p->b1_ent, p->b2_col, p->bab_ent, p->alen, p->blen, p->order,
                        p->place, v->a1, v->a2, v->dep, v->ctab, v->wtab, v->tail, v->b2, diag};
}

template <class ET>
uint32_t prod_lds(const qsd_ham *h, int V) {
    return lds_bytes<ET>(h->prod, V);
}

// As many vectors per workgroup as there are and fit its LDS: they share the lists and the
// coefficients (one vector always fits: prod_build).
template <class ET>
int prod_width(const qsd_ham *h, int nvec) {
    int V = nvec >= 3 ? 4 : nvec == 2 ? 2 : 1;
    while (V > 1 && lds_bytes<ET>(h->prod, V) > kLdsBytes) V >>= 1;
    return V;
}

uint32_t prod_blocks(const qsd_ham *h, int nvec, int V) {
    return tiles_of(h->prod) * h->prod->nb * (uint32_t)((nvec + V - 1) / V);
}

template <class ET>
void prod_matvec(const qsd_ham *h, const void *x, int64_t ldx, void *y, int64_t ldy, int nvec, hipStream_t st) {
    const int V = prod_width<ET>(h, nvec);
    const uint32_t lds = prod_lds<ET>(h, V);
    const ProdView<ET> p = prod_view<ET>(h);
    const ET *xe = (const ET *)x;
    ET *ye = (ET *)y;
    const unsigned tiles = tiles_of(h->prod), T = h->prod->T;
    const dim3 grid(tiles * p.nb, (unsigned)((nvec + V - 1) / V));
    if (V == 4)
        k_prod_matvec<ET, 4><<<grid, T, lds, st>>>(p, xe, ldx, ye, ldy, nvec);
    else if (V == 2)
        k_prod_matvec<ET, 2><<<grid, T, lds, st>>>(p, xe, ldx, ye, ldy, nvec);
    else
        k_prod_matvec<ET, 1><<<grid, T, lds, st>>>(p, xe, ldx, ye, ldy, nvec);
}

template <class ET>
void prod_matvec_batched(const ProdReq<ET> *d_reqs, int n, uint32_t blocks, uint32_t T, int V, uint32_t lds,
                         hipStream_t st) {
    const dim3 grid = folded_grid(blocks, (int)T);
    if (V == 4)
        k_prod_batched<ET, 4><<<grid, T, lds, st>>>(d_reqs, n, blocks);
    else if (V == 2)
        k_prod_batched<ET, 2><<<grid, T, lds, st>>>(d_reqs, n, blocks);
    else
        k_prod_batched<ET, 1><<<grid, T, lds, st>>>(d_reqs, n, blocks);
}

#define QSD_PROD_FOR(ET)                                                                                     \
    template ProdView<ET> prod_view<ET>(const qsd_ham *);                                                    \
    template uint32_t prod_lds<ET>(const qsd_ham *, int);                                                    \
    template int prod_width<ET>(const qsd_ham *, int);                                                       \
    template void prod_matvec<ET>(const qsd_ham *, const void *, int64_t, void *, int64_t, int, hipStream_t); \
    template void prod_matvec_batched<ET>(const ProdReq<ET> *, int, uint32_t, uint32_t, int, uint32_t, hipStream_t);
QSD_PROD_FOR(double)
QSD_PROD_FOR(float)
#undef QSD_PROD_FOR

}  // namespace qsd
