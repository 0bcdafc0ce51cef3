// CSR assembly of a factored operator (product.h): the columns of a row come out of the per-part
// lists in ascending order, so the two passes need no scratch for unsorted entries and no sort.
//
// Rows (a, b) have the blocks b' of their high part's list, ascending, with the row's own block among
// them; a block holds the columns a' of the low part's list (class AB), the column a (class B), or,
// the own block, the class A columns and the diagonal.  The lists are put in column order once
// per build; the stored entries and their values are those of the row engine's build.
#include <type_traits>

#include "common.h"
#include "device.h"
#include "matvec.h"
#include "product.h"

namespace qsd {
namespace {

// The lists in column order.  Low parts, [na][k]: class A columns with their sums, and class AB
// columns with their keys.  High parts, [nb][k]: blocks, the own one among them.
template <class ET>
struct Sorted {
    uint32_t *a = nullptr;    // column | (2 key + sign + 1) << 16 (0 there: nothing follows the sum)
    ET *av = nullptr;         // the sum
    uint32_t *ab = nullptr;   // column | (2 key + sign) << 16
    uint32_t *pos = nullptr;  // [na][2] class A and AB columns below the part itself
    uint3 *b = nullptr;       // block << 16 | AB position + 1 (0: none); kBNone, kBOwn, or kB1 / kB2 |
                              // position; AB columns' blocks and B entries of the blocks before
    uint32_t *nblk = nullptr; // [nb]
    uint32_t nA = 0, nB = 0;  // longest class A list and block list
};
constexpr uint32_t kBPos = (1u << 14) - 1u, kB1 = 1u << 14, kB2 = 2u << 14, kBNone = 0u, kBOwn = 3u << 14;
constexpr uint32_t kMaxBlocks = 4096;  // of a high part (12 bytes each in LDS)

// One wave per low part; an entry's place is the number of entries before it (the columns within a
// list are distinct).
template <class ET>
__global__ __launch_bounds__(256) void k_prod_sort_low(ProdView<ET> p, uint32_t nAB, Sorted<ET> s) {
    const uint32_t a = blockIdx.x * 4u + (threadIdx.x >> 6), lane = threadIdx.x & 63u;
    if (a >= p.na) return;
    const uint32_t at = p.place[a];
    const uint32_t n1 = p.alen[at], n = n1 + p.alen[p.na + at], n3 = p.alen[2 * (int64_t)p.na + at];
    auto col_a = [&](uint32_t k) {
        return k < n1 ? p.a1_ent[(int64_t)k * p.na + at] & 0xFFFFu : (uint32_t)p.a2_col[prod_at(k - n1, p.na, at)];
    };
    uint32_t below_a = 0, below_ab = 0;
    for (uint32_t k = lane; k < n; k += 64u) {
        const uint32_t c = col_a(k);
        uint32_t rank = 0;
        for (uint32_t q = 0; q < n; ++q) rank += col_a(q) < c;
        const int64_t o = (int64_t)a * s.nA + rank;
        s.a[o] = c | (k < n1 ? (p.a1_ent[(int64_t)k * p.na + at] >> 16) + 1u : 0u) << 16;
        s.av[o] = k < n1 ? p.a1[(int64_t)k * p.na + at] : p.a2[prod_at(k - n1, p.na, at)];
        below_a += c < a;
    }
    for (uint32_t k = lane; k < n3; k += 64u) {
        const uint32_t e = p.ab_ent[prod_at(k, p.na, at)];
        uint32_t rank = 0;
        for (uint32_t q = 0; q < n3; ++q) rank += (p.ab_ent[prod_at(q, p.na, at)] & 0xFFFFu) < (e & 0xFFFFu);
        s.ab[(int64_t)a * nAB + rank] = e;
        below_ab += (e & 0xFFFFu) < a;
    }
    for (int d = 32; d >= 1; d >>= 1) {
        below_a += __shfl_xor(below_a, d, 64);
        below_ab += __shfl_xor(below_ab, d, 64);
    }
    if (lane == 0) {
        s.pos[2 * a] = below_a;
        s.pos[2 * a + 1] = below_ab;
    }
}

// One workgroup per high part: its AB blocks, its B blocks (some are AB blocks too) and the own one.
template <class ET>
__global__ __launch_bounds__(256) void k_prod_sort_high(ProdView<ET> p, Sorted<ET> s) {
    extern __shared__ uint32_t bp[];  // block of every entry; bit 31: an AB entry has it too
    const uint32_t b = blockIdx.x;
    const uint32_t n1 = p.blen[b], n2 = p.blen[p.nb + b], n3 = p.blen[2 * (int64_t)p.nb + b], n = n3 + n1 + n2 + 1u;
    for (uint32_t k = threadIdx.x; k < n; k += 256u) {
        uint32_t c;
        if (k < n3) c = p.bab_ent[2 * ((int64_t)b * p.nBAB + k)];
        else if (k < n3 + n1) c = p.b1_ent[2 * ((int64_t)b * p.nB1 + (k - n3))];
        else if (k < n - 1u) c = p.b2_col[(int64_t)b * p.nB2 + (k - n3 - n1)];
        else c = b;
        bp[k] = c;
    }
    __syncthreads();
    for (uint32_t k = n3 + threadIdx.x; k < n - 1u; k += 256u) {
        bool dup = false;
        for (uint32_t q = 0; q < n3; ++q) dup |= (bp[q] & 0xFFFFu) == bp[k];
        if (dup) bp[k] |= 1u << 31;
    }
    __syncthreads();
    uint32_t blocks = 0;
    for (uint32_t k = threadIdx.x; k < n; k += 256u) {
        const uint32_t c = bp[k] & 0xFFFFu;
        const bool dup = (bp[k] >> 31) != 0u;
        uint32_t rank = 0, cab = 0, cb = 0, own = 0, partner = kBNone;
        for (uint32_t q = 0; q < n; ++q) {
            const uint32_t cq = bp[q] & 0xFFFFu;
            const bool less = cq < c;
            rank += less && !(bp[q] >> 31);
            if (q < n3) cab += less;
            else if (q < n - 1u) {
                cb += less;
                if (k < n3 && cq == c) partner = q < n3 + n1 ? kB1 | (q - n3) : kB2 | (q - n3 - n1);
            } else own = less;
        }
        blocks += !dup;
        if (dup) continue;  // its AB entry writes the block
        uint3 w;
        w.x = c << 16 | (k < n3 ? k + 1u : 0u);
        w.y = k < n3 ? partner : k < n3 + n1 ? kB1 | (k - n3) : k < n - 1u ? kB2 | (k - n3 - n1) : kBOwn;
        w.z = cab | cb << 14 | own << 31;
        s.b[(int64_t)b * s.nB + rank] = w;
    }
    __shared__ uint32_t total;
    if (threadIdx.x == 0) total = 0u;
    __syncthreads();
    if (blocks) atomicAdd(&total, blocks);
    __syncthreads();
    if (threadIdx.x == 0) s.nblk[b] = total;
}

// Stored entries per row: of an AB block those pairs of keys that have a term.
template <class ET>
__global__ __launch_bounds__(256) void k_prod_csr_count(ProdView<ET> p, int64_t *__restrict__ counts) {
    const uint32_t tiles = (p.na + 255u) / 256u;
    const uint32_t b = blockIdx.x / tiles, a = (blockIdx.x - b * tiles) * 256u + threadIdx.x;
    if (a >= p.na) return;
    const uint32_t at = p.place[a], n3 = p.alen[2 * (int64_t)p.na + at], nab = p.blen[2 * (int64_t)p.nb + b];
    int64_t n = 1 + (int64_t)p.alen[at] + p.alen[p.na + at] + p.blen[b] + p.blen[p.nb + b];
    if (p.full) {
        n += (int64_t)n3 * nab;
    } else {
        for (uint32_t e = 0; e < nab; ++e) {
            const uint32_t w = p.bab_ent[2 * ((int64_t)b * p.nBAB + e) + 1];
            const ET *ct = p.ctab + (int64_t)(w >> 1) * p.nU;
            for (uint32_t k = 0; k < n3; ++k) n += ct[p.ab_ent[prod_at(k, p.na, at)] >> 17] != (ET)0;
        }
    }
    counts[(int64_t)b * p.na + a] = n;
}

// What a row's entries are made of.  `dep` and `tail` are the class A table (a row per high qubit) and
// the block's class B tails; staged, their copies in LDS, the table's rows only those that the high
// part has set.
template <class ET, bool STAGED>
struct Row {
    const ProdView<ET> &p;
    const Sorted<ET> &s;
    uint32_t nAB, a, b, occ;
    int64_t row;
    const ET *dep, *tail;

    __device__ __forceinline__ ET class_a(uint32_t k, uint32_t &col) const {
        const int64_t o = (int64_t)a * s.nA + k;
        const uint32_t e = s.a[o];
        ET v = s.av[o];
        col = e & 0xFFFFu;
        if (e >> 16) {
            const uint32_t f = (e >> 16) - 1u;
            uint32_t r = 0;
            for (uint32_t m = occ; m; m &= m - 1u, ++r) {
                const ET c = dep[(STAGED ? r : (uint32_t)__builtin_ctz(m)) * p.nUa + (f >> 1)];
                v += (f & 1u) ? -c : c;
            }
        }
        return v;
    }
    __device__ __forceinline__ ET class_b(uint32_t code) const {  // a block's column a
        const uint32_t k = code & kBPos;
        if ((code & ~kBPos) == kB2) return p.b2[(int64_t)b * p.nB2 + k];
        const int64_t at = (int64_t)b * p.nB1 + k;
        const uint32_t e = p.b1_ent[2 * at + 1];
        const ET w = p.wtab[(int64_t)((e & 0xFFFFFFu) >> 1) * p.na + a];
        ET v = (e & 1u) ? -w : w;
        for (uint32_t t = 0; t < e >> 24; ++t) v += tail[k * p.tail_len + t];
        return v;
    }
    __device__ __forceinline__ ET class_ab(uint32_t ab, uint32_t k, uint32_t &col) const {
        const uint32_t w = p.bab_ent[2 * ((int64_t)b * p.nBAB + ab) + 1];
        const uint32_t e = s.ab[(int64_t)a * nAB + k];
        const ET c = p.ctab[(int64_t)(w >> 1) * p.nU + (e >> 17)];
        col = e & 0xFFFFu;
        return ((w ^ (e >> 16)) & 1u) ? -c : c;
    }
};

// Operators whose pairs of keys all have a term: a block's first entry has a closed form, so a wave
// writes a row's entries 64 at a time, each lane finding its entry's block by bisection of the
// block list (in LDS, uniform over the workgroup's rows).  A lane per row instead, walking its
// entries, wrote 64 lines an instruction: 315 us for 8.9M entries (301 x 301) and 2250 us for 80M.
// A wave has entries of every class in nearly every instruction, and the sums over the high part's
// set qubits and over the tails are chains of reads: from LDS, not from L2 (whole builds of 301 x 301
// 250 -> 202 us, of 600 x 600 892 -> 735).  Rows per workgroup, which share the tables: 8 204 and
// 800 us, 16 202 and 734, 32 211 and 745, 64 213 and 785.
constexpr uint32_t kFillRows = 16;

template <class ET>
size_t fill_lds(const qsd_prod *p, uint32_t nB) {
    return (nB * sizeof(uint3) + 15u) / 16u * 16u + ((size_t)p->max_occ * p->nUa + (size_t)p->nB1 * p->tail_len) * sizeof(ET);
}

template <class ET, class IT>
__global__ __launch_bounds__(256) void k_prod_csr_fill(ProdView<ET> p, Sorted<ET> s, uint32_t nAB,
                                                       const int64_t *__restrict__ indptr, IT *__restrict__ idx,
                                                       ET *__restrict__ val) {
    extern __shared__ __align__(16) char fill_smem[];
    uint32_t *bz = (uint32_t *)fill_smem, *bx = bz + s.nB, *by = bx + s.nB;  // the block list, by component
    ET *tail = (ET *)(fill_smem + (s.nB * sizeof(uint3) + 15u) / 16u * 16u), *dep = tail + p.nB1 * p.tail_len;
    const uint32_t tiles = (p.na + kFillRows - 1u) / kFillRows;
    const uint32_t block = blockIdx.y * gridDim.x + blockIdx.x;
    const uint32_t b = block / tiles, a0 = (block - b * tiles) * kFillRows, lane = threadIdx.x & 63u;
    if (b >= p.nb) return;
    const uint32_t nblk = s.nblk[b];
    for (uint32_t k = threadIdx.x; k < nblk; k += 256u) {
        const uint3 w = s.b[(int64_t)b * s.nB + k];
        bx[k] = w.x;
        by[k] = w.y;
        bz[k] = w.z;
    }
    const uint32_t ntail = p.blen[b] * p.tail_len, occ = p.blen[3 * (int64_t)p.nb + b] & p.rmask;
    for (uint32_t k = threadIdx.x; k < ntail; k += 256u) tail[k] = p.tail[(int64_t)b * p.nB1 * p.tail_len + k];
    uint32_t q = 0;
    for (uint32_t m = occ; m; m &= m - 1u, ++q)
        for (uint32_t u = threadIdx.x; u < p.nUa; u += 256u) dep[q * p.nUa + u] = p.dep[__builtin_ctz(m) * p.nUa + u];
    __syncthreads();
    for (uint32_t a = a0 + (threadIdx.x >> 6); a < min(a0 + kFillRows, p.na); a += 4u) {
        const Row<ET, true> R{p, s, nAB, a, b, occ, (int64_t)b * p.na + a, dep, tail};
        const uint32_t at = p.place[a];
        const uint32_t n3 = p.alen[2 * (int64_t)p.na + at], nown = p.alen[at] + p.alen[p.na + at] + 1u;
        const uint32_t pos_a = s.pos[2 * a], pos_ab = s.pos[2 * a + 1];
        const int64_t o = indptr[R.row];
        const uint32_t len = (uint32_t)(indptr[R.row + 1] - o);
        auto first = [&](uint32_t i) {  // entries before block i
            const uint32_t z = bz[i];
            return (z & kBPos) * n3 + ((z >> 14) & kBPos) + ((z >> 31) ? nown : 0u);
        };
        for (uint32_t e = lane; e < len; e += 64u) {
            uint32_t lo = 0, hi = nblk - 1u;  // the last block whose first entry is at most e
            while (lo < hi) {
                const uint32_t mid = (lo + hi + 1u) >> 1;
                if (first(mid) <= e)
                    lo = mid;
                else
                    hi = mid - 1u;
            }
            uint32_t m = e - first(lo), col = a;
            const uint2 w = {bx[lo], by[lo]};
            ET v;
            if (w.y == kBOwn) {
                if (m == pos_a)
                    v = p.diag[R.row];
                else
                    v = R.class_a(m - (m > pos_a), col);
            } else if ((w.x & 0xFFFFu) && !(w.y != kBNone && m == pos_ab)) {
                v = R.class_ab((w.x & 0xFFFFu) - 1u, m - (w.y != kBNone && m > pos_ab), col);
            } else {
                v = R.class_b(w.y);
            }
            idx[o + e] = (IT)((int64_t)(w.x >> 16) * p.na + col);
            val[o + e] = v;
        }
    }
}

// Operators with pairs of keys that have no term (or with tables that LDS cannot hold): a lane per row
// walks its blocks.
template <class ET, class IT>
__global__ __launch_bounds__(256) void k_prod_csr_walk(ProdView<ET> p, Sorted<ET> s, uint32_t nAB,
                                                       const int64_t *__restrict__ indptr, IT *__restrict__ idx,
                                                       ET *__restrict__ val) {
    const uint32_t tiles = (p.na + 255u) / 256u;
    const uint32_t b = blockIdx.x / tiles, a = (blockIdx.x - b * tiles) * 256u + threadIdx.x;
    if (a >= p.na) return;
    const Row<ET, false> R{p, s, nAB, a, b, p.blen[3 * (int64_t)p.nb + b] & p.rmask, (int64_t)b * p.na + a, p.dep,
                           p.tail + (int64_t)b * p.nB1 * p.tail_len};
    const uint32_t at = p.place[a], n3 = p.alen[2 * (int64_t)p.na + at], nA = p.alen[at] + p.alen[p.na + at];
    int64_t o = indptr[R.row];
    auto put = [&](int64_t col, ET v) {
        idx[o] = (IT)col;
        val[o] = v;
        ++o;
    };
    const uint32_t pos_a = s.pos[2 * a], pos_ab = s.pos[2 * a + 1];
    for (uint32_t i = 0; i < s.nblk[b]; ++i) {
        const uint3 w = s.b[(int64_t)b * s.nB + i];
        const int64_t c0 = (int64_t)(w.x >> 16) * p.na;
        uint32_t col;
        if (w.y == kBOwn) {
            for (uint32_t k = 0; k <= nA; ++k) {
                if (k == pos_a) put(R.row, p.diag[R.row]);
                if (k == nA) break;
                const ET v = R.class_a(k, col);
                put(c0 + col, v);
            }
            continue;
        }
        const uint32_t n = (w.x & 0xFFFFu) ? n3 : 0u, mid = (w.x & 0xFFFFu) ? pos_ab : 0u;
        for (uint32_t k = 0; k <= n; ++k) {
            if (w.y != kBNone && k == mid) put(c0 + a, R.class_b(w.y));
            if (k == n) break;
            const ET v = R.class_ab((w.x & 0xFFFFu) - 1u, k, col);
            if (v != (ET)0) put(c0 + col, v);
        }
    }
}

}  // namespace

bool prod_csr_usable(const qsd_ham *h) {
    return prod_usable(h) && (uint64_t)h->prod->nB1 + h->prod->nB2 + h->prod->nBAB + 1u <= kMaxBlocks;
}

void prod_csr_count(const qsd_ham *h, int64_t *counts, hipStream_t st) {
    k_prod_csr_count<double><<<(h->prod->na + 255u) / 256u * h->prod->nb, 256, 0, st>>>(prod_view<double>(h), counts);
}

template <class ET, class IT>
int prod_csr_fill(const qsd_ham *h, const int64_t *indptr, void *indices, void *data, hipStream_t st) {
    const qsd_prod *p = h->prod;
    Sorted<ET> s;
    s.nA = p->nA1 + p->nA2;
    s.nB = p->nB1 + p->nB2 + p->nBAB + 1u;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t o1 = take((size_t)s.nA * p->na * 4), o2 = take((size_t)s.nA * p->na * sizeof(ET));
    const size_t o3 = take((size_t)p->nAB * p->na * 4), o4 = take(8 * (size_t)p->na);
    const size_t o5 = take((size_t)s.nB * p->nb * sizeof(uint3)), o6 = take(4 * (size_t)p->nb);
    uint8_t *mem = nullptr;
    QSD_TRY(dev_alloc(&mem, off));
    s.a = (uint32_t *)(mem + o1);
    s.av = (ET *)(mem + o2);
    s.ab = (uint32_t *)(mem + o3);
    s.pos = (uint32_t *)(mem + o4);
    s.b = (uint3 *)(mem + o5);
    s.nblk = (uint32_t *)(mem + o6);
    const ProdView<ET> v = prod_view<ET>(h);
    k_prod_sort_low<ET><<<(p->na + 3u) / 4u, 256, 0, st>>>(v, p->nAB, s);
    k_prod_sort_high<ET><<<p->nb, 256, s.nB * 4u, st>>>(v, s);
    const size_t lds = fill_lds<ET>(p, s.nB);
    if (p->full && lds <= 64u * 1024u)
        k_prod_csr_fill<ET, IT><<<folded_grid((int64_t)((p->na + kFillRows - 1u) / kFillRows) * p->nb, 256), 256, lds, st>>>(
            v, s, p->nAB, indptr, (IT *)indices, (ET *)data);
    else
        k_prod_csr_walk<ET, IT><<<(p->na + 255u) / 256u * p->nb, 256, 0, st>>>(v, s, p->nAB, indptr, (IT *)indices, (ET *)data);
    const bool ok = hipGetLastError() == hipSuccess;
    dev_free(mem);
    return ok ? QSD_OK : fail(QSD_ERR_HIP, "CSR fill launch failed");
}

template int prod_csr_fill<double, int32_t>(const qsd_ham *, const int64_t *, void *, void *, hipStream_t);
template int prod_csr_fill<double, int64_t>(const qsd_ham *, const int64_t *, void *, void *, hipStream_t);
template int prod_csr_fill<float, int32_t>(const qsd_ham *, const int64_t *, void *, void *, hipStream_t);
template int prod_csr_fill<float, int64_t>(const qsd_ham *, const int64_t *, void *, void *, hipStream_t);

}  // namespace qsd
