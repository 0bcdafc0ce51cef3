// Factored form of an operator on an alpha x beta product subspace (Results, fermionic examples).
//
// A row is a pair (a, b) of a low and a high part.  A group flips the low part only (class A), both
// (class AB) or the high part only (class B), and for the operators of the fermionic workloads a
// matrix element needs little more than what each part knows by itself: whether the flipped part
// was sampled, its rank, the projector bits that select a term and the sign of that part's Z string.
// These facts are worked out once per part (1500 + 1500 strings on the 2.25M-row workload) and kept
// as lists; the SpMV combines the two lists of a row instead of testing its 18 280 groups.
//
//   A   per low part, in group order: column rank and the sum of the group's matching terms; in
//       segment 1 the sum continues with terms that want one high qubit set (the spectators'
//       number operators), kept as a table by (high qubit, term key)
//   AB  per low part and per high part, in flip order: rank and term key with its sign; the
//       element is the coefficient of the pair of keys
//   B   per high part, in group order: rank and the element; in segment 1 it starts from a table by
//       (term key, low part) and continues with the row's remaining terms
//
// Every element is the same sum of the same terms in the same order as in the table kernels, and a
// row takes its elements in the same order, so the results are bitwise the same.
#pragma once

#include "common.h"

namespace qsd {

// Device arrays of the plan; `f` = FP32 copies (sums formed in FP32, as the FP32 path does).
template <class ET>
struct ProdVals {
    ET *a1 = nullptr;    // [nA1][na] sums of the terms that depend on the low part alone
    ET *a2 = nullptr;    // [nA2 / 4][na][4]
    ET *dep = nullptr;   // [high qubits][nUa] coefficients of the class A terms that want a high qubit
    ET *ctab = nullptr;  // [nW][nU] class AB coefficients (0: no such term)
    ET *wtab = nullptr;  // [nWb][na] class B sums up to the terms that want a low qubit
    ET *tail = nullptr;  // [nb][nB1][tail_len] signed coefficients added after them
    ET *b2 = nullptr;    // [nb][nB2]
};

}  // namespace qsd

struct qsd_prod {
    int32_t split = 0;
    uint32_t na = 0, nb = 0;
    uint32_t T = 0;         // low parts per workgroup (a tile)
    // longest list over the parts, per segment
    uint32_t nA1 = 0, nA2 = 0, nAB = 0, nB1 = 0, nB2 = 0, nBAB = 0;
    uint32_t nUa = 0, nU = 0, nW = 0, nWb = 0, tail_len = 0;
    uint32_t rmask = 0;     // high qubits (shifted to 0) that class A terms want
    uint32_t max_occ = 0;   // most of them set in one sampled high part
    bool full = false;      // every pair of class AB keys has a term
    // lists: low parts by position (order[position] = rank, place[rank] = position; within a tile by
    // the length of the AB list), A1 [k][na], A2 and AB four entries together (prod_at), padded with
    // entries that add nothing; high parts [nb][k]
    uint32_t *order = nullptr, *place = nullptr;
    uint32_t *a1_ent = nullptr;  // column rank | (2 key + sign) << 16
    uint16_t *a2_col = nullptr;  // column rank
    uint32_t *ab_ent = nullptr;  // column rank | (2 key + sign) << 16
    uint32_t *b1_ent = nullptr;  // [nb][nB1][2] row-block rank, 2 key + sign | tail count << 24
    uint32_t *b2_col = nullptr;  // row-block rank
    uint32_t *bab_ent = nullptr; // [nb][nBAB][2] row-block rank, 2 key + sign
    uint32_t *alen = nullptr;    // [3][na] lengths A1, A2, AB, by position
    uint32_t *blen = nullptr;    // [4][nb] lengths B1, B2, AB, and the high part itself
    qsd::ProdVals<double> d;
    qsd::ProdVals<float> f;
    uint8_t *mem[2] = {nullptr, nullptr};  // the two allocations that all of these lie in
};

namespace qsd {

// Place of entry k of the low part at position `at` in the A2 and AB lists.
__host__ __device__ inline int64_t prod_at(uint32_t k, uint32_t na, uint32_t at) {
    return ((int64_t)(k >> 2) * na + at) * 4 + (k & 3u);
}

// What the SpMV kernels read of a plan, by value (or in a request table).
template <class ET>
struct ProdView {
    uint32_t na, nb, T, aux, nB1, nB2, nBAB, nUa, nU, tail_len, rmask, full;
    const uint32_t *__restrict__ a1_ent;
    const uint16_t *__restrict__ a2_col;
    const uint32_t *__restrict__ ab_ent;
    const uint32_t *__restrict__ b1_ent, *__restrict__ b2_col, *__restrict__ bab_ent;
    const uint32_t *__restrict__ alen, *__restrict__ blen, *__restrict__ order, *__restrict__ place;
    const ET *__restrict__ a1, *__restrict__ a2, *__restrict__ dep, *__restrict__ ctab, *__restrict__ wtab,
        *__restrict__ tail, *__restrict__ b2;
    const ET *__restrict__ diag;
};

// One request of a batched launch; its workgroups are [first, the next request's first).
template <class ET>
struct ProdReq {
    ProdView<ET> p;
    const ET *x;
    ET *y;
    int64_t ld;
    int32_t nv;
    uint32_t first;
    const int *kdev;  // batched Lanczos: the request idles once *kdev >= m (NULL: never)
    int32_t m;
};

// Builds h->prod when the subspace has a product map and the operator factors as above (the group
// order keeps the classes apart); leaves it NULL otherwise.  The operator's tables must have been
// uploaded (`tables` bytes).  Waits once for the list lengths; the lists themselves are enqueued.
int prod_build(qsd_ham *h, size_t tables, hipStream_t st);
void prod_free(qsd_prod *&p);

// Whether the SpMV of `h` runs from the plan.
bool prod_usable(const qsd_ham *h);

template <class ET>
ProdView<ET> prod_view(const qsd_ham *h);

// Vectors that one workgroup takes when a launch's widest request has nvec of them, and the LDS
// bytes and workgroups a request needs then.
template <class ET>
int prod_width(const qsd_ham *h, int nvec);
template <class ET>
uint32_t prod_lds(const qsd_ham *h, int V);
uint32_t prod_blocks(const qsd_ham *h, int nvec, int V);

// Y = H X from the plan (real operators); nvec interleaved vectors.
template <class ET>
void prod_matvec(const qsd_ham *h, const void *x, int64_t ldx, void *y, int64_t ldy, int nvec, hipStream_t st);

// The same for n requests of a device table in one launch of workgroups of T threads (the largest
// of the requests'); every row is evaluated as above.
template <class ET>
void prod_matvec_batched(const ProdReq<ET> *d_reqs, int n, uint32_t blocks, uint32_t T, int V, uint32_t lds,
                         hipStream_t st);

// CSR assembly (product_csr.hip): entries per row, and the rows' entries in column order.
bool prod_csr_usable(const qsd_ham *h);
void prod_csr_count(const qsd_ham *h, int64_t *counts, hipStream_t st);
template <class ET, class IT>
int prod_csr_fill(const qsd_ham *h, const int64_t *indptr, void *indices, void *data, hipStream_t st);

}  // namespace qsd
