// Sparse operators (at most one off-diagonal element per row on average, as on strings sampled far
// apart): the rows that have elements, with each element's column and term range, found once.  The
// SpMV then evaluates the elements' terms and touches no group, hash slot or key of the other rows.
#pragma once

#include "common.h"

// One off-diagonal element: its column and the terms [t0, t0 + len) of its group that the row's
// ladder integer selects (the row's projector bits and signs are applied when it is evaluated).
struct qsd_hit {
    uint32_t col, t0, len, unused;
};

struct qsd_hits {
    int64_t M = 0, H = 0, L = 0;  // rows with elements, elements, rows with many
    uint64_t *rowbits = nullptr;  // [ceil(N / 64)] bit r = row r has elements
    uint32_t *rows = nullptr;     // [M] ascending
    uint32_t *ptr = nullptr;      // [M + 1] first element of each listed row
    uint32_t *lng = nullptr;      // [L] positions in `rows` of the rows with many elements, any order
    qsd_hit *rec = nullptr;       // [H] in group order within a row
    uint8_t *mem = nullptr;       // rows, ptr, lng and rec lie in it
};

namespace qsd {

// Builds the list when the operator has at most N off-diagonal elements (a sample of the rows is
// counted first) and the list fits the memory; *out stays NULL otherwise.  Device memory from the
// current allocator scope.  Synchronizes.
int hits_build(const qsd_ham *h, qsd_hits **out, hipStream_t st);
void hits_free(qsd_hits *&p);

// Y = H X from the list; nvec (1..16) interleaved vectors of `dtype` (matching the operator).
int hits_matvec(const qsd_ham *h, const qsd_hits *p, int nvec, const void *x, int64_t ldx, void *y, int64_t ldy,
                int32_t dtype, hipStream_t st);

}  // namespace qsd
