// Shared by the two forms of the coarse search.
#pragma once
#include "scan_device.h"

#define CS_MAX_NPROBE 1024

__device__ inline void cs_rank_and_write(const uint64_t *A, int na, int k, int nprobe, int32_t *oid,
                                         float *osc) {
    for (int i = threadIdx.x; i < na; i += blockDim.x) {
        const uint64_t mine = A[i];
        int r = 0;
        for (int j = 0; j < na; ++j) r += A[j] < mine ? 1 : 0;
        if (r < k) {
            oid[r] = (int32_t)(uint32_t)mine;
            if (osc) osc[r] = qadc_ord2f((uint32_t)(mine >> 32));
        }
    }
    for (int r = k + threadIdx.x; r < nprobe; r += blockDim.x) {
        oid[r] = -1;
        if (osc) osc[r] = INFINITY;
    }
}

static inline size_t cs_up256(size_t x) { return (x + 255) & ~(size_t)255; }

// The half-precision form (coarse_half.hip) of a call, if it takes it.  Offsets in bytes from the score
// matrix on.
struct CoarseHalf {
    bool use;
    int S;       // product steps of 16 columns: d and three pieces of the norm
    int P;       // cells of the pilot
    int ntiles;  // tiles of 32 cells
    int nslots;  // candidate lists per query
    size_t minima, qs, err, bounds, ent, ids, counts;  // of a pass
    size_t cells, bmax, bnorm, flag;                   // of the call
    size_t total;
};
// The plan of a call of nq queries in passes of qc, with a score matrix of matrix_bytes and room for
// `room` bytes from it on (less than the plan's total: not used).
CoarseHalf qadc_coarse_half_plan(int nq, int qc, int K, int d, int nprobe, size_t matrix_bytes, size_t room);
// the largest such total over all d and nprobe (0 if no call of nq queries takes the form)
size_t qadc_coarse_half_bytes(int nq, int qc, int K, size_t matrix_bytes);
// norms (always) and, with hp.use, the cells' operand; base = the score matrix
int qadc_coarse_cells(const float *centroids, int K, int d, const CoarseHalf &hp, float *cnorm, char *base, hipStream_t s);
// one pass: results of nqc <= qc queries; the flag (cleared here) is raised when the exact form must take
// the pass instead
int qadc_coarse_half_pass(const float *queries, int nqc, const float *centroids, int K, int d, int nprobe,
                          const CoarseHalf &hp, const float *cnorm, char *base, int32_t *probe_ids,
                          float *probe_scores, hipStream_t s);
// Exact scores [nq][ld] of at most QADC_DIRECT_NQ queries, and the smallest of every 64 cells
// [nq][ld].  (Calls of up to 16 queries: 65,536 cells, d = 96: 1 query 75 -> 14 us, 16 queries 78 -> 25.
// 32 queries, with the selection over whole rows, against the batched form: 1024 cells 44 / 36 us,
// 65,536 cells 76 / 68, but 16,384 cells 49 / 65; their chains are what bounds a block then.)
#define QADC_DIRECT_NQ 16
int qadc_coarse_direct(const float *queries, int nq, const float *centroids, int K, int d, float *scores, size_t ld,
                       float *minima, hipStream_t s);
