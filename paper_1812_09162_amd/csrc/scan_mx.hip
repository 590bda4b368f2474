// Batched matrix-core scan: when a call takes it, and its dispatch by layout.
#include "scan_mx.h"

// (the irregular 64- and 128-bit kinds are instantiated in a file of their own: compile time)
#define MX_ARGS const pq_index *, const pq_qparams_t *, int, const uint8_t *, int64_t, int, int32_t *, uint16_t *, float *, \
                char *, const ScanPlan &, const MxPlan &, hipStream_t
extern template int mx_launch<SCAN_W64, uint8_t>(MX_ARGS);
extern template int mx_launch<SCAN_W64, uint16_t>(MX_ARGS);
extern template int mx_launch<SCAN_W128, uint8_t>(MX_ARGS);
extern template int mx_launch<SCAN_W128, uint16_t>(MX_ARGS);

// Queries from which the matrix cores win: up to four share one pass of k_scan_mq / k_scan_mqg (16 x 4
// bits, 10^7 codes: 61 us against 57 here; {6,6,4} x 8, 5 * 10^6 codes: 129 against 186), the fifth costs
// those a second pass (87 against 58; 209 against 187), while 32 queries are one product here.
#define MX_MIN_NQ 5
// ... and sizes: the launches and the picking take some 28 us whatever the size, look-ups a time in
// proportion to the codes of all their passes (of four queries).  m x 4 bits: 400,000 codes, 8 queries,
// R = 100: 38.8 us there, 33.6 here; 200,000: 30.5 and 33.2; 100,000 codes, 64 queries: 49.7 and 43.0.
// Irregular layouts, where a code is dearer to score again: 400,000 codes, 64 queries: 156 and 164;
// 10^6: 186 and 87.  With few codes per result too many groups hold one: {6,6,4} x 4, 10^6 codes, R = 400,
// 64 queries: 233 and 487; 16 x 4 bits, 400,000 codes: 99 and 63.
#define MX_MIN_CODES_NIB 800000
#define MX_MIN_CODES 6000000
#define MX_MIN_RATIO_NIB 1000
#define MX_MIN_RATIO 8000

MxPlan qadc_mx_plan(const pq_index *idx, int nq, int64_t n, int R, const ScanPlan &sp) {
    MxPlan p;
    memset(&p, 0, sizeof(p));
    const DevLayout &h = idx->h;
    if (h.mx_steps == 0 || nq < MX_MIN_NQ || qadc_option(PQ_OPT_SHARED_PASSES) == 0) return p;
    const bool nib = h.kind == SCAN_NIB8 || h.kind == SCAN_NIB16;
    if (n * ((nq + 3) / 4) < (nib ? MX_MIN_CODES_NIB : MX_MIN_CODES) || n < (int64_t)(nib ? MX_MIN_RATIO_NIB : MX_MIN_RATIO) * R)
        return p;
    // A few results of irregular layouts: the calibration ends the range of the keys close to the R-th, the
    // levels are coarse there, and where distances are alike most groups hold a code within them (40-bit
    // codes, 2.5 * 10^6, R = 10, 64 queries: 151 us as look-ups, 432 here; R = 100: 165 and 78).  For the
    // single best code the look-up kernels have no bound below the top of the range either (R = 1: 22 ms
    // and 10; {6,6,4} x 4: 24 ms and 0.12).
    if (!nib && R > 1 && R < 32) return p;
    const int tiles = (nq + 31) / 32;  // of 32 queries
    const int most = mx_most(h.kind, h.mx_pat != 0);
    p.groups = (tiles + most - 1) / most;
    p.ncol = (tiles + p.groups - 1) / p.groups;
    p.btab_off = sp.cand_off;
    p.min_off = sp.cand_off + (((size_t)h.mx_steps * 48 + 255) & ~(size_t)255);
    // groups of 64 codes, or larger ones where the workspace has no room for their minima; chunks of
    // 16 groups per lane, or of 4 where that would leave too few waves
    for (p.nb = 1; p.nb <= 8; p.nb *= 2) {
        p.gpc = (n / (2048 * (int64_t)p.nb)) * p.groups >= 2048 ? 16 : 4;
        const int64_t nchunks = n / ((int64_t)p.gpc * p.nb * 128);
        const int64_t nmin = nchunks * 2 * p.gpc;
        if (nmin < 8 * (int64_t)R || nmin >= ((int64_t)1 << 24)) continue;
        if (p.min_off + (size_t)((nmin + 15) & ~(int64_t)15) > sp.per_query) continue;
        p.nchunks = (int)nchunks;
        p.nmin = (int)nmin;
        p.use = true;
        return p;
    }
    return p;
}

int qadc_scan_mx(const pq_index *idx, const pq_qparams_t *qparams, int nq, const uint8_t *codes, int64_t n, int R,
                 int32_t *out_ids, uint16_t *out_keys, float *out_dist, char *ws, const ScanPlan &sp, const MxPlan &p,
                 hipStream_t s) {
    const bool u8 = idx->h.acc_bits == 8;
#define QADC_GO(KIND)                                                                                                 \
    return u8 ? mx_launch<KIND, uint8_t>(idx, qparams, nq, codes, n, R, out_ids, out_keys, out_dist, ws, sp, p, s)    \
              : mx_launch<KIND, uint16_t>(idx, qparams, nq, codes, n, R, out_ids, out_keys, out_dist, ws, sp, p, s)
    switch (idx->h.kind) {
        case SCAN_NIB8: QADC_GO(SCAN_NIB8);
        case SCAN_NIB16: QADC_GO(SCAN_NIB16);
        case SCAN_C5: QADC_GO(SCAN_C5);
        case SCAN_W64: QADC_GO(SCAN_W64);
        default: QADC_GO(SCAN_W128);
    }
#undef QADC_GO
}
