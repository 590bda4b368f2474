// Batched matrix-core scan: when a call takes it, and its dispatch by layout.
#include "scan_mx.h"

// (the irregular 64- and 128-bit kinds are instantiated in a file of their own: compile time)
#define MX_ARGS const pq_index *, const pq_qparams_t *, int, const uint8_t *, int64_t, int, int32_t *, uint16_t *, float *, \
                char *, const ScanPlan &, const MxPlan &, hipStream_t
extern template int mx_launch<SCAN_W64, uint8_t>(MX_ARGS);
extern template int mx_launch<SCAN_W64, uint16_t>(MX_ARGS);
extern template int mx_launch<SCAN_W128, uint8_t>(MX_ARGS);
extern template int mx_launch<SCAN_W128, uint16_t>(MX_ARGS);

// When the matrix cores win.  Look-ups take a time in proportion to codes times passes (of four queries);
// here 32 queries are one product, but some 28 us go to launches and picking whatever the size, and the
// picking of a query, by one block, grows with the results and with what a code costs to score again.  The
// lines below are where, in 29,088 pairs of timings of both forms (16 layouts, 20,000 to 8 * 10^6 codes, 5
// to 256 queries, R = 1 to 2000, two kinds of data), this form stops being the slower one.  Figures in us,
// look-ups / here.
//
// Up to one pass (four queries) the look-ups: 16 x 4 bits, 10^7 codes, 4 queries: 61 / 58, 5: 87 / 58.
#define MX_MIN_NQ 5
// m x 4 bits.  Codes times passes from 800,000 on (400,000 codes, 8 queries, R = 100: 39 / 34; 200,000: 30
// and 34) and 1000 codes per result (400,000 codes, R = 500, 48 queries: 97 / 130).  Short lists with long
// batches: 100,000 codes, 32 queries, R = 10: 33 / 47, and 256 queries 87 / 67; 32 x 4 bits, twice the
// look-ups per code, from 50,000 codes on (100 queries, R = 1: 76 / 45).
#define MX_MIN_CODES_NIB 800000
#define MX_MIN_RATIO_NIB 1000
#define MX_MIN_LIST_8 200000
#define MX_MIN_LIST_16 50000
#define MX_LONG_NIB 6000000
// Irregular layouts, where a code is dearer to score again: 6 * 10^6 ({6,6,4} x 4, R = 100, 64 queries:
// 400,000 codes 153 / 148, 800,000 177 / 85) and 8000 codes per result ({6,6,4} x 4, 800,000 codes, R = 250, 64 queries: 202
// and 240).
#define MX_MIN_CODES 6000000
#define MX_MIN_RATIO 8000
// The single best code: the look-ups have no bound below the top of the range (40-bit codes, 3.2 * 10^6, 256
// queries: 28 ms / 0.25) but in a short list one query in some dozens has most of it near its best code,
// and its block all of it to score again ({6,5,5,6,5,5,4,4}, 800,000 codes, 32 queries: 0.10 ms / 2.5 ms).
#define MX_MIN_LIST_ONE 1600000

// 128-bit codes of other field patterns, R up to 100: 64 queries, 1.6 * 10^6 codes 475 / 324, 3.2 * 10^6 605 / 563;
// 100 queries 599 / 545 and 802 / 896
#define MX_MOST_128 2000000

// Passes that the look-ups must take at least.
static int mx_min_passes(const DevLayout &h, int R) {
    const bool wide = h.acc_bits != 8, w128 = h.kind == SCAN_NIB16 || h.kind == SCAN_W128;
    // m x 4 bits: R = 1000, 8 * 10^6 codes, 8 queries 124 / 126, 12 queries 170 / 126; with 16-bit tables
    // (32 x 4) 3.2 * 10^6 codes, R = 250, 8 queries 124 / 197, 16 queries 220 / 200
    if (h.kind == SCAN_NIB8) return 2 + R / (wide ? 200 : 1000);
    if (h.kind == SCAN_NIB16) return wide ? (R < 32 ? 2 : 3 + R / 100) : 2 + R / 1000;
    // field patterns known at compile time: {6,6,4} x 4, 3.2 * 10^6 codes, 5 queries, R = 100: 100 / 78, R = 500
    // 130 / 164; {6,5,5} x 8, R = 250: 200 / 314, 16 queries 397 / 319
    if (h.mx_pat != 0) {
        const int need = (w128 ? 3 : 2) + R / 200;
        return R < 100 && need < 3 ? 3 : need;
    }
    // others, one tile of queries per wave: 3.2 * 10^6 codes, R = 100, 5 queries 69 / 115, 8: 91 / 116, 16: 160 / 117
    // (128-bit codes, twice the products: see MX_MOST_128)
    return (w128 ? 8 : 4) + R / 400;
}

MxPlan qadc_mx_plan(const pq_index *idx, int nq, int64_t n, int R, const ScanPlan &sp) {
    MxPlan p;
    memset(&p, 0, sizeof(p));
    const DevLayout &h = idx->h;
    if (h.mx_steps == 0 || nq < MX_MIN_NQ || qadc_option(PQ_OPT_SHARED_PASSES) == 0) return p;
    const bool nib = h.kind == SCAN_NIB8 || h.kind == SCAN_NIB16;
    const int passes = (nq + 3) / 4;
    if (passes < mx_min_passes(h, R)) return p;
    if (nib) {
        if (n * passes < MX_MIN_CODES_NIB || n < (int64_t)MX_MIN_RATIO_NIB * R) return p;
        if (n < (h.kind == SCAN_NIB8 ? MX_MIN_LIST_8 : MX_MIN_LIST_16) && n * passes < MX_LONG_NIB) return p;
    } else {
        // A few results: the calibration ends the range of the keys close to the R-th, the levels are coarse
        // there, and where distances are alike most groups hold a code within them (40-bit codes, 2.5 * 10^6,
        // R = 10, 64 queries: 151 / 432, R = 100 165 / 78).  40-bit codes, of which more are equal, from R = 100
        // on (1.6 * 10^6 codes, R = 64, 64 queries: 150 / 395) and with twice the codes per result (3.2 * 10^6,
        // R = 500, 64 queries: 231 / 709).
        const bool c5 = h.kind == SCAN_C5, plain = h.mx_pat != 0 && h.acc_bits == 16 && !c5;
        if (n * passes < MX_MIN_CODES || n < (int64_t)(c5 ? 2 * MX_MIN_RATIO : MX_MIN_RATIO) * R) return p;
        if (h.kind == SCAN_W128 && h.mx_pat == 0 && (n > MX_MOST_128 || R > 100)) return p;
        if (R > 1 && R < (c5 ? 100 : 32)) return p;
        if (R == 1 && ((!plain && n < MX_MIN_LIST_ONE) || (c5 && h.mx_pat == 0))) return p;
    }
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
        // (2^24 minima per query at most: beyond 2^30 codes the groups are larger)
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

extern "C" int pq_search_form(const pq_index_t *idx, int nq, int64_t n, int R) {
    if (!idx || nq < 0 || n < 0 || R < 1 || R > PQ_MAX_R) {
        qadc_set_error("pq_search_form: bad handle, nq, n or R");
        return PQ_EINVAL;
    }
    return qadc_mx_plan(idx, nq, n, R, qadc_scan_plan(idx, nq, n, R)).use ? PQ_SCAN_MATRIX : PQ_SCAN_LOOKUP;
}
