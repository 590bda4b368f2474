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
// picking of a query, by one block, grows with the results and with what a code costs to score again; where
// its keys leave many codes as near as the R-th, that block has most of the list to score again.  The lines
// are where, in 29,088 pairs of timings of both forms (16 layouts, 20,000 to 8 * 10^6 codes, 5 to 256
// queries, R = 1 to 2000, two kinds of data), this form stops being the slower one: of the 6576 that it takes
// 76 are slower by 4 % or more.  Figures in us, look-ups / here; k = 1000 codes, M = 10^6.
//
// Codes times passes, and codes per result.  m x 4 bits, R = 100, 8 queries: 400k 39 / 34, 200k 30 / 34; R = 500,
// 48 queries, 400k: 97 / 130.  Irregular layouts, where a code is dearer to score again: {6,6,4} x 4, 64 queries,
// R = 100: 400k 153 / 148, 800k 177 / 85; R = 250, 800k: 202 / 240.
#define MX_MIN_CODES_NIB 800000
#define MX_MIN_RATIO_NIB 1000
#define MX_MIN_CODES 6000000
#define MX_MIN_RATIO 8000
// Short lists, m x 4 bits: 16 x 4, 100k: R = 10, 32 queries 33 / 47, 256 queries 87 / 67; R = 100, 64
// queries 49 / 43; 32 x 4 (twice the look-ups), R = 1, 50k, 100 queries: 76 / 45.
#define MX_MIN_LIST_8 200000
#define MX_MIN_LIST_8_LONG 100000
#define MX_MIN_LIST_16 50000
#define MX_LONG_NIB 6000000
// Of 40-bit codes more are equal, and of many queries one has a crowd of them near its R-th: {6,5,5,6,5,5,4,4},
// R = 500, 3.2M: 32 queries 187 / 127, 64 queries 231 / 709; R = 100, 800k: 110 / 57 and 136 / 191.
#define MX_MANY_40 40
// 128-bit codes of other field patterns (twice the products, one tile of queries per wave): R = 64, 64 queries,
// 1.6M 475 / 324, 3.2M 605 / 563; 100 queries 599 / 545 and 802 / 896.
#define MX_MOST_128 2000000

// Queries that it takes at least, with which the picking is worth the passes.
static int mx_min_queries(const DevLayout &h, int R) {
    const bool wide = h.acc_bits != 8, known = h.mx_pat != 0;
    switch (h.kind) {
        // m x 4 bits: 16 x 4, 10M, R = 100, 4 queries 61 / 58, 5: 87 / 58; R = 1000, 8M: 8 queries 124 / 126, 12: 170 / 126.
        // 16-bit tables, 3.2M: 16 x 4, R = 500, 8 queries 79 / 93, 12: 104 / 94; 32 x 4, R = 250, 12: 173 / 199, 16: 220 / 200
        case SCAN_NIB8: return wide ? (R < 32 ? 5 : 5 + R / 60) : 5 + 4 * (R / 1000);
        case SCAN_NIB16: return wide ? (R < 32 ? 5 : 5 + R / 30) : 5 + 4 * (R / 1000);
        // {6,6,4} x 4 (a known pattern), 3.2M: R = 500, 8 queries 143 / 165, 12: 203 / 168; R = 1, 8M, 8 queries 117 / 136.  Other
        // patterns, one tile of queries per wave: 3.2M, R = 100, 8 queries 91 / 116, 12: 123 / 117
        case SCAN_W64:
            if (known) return R == 1 ? 9 : (R <= 100 ? 5 : 5 + R / 70);
            return R == 1 ? 16 : 12 + R / 100;
        // {6,5,5} x 8, 3.2M, R = 250: 8 queries 216 / 315, 12: 316 / 317; other patterns, 1.6M, R = 64, 16 queries 282 / 208
        case SCAN_W128: return known ? (R <= 100 ? 5 : 6 + R / 50) : 16 + R / 12;
        // {5} x 8, 1.6M, R = 100: 5 queries 60 / 68, 8: 75 / 68
        default: return known ? 5 + R / 150 : 8 + R / 250;
    }
}

// Codes of an irregular layout that a few results need.  The single best code: the look-ups have no bound
// below the top of the range (40-bit codes, 3.2M, 256 queries: 28 ms / 0.25) but in a short list one query in
// some dozens has most of it near its best code ({6,5,5,6,5,5,4,4}, 800k, 32 queries: 104 / 2500; {5} x 7, 1.6M:
// 167 / 5100; {6,6,4} x 4 with 8-bit tables, 800k, 100 queries 207 / 2190).  Up to 99: R = 64, 1.6M codes of 40 bits: 32
// queries 122 / 51, 64 queries 150 / 395; other patterns, 400k, R = 32, 60 queries: 143 / 167.
static int64_t mx_min_list(const DevLayout &h, int nq, int R) {
    const bool c5 = h.kind == SCAN_C5, known = h.mx_pat != 0;
    if (R == 1) return c5 ? (known ? 1600000 : 3200000) : (h.acc_bits == 8 ? 1600000 : (known ? 0 : 800000));
    if (R < 100 && c5 && known) return nq > MX_MANY_40 ? 6400000 : 1600000;
    return R < 100 && !known ? 800000 : 0;
}

// The same for a call that is given a bound with its tables (pq_adc_scan_topk): the pilot, which the batched scan
// does without and which is most of what a short list costs the look-ups, is paid for already.  Lines from
// 26,240 pairs of timings of that call; of the 3974 that it takes 28 are slower by 4 % or more.  16 x 4 bits,
// R = 100, 8 queries: 400k 18 / 29, 1.6M 28 / 30, 5 queries 3.2M 36 / 34; R = 10, 800k: 12 queries 19 / 24, 32: 31 / 24;
// R = 500, 3.2M: 8 queries 56 / 60, 16: 80 / 61; R = 1, 3.2M, 64 queries: 92 / 160 on one kind of data, 101 / 54 on the other.
#define MX_MIN_CODES_BOUNDED 6400000
static bool mx_pays_bounded(const DevLayout &h, int nq, int64_t n, int R) {
    const bool wide = h.acc_bits != 8, known = h.mx_pat != 0;
    const int64_t work = n * ((nq + 3) / 4);
    // (32 x 4 bits with 16-bit tables, 3.2M, R = 250: 16 queries 168 / 191, 32: 290 / 195)
    const int step = wide && h.kind == SCAN_NIB16 ? 125 : 250;
    if (work < (int64_t)MX_MIN_CODES_BOUNDED * (R < step ? 1 : R / step)) return false;
    switch (h.kind) {
        case SCAN_NIB8:
        case SCAN_NIB16:
            if (R < 32) return n >= 800000 && nq >= 12 && !(R == 1 && h.kind == SCAN_NIB8 && !wide);
            return n >= 400000 && nq >= (R >= 500 || (wide && h.kind == SCAN_NIB16 && R >= 100) ? 12 : 5);
        // {6,6,4} x 8, 8M, R = 250: 12 queries 330 / 392, 24: 499 / 397; other patterns, 1.6M, R = 64, 64 queries: 320 / 308
        case SCAN_W128: return known && R < 1000 && nq >= (R < 100 ? 5 : (R < 250 ? 12 : 24)) && (R > 1 || n >= 800000);
        // {6,6,4} x 4, 3.2M, R = 100: 8 queries 61 / 66, 16: 97 / 70; other patterns, 1.6M: 16 queries 76 / 92, 32: 111 / 92
        case SCAN_W64:
            if (!known && (work < 2 * (int64_t)MX_MIN_CODES_BOUNDED || (R < 100 && n < 1600000))) return false;
            return R > 1 && n >= 800000 && nq >= (R < 1000 ? 12 : 24) && (R < 500 || work >= 25000000);
        // 40 bits: {6,5,5,6,5,5,4,4}, 3.2M, R = 100: 8 queries 45 / 51, 16: 66 / 53
        default:
            if (known) return R > 1 && R < 500 && nq >= 12 && n >= (R < 100 ? 6400000 : (R < 250 ? 1600000 : 3200000));
            return R > 1 && nq >= 8 && n >= (R < 100 ? 3200000 : 800000) && (R < 500 || work >= 25000000);
    }
}

MxPlan qadc_mx_plan(const pq_index *idx, int nq, int64_t n, int R, const ScanPlan &sp, bool bounded) {
    MxPlan p;
    memset(&p, 0, sizeof(p));
    const DevLayout &h = idx->h;
    if (h.mx_steps == 0 || nq < mx_min_queries(h, R) || qadc_option(PQ_OPT_SHARED_PASSES) == 0) return p;
    const int passes = (nq + 3) / 4;
    if (h.kind == SCAN_NIB8 || h.kind == SCAN_NIB16) {
        if (n * passes < MX_MIN_CODES_NIB || n < (int64_t)MX_MIN_RATIO_NIB * R) return p;
        const int list = h.kind == SCAN_NIB16 ? MX_MIN_LIST_16 : (R < 100 ? MX_MIN_LIST_8 : MX_MIN_LIST_8_LONG);
        if (n < list && n * passes < MX_LONG_NIB) return p;
    } else {
        const bool many = h.kind == SCAN_C5 && nq > MX_MANY_40;
        if (n * passes < MX_MIN_CODES || n < (int64_t)(many ? 2 * MX_MIN_RATIO : MX_MIN_RATIO) * R) return p;
        // A few results: the calibration ends the range of the keys close to the R-th, the levels are coarse
        // there, and where distances are alike most groups hold a code within them (40-bit codes, 2.5M, R = 10,
        // 64 queries: 151 / 432).
        if ((R > 1 && R < 32) || n < mx_min_list(h, nq, R)) return p;
        if (h.kind == SCAN_W128 && h.mx_pat == 0 && (n > MX_MOST_128 || R > 100)) return p;
    }
    if (bounded && !mx_pays_bounded(h, nq, n, R)) return p;
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

static int mx_form(const char *who, const pq_index_t *idx, int nq, int64_t n, int R, bool bounded) {
    if (!idx || nq < 0 || n < 0 || R < 1 || R > PQ_MAX_R) {
        qadc_set_error("%s: bad handle, nq, n or R", who);
        return PQ_EINVAL;
    }
    return qadc_mx_plan(idx, nq, n, R, qadc_scan_plan(idx, nq, n, R), bounded).use ? PQ_SCAN_MATRIX : PQ_SCAN_LOOKUP;
}
extern "C" int pq_search_form(const pq_index_t *idx, int nq, int64_t n, int R) {
    return mx_form("pq_search_form", idx, nq, n, R, false);
}
extern "C" int pq_scan_form(const pq_index_t *idx, int nq, int64_t n, int R) {
    return mx_form("pq_scan_form", idx, nq, n, R, true);
}
