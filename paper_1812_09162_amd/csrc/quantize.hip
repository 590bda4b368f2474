// pq_quantize_tables: the query-time distance quantizer of Section 3.4.
#include <math.h>
#include <stdlib.h>


#include "quotient.h"
#include "rules.h"
#include "scan_device.h"

// P blocks per query (grid = nq * P, block q*P + p).  Every block of a query computes
//   0. (fused form only) the float table from the query, eq. (1)
//   1. p_min(j), d_min = sum_j p_min(j) (fp64, ascending j)
//   2. float ADC (eq. (2), fp32, ascending j) of the first t_eff codes; d_max is
//      the k-th smallest of them, k = min(R, t_eff)
//   3. delta = (d_max - d_min)/q_max; q = min(q_max, floor((p - p_min)/delta))
// (a few thousand operations, cheaper to repeat than to hand over between kernels) and then
// its share of
//   4. key_bound: an upper bound of the k-th smallest quantized key among the first `pilot`
//      codes (pilot >= t_eff), from a 256-bin histogram of the keys (of their high bytes for
//      16-bit keys).  It bounds the R-th best key of the whole list from above and lets the
//      scan drop almost every code with one compare.
// Block p counts the codes [p*slice, (p+1)*slice) of the pilot.  With P == 1 the block selects
// the bound itself and stores it in the query's parameters.  With P > 1 no block waits for
// another: each leaves a record of 64 cumulative counts (how many of its codes have a key in
// coarse bin t or below, a coarse bin being four bins of the 256-bin histogram) in `bound_rec`,
// and the scan kernel adds the P records up (scan_bound_from_records); the parameters then
// carry q_max as the bound.  Block 0 of a query stores the tables and the parameters.
// `queries` non-null: tables are computed here (and stored to tables_out if
// that is non-null); otherwise they are read from tables_in.
// Threads of a block: a block's time is a chain of dependent steps, each shorter with QUANT_WIDE of them; where that
// pays is in quantize_wide.
#define QUANT_THREADS 256
#define QUANT_WIDE 1024
// The few layout numbers the kernel needs before anything else, as kernel arguments (reading
// them through the layout pointer would be a memory round trip ahead of every other load).
#define QUANT_MAX_GROUPS 16
struct QuantShape {
    int T, m, cs, qmax, d;
    int ubits, uds;  // bits and dimensions of every sub-quantizer if they are all alike, else 0
    int groups;      // groups described in grp (none: more of them, or of more than three sub-quantizers)
    uint32_t grp[QUANT_MAX_GROUPS][2];  // first group-table entry | bits << 16 | sub-quantizers << 24; bits of the first two of them | the first one's table entry << 16
};
// Pilot codes of a thread per batch (a wide block's batch is 4096 codes, the longest slice that is usual)
#define PILOT_PER_THREAD 8
#define PILOT_PER_THREAD_WIDE 4
// An entry of eq. (1): DS dimensions in ascending order, the codebook values requested eight at a time.  (24 at a time for sub-spaces of
// different widths: 40-bit codes, 10^7, one query 39.2 us a call, 37.1 so; {6,6,4} x 4, 621,640, one 29.4 / 27.4, seven queries 57.3 / 53.4.)
__device__ __forceinline__ float quant_entry(const float *z, const float *__restrict__ c, int ds) {
    float acc = 0.0f;
    int l = 0;
    for (; l + 8 <= ds; l += 8) {
        float cv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) cv[u] = c[l + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float diff = __fsub_rn(z[l + u], cv[u]);
            acc = __fadd_rn(acc, __fmul_rn(diff, diff));
        }
    }
    if (l < ds) {
        float cv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) cv[u] = l + u < ds ? c[l + u] : 0.0f;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (l + u < ds) {
                const float diff = __fsub_rn(z[l + u], cv[u]);
                acc = __fadd_rn(acc, __fmul_rn(diff, diff));
            }
    }
    return acc;
}
#define QUANT_PARAMS                                                                                                             \
    const DevLayout *__restrict__ L, const QuantShape shape, const EntryDesc *__restrict__ edesc, const float *__restrict__ cb, \
    const float *__restrict__ queries, const float *__restrict__ tables_in, float *__restrict__ tables_out,                      \
    const uint8_t *__restrict__ codes, int t_eff, int k, int pilot, int slice, int P, void *__restrict__ qtables,                \
    pq_qparams_t *__restrict__ qparams, char *__restrict__ gtab_out, size_t gtab_stride, size_t btab_rel,                        \
    char *__restrict__ hdr_out, uint16_t *__restrict__ bound_rec
#define QUANT_ARGS                                                                                                                \
    L, shape, edesc, cb, queries, tables_in, tables_out, codes, t_eff, k, pilot, slice, P, qtables, qparams, gtab_out, gtab_stride, \
    btab_rel, hdr_out, bound_rec
// fp32 sum in ascending order of the sixteen entries that the nibbles of two dwords select, all reads in flight
__device__ __forceinline__ float adc_sum16(const float *tab, uint32_t lo, uint32_t hi, float s) {
    float r[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) r[j] = tab[16 * j + (((j < 8 ? lo : hi) >> (4 * (j & 7))) & 15u)];
    asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7]),
                      "+v"(r[8]), "+v"(r[9]), "+v"(r[10]), "+v"(r[11]), "+v"(r[12]), "+v"(r[13]), "+v"(r[14]), "+v"(r[15]));
#pragma unroll
    for (int j = 0; j < 16; ++j) s = __fadd_rn(s, r[j]);
    return s;
}
// SHORT: the pilot is the whole list, and instead of a record a block leaves the codes that can be results (k_quantize_short).
template <int KIND, typename QT, int NT, bool SHORT>
__device__ __forceinline__ void quantize_block(QUANT_PARAMS, size_t cand_rel, int short_cap) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = shape.T, m = shape.m, cs = shape.cs, qmax = shape.qmax, d = shape.d;
    float *tab = (float *)smem;
    uint32_t *ord = (uint32_t *)(tab + T);                    // max(t_eff, d) words
    const int nord = (t_eff > d ? t_eff : d) > 0 ? (t_eff > d ? t_eff : d) : 1;
    float *pmin = (float *)(ord + nord);
    uint16_t *qt = (uint16_t *)(pmin + PQ_MAX_M);
    uint8_t *esub = (uint8_t *)(qt + T);
    QT *gtab = (QT *)(smem + (((size_t)T * 4 + (size_t)nord * 4 + PQ_MAX_M * 4 + (size_t)T * 3 + 15) &
                              ~(size_t)15));
    uint16_t *skey = SHORT ? (uint16_t *)(gtab + ((L->gtab_len + 7) & ~7)) : nullptr;  // [slice] keys of the block's codes
    __shared__ __align__(16) uint32_t hist[256];
    __shared__ uint32_t sel[8];
    __shared__ uint32_t kmem[QADC_KTH_MEM];
    __shared__ double s_dmin;
    __shared__ uint32_t s_range[2];  // smallest and largest calibration sum, as ordered words
    __shared__ __align__(16) uint32_t sdesc[PQ_MAX_M];  // table offset | bit offset << 12 | bits << 24 of each sub-quantizer; beyond: 0
    __shared__ uint32_t pmin_ord[PQ_MAX_M];  // table minima as ordered words (qadc_f2ord), by LDS atomic min
    if ((int)threadIdx.x >= m && threadIdx.x < PQ_MAX_M) sdesc[threadIdx.x] = 0u;
    if ((int)threadIdx.x < m) {  // (read after the barriers of the table set-up)
        sdesc[threadIdx.x] = (uint32_t)L->toff[threadIdx.x] | ((uint32_t)L->bitoff[threadIdx.x] << 12) |
                             ((uint32_t)L->nbits[threadIdx.x] << 24);
        pmin_ord[threadIdx.x] = 0xffffffffu;
    }

    if (threadIdx.x == 0) {
        s_range[0] = 0xffffffffu;
        s_range[1] = 0u;
    }
    const size_t q = blockIdx.x / (unsigned)P;
    const int p = (int)(blockIdx.x % (unsigned)P);
    const bool first = p == 0;
    const int lo = (int64_t)p * slice < pilot ? p * slice : pilot;
    const int hi = (int64_t)lo + slice < pilot ? lo + slice : pilot;
    constexpr int PPT = NT > QUANT_THREADS ? PILOT_PER_THREAD_WIDE : PILOT_PER_THREAD;
    const int step = PPT * NT;

    // The first batch of this block's pilot codes is requested now and used at the very end.
    uint2 pc[PPT];
    if (KIND == SCAN_NIB8 && hi > lo) {
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            int id = lo + u * NT + (int)threadIdx.x;
            id = id < hi ? id : hi - 1;
            pc[u] = *(const uint2 *)(codes + (size_t)id * 8);
        }
    }

    // The calibration code of this thread (at most one per thread in the common case) and the
    // descriptor of its table entry are requested now as well: they do not depend on anything.
    const bool cal_pre = t_eff <= 2 * NT && cs <= 16;  // up to two per thread
    uint32_t cw[2][4] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
    if (cal_pre) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int pp = r * NT + (int)threadIdx.x;
            if (pp < t_eff) qadc_load_code16(codes + (size_t)pp * cs, cs, cw[r]);
        }
    }
    EntryDesc ed0 = {0, 0, 0, 0};
    const bool alike = queries && shape.ubits > 0 && shape.uds > 0;
    if (!alike && (int)threadIdx.x < T) ed0 = edesc[threadIdx.x];

    if (alike) {
        // sub-quantizers that are all alike (m x 4 or m x 8 bits): entry e is centroid
        // e mod 2^bits of sub-quantizer e >> bits at codebook offset e * ds, so nothing has to
        // be looked up before the codebook values are requested, and the loop over the
        // dimensions has the same length in every lane
        float *zs = (float *)ord;  // the query lives where the ADC sums go later
        const int ub = shape.ubits, ds = shape.uds;
        // where a thread has one entry of up to eight dimensions, its codebook values travel while the query settles in
        // LDS (with more entries the registers only cost: 8 x 8 bits, 64 queries, 72 us with them, 67 without)
        const bool early = ds <= 8 && T <= NT;
        float c0[8];
        const float *cp = cb + ((int)threadIdx.x < T ? (size_t)threadIdx.x * ds : 0);
#pragma unroll
        for (int l = 0; l < 8; ++l) c0[l] = early && l < ds ? cp[l] : 0.0f;
        for (int i = threadIdx.x; i < d; i += NT) zs[i] = queries[q * d + i];
        __syncthreads();
        for (int e = threadIdx.x; e < T; e += NT) {
            const int j = e >> ub;
            const float *c = cb + (size_t)e * ds;
            const float *z = zs + j * ds;
            float acc = 0.0f;
            if (early) {
#pragma unroll
                for (int l = 0; l < 8; ++l)
                    if (l < ds) {
                        float diff = __fsub_rn(z[l], c0[l]);
                        acc = __fadd_rn(acc, __fmul_rn(diff, diff));
                    }
            } else {
                acc = quant_entry(z, c, ds);
            }
            tab[e] = acc;
            esub[e] = (uint8_t)j;
            atomicMin(&pmin_ord[j], qadc_f2ord(acc));
            if (tables_out && first) tables_out[q * T + e] = acc;
        }
        __syncthreads();
    } else if (queries) {
        float *zs = (float *)ord;
        for (int i = threadIdx.x; i < d; i += NT) zs[i] = queries[q * d + i];
        __syncthreads();
        for (int e = threadIdx.x; e < T; e += NT) {
            const EntryDesc ed = e == (int)threadIdx.x ? ed0 : edesc[e];
            const float acc = quant_entry(zs + ed.dim_off, cb + ed.cb_off, ed.ds);
            tab[e] = acc;
            esub[e] = (uint8_t)ed.j;
            atomicMin(&pmin_ord[ed.j], qadc_f2ord(acc));
            if (tables_out && first) tables_out[q * T + e] = acc;
        }
        __syncthreads();
    } else {
        __syncthreads();  // pmin_ord is set up
        for (int e = threadIdx.x; e < T; e += NT) {
            const float v = tables_in[q * T + e];
            const int j = e == (int)threadIdx.x ? ed0.j : edesc[e].j;
            tab[e] = v;
            esub[e] = (uint8_t)j;
            atomicMin(&pmin_ord[j], qadc_f2ord(v));
        }
        __syncthreads();
    }
    if ((int)threadIdx.x < m) pmin[threadIdx.x] = qadc_ord2f(pmin_ord[threadIdx.x]);
    // float ADC of the calibration codes, and on the way their smallest and largest
    uint32_t omin = 0xffffffffu, omax = 0u;
    for (int pp = threadIdx.x, r = 0; pp < t_eff; pp += NT, ++r) {
        const uint8_t *code = codes + (size_t)pp * cs;
        float s = 0.0f;
        const uint32_t *cwr = cw[r & 1];  // (r < 2 whenever cal_pre)
        if (KIND == SCAN_NIB8) {  // sub-code j is nibble j of the 8-byte code
            const uint2 v = cal_pre ? make_uint2(cwr[0], cwr[1]) : *(const uint2 *)code;
            s = adc_sum16(tab, v.x, v.y, s);
        } else if (KIND == SCAN_NIB16) {  // ... of the 16-byte code
            const uint4 v = cal_pre ? make_uint4(cwr[0], cwr[1], cwr[2], cwr[3]) : *(const uint4 *)code;
            s = adc_sum16(tab + 256, v.z, v.w, adc_sum16(tab, v.x, v.y, s));
        } else if (cs <= 16) {  // the code in registers, the sub-quantizers' fields from LDS
            uint32_t w[4];
            if (cal_pre) {
                w[0] = cwr[0]; w[1] = cwr[1]; w[2] = cwr[2]; w[3] = cwr[3];
            } else {
                qadc_load_code16(code, cs, w);
            }
            // (four sub-quantizers' descriptors, then their entries, in flight together; behind the last it is entry 0, not added)
            for (int j = 0; j < m; j += 4) {
                const uint4 dq = *(const uint4 *)&sdesc[j];
                const uint32_t ds[4] = {dq.x, dq.y, dq.z, dq.w};
                float r[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) r[i] = tab[(ds[i] & 0xfffu) + qadc_extract_sub16(w, (ds[i] >> 12) & 0xfffu, ds[i] >> 24)];
                asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
#pragma unroll
                for (int i = 0; i < 4; ++i) s = j + i < m ? __fadd_rn(s, r[i]) : s;
            }
        } else {
            for (int j = 0; j < m; ++j)
                s = __fadd_rn(s, tab[L->toff[j] + qadc_extract_sub(code, L->bitoff[j], L->nbits[j])]);
        }
        const uint32_t o = qadc_f2ord(s);
        ord[pp] = o;
        omin = o < omin ? o : omin;
        omax = o > omax ? o : omax;
    }
    omin = qadc_wave_min(omin);
    omax = qadc_wave_max(omax);
    if (threadIdx.x % QADC_WAVE == 0 && omin <= omax) {  // (s_range is set up before the table's barriers)
        atomicMin(&s_range[0], omin);
        atomicMax(&s_range[1], omax);
    }
    for (int i = threadIdx.x; i < 256; i += NT) hist[i] = 0;
    __syncthreads();
    if (threadIdx.x >= NT - QADC_WAVE) {  // d_min = sum of the minima in fp64, ascending j (m <= 64: one per lane)
        const int lane = (int)(threadIdx.x % QADC_WAVE);
        const double mine = lane < m ? (double)pmin[lane] : 0.0;
        const unsigned long long bits = (unsigned long long)__double_as_longlong(mine);
        double dm = 0.0;
        for (int j = 0; j < m; ++j) {  // (lane reads: no memory involved)
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, j);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(bits >> 32), j);
            dm = dm + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
        }
        if (lane == 0) s_dmin = dm;
    }
    float dmax = INFINITY;
    if (t_eff > 0) dmax = qadc_ord2f(qadc_block_kth_f32(ord, t_eff, k, hist, sel, kmem, s_range[0], s_range[1]));
    __syncthreads();
    // (every thread divides: no barrier behind one that does)
    const double dmin = s_dmin;
    double delta = ((double)dmax - dmin) / (double)qmax;
    const bool ok = (delta > 0.0) && isfinite(delta);
    delta = ok ? delta : 0.0;
    const uint32_t mx_scale = btab_rel ? mx_scale_of(ok && t_eff > 0 ? (float)(((double)qadc_ord2f(s_range[0]) - dmin) / delta) : (float)qmax, (uint32_t)qmax) : 0u;
    // floor((p - p_min) / delta) in fp32 where that cannot differ, else (or with a delta not of ordinary size) in fp64.
    // (16-bit tables: too few bits are left.)
    const float inv = sizeof(QT) == 1 && delta > 1e-30 && delta < 1e30 ? (float)(1.0 / delta) : 0.0f;
    for (int e = threadIdx.x; e < T; e += NT) {
        const float p = tab[e], pm = pmin[esub[e]];
        uint32_t qv = 0;
        const float xf = (p - pm) * inv;
        if (inv > 0.0f && quotient_sure(xf, QUOTIENT_SLACK)) {
            qv = (uint32_t)fminf(xf, 255.0f);
        } else if (delta > 0.0) {
            double x = floor(((double)p - (double)pm) / delta);
            qv = (x >= (double)qmax) ? (uint32_t)qmax : (uint32_t)x;
        }
        qt[e] = (uint16_t)qv;
        if (first) {
            if (sizeof(QT) == 1)
                ((uint8_t *)qtables)[q * T + e] = (uint8_t)qv;
            else
                ((uint16_t *)qtables)[q * T + e] = (uint16_t)qv;
        }
    }
    __syncthreads();
    uint32_t bound = (uint32_t)qmax;
    if (pilot > 0 || gtab_out) {
        if ((KIND != SCAN_NIB8 && KIND != SCAN_NIB16) && shape.groups > 0) {
            // build_gtab with the groups' descriptors at hand: read from the layout, they are two memory round trips a group
#pragma unroll
            for (int g = 0; g < QUANT_MAX_GROUPS; ++g)
                if (g < shape.groups) {
                    const uint32_t a = shape.grp[g][0], b = shape.grp[g][1];
                    const int cnt = (int)(a >> 24), entries = 1 << ((a >> 16) & 255u), b0 = (int)(b & 15u), b1 = (int)((b >> 4) & 15u);
                    const uint16_t *t0 = qt + (b >> 16), *t1 = t0 + (1 << b0), *t2 = t1 + (1 << b1);
                    for (int e = threadIdx.x; e < entries; e += NT) {
                        uint32_t s = t0[e & ((1 << b0) - 1)];
                        if (cnt > 1) s += t1[(e >> b0) & ((1 << b1) - 1)];
                        if (cnt > 2) s += t2[e >> (b0 + b1)];
                        gtab[(a & 0xffffu) + e] = (QT)(s > (uint32_t)qmax ? (uint32_t)qmax : s);
                    }
                }
            __syncthreads();
        } else {
            build_gtab<KIND, QT>(L, qt, gtab);
        }
        if (gtab_out && first) {  // hand the prepared group tables to the scan kernel
            QT *dst = (QT *)(gtab_out + q * gtab_stride);
            for (int e = threadIdx.x; e < L->gtab_len; e += NT) dst[e] = gtab[e];
            if (btab_rel) {
                build_btab(L, qt, mx_scale, (uint32_t *)(gtab_out + q * gtab_stride + btab_rel));
                if (threadIdx.x == 0) ((ScanHdr *)(hdr_out + q * gtab_stride))->scale = mx_scale;
            }
        }
    }
    if (!SHORT && hdr_out && first) scan_hdr_clear((ScanHdr *)(hdr_out + q * gtab_stride));  // empty candidate lists
    // (A block's time is a chain of LDS round trips: the entries of an irregular code are read in flight together, and saturated keys, three in four,
    // are not counted by a vote and an atomic of their own.  10^7 codes of 16 x 4 bits, one query, us a call 34.0 / 32.6, two streams 20.2 / 19.6, three
    // 16.1 / 15.6; on four, where scans of three queries share the memory system, 12.6 / 12.6 (12.5 with the vote, and as much with a pause of its length.
    // Entries of two codes of 16 x 4 bits in flight together: one stream the same, four 12.7.)  {6,6,4} x 4, 621,640 codes 32.0 / 27.9.)
    if (pilot > 0) {
        const int shift = sizeof(QT) == 1 ? 0 : 8;
        for (int i = threadIdx.x; i < 256; i += NT) hist[i] = 0;
        __syncthreads();
        // count one key (0xffffffff = none); not those of the last bin, every saturated key among them: where the others are fewer
        // than k it is the answer all the same
        auto count_key = [&](uint32_t key, int id) {
            if (SHORT && key != 0xffffffffu) skey[id - lo] = (uint16_t)key;
            const uint32_t bin = key >> shift;
            if (bin < 255u) atomicAdd(&hist[bin], 1u);
        };
        if (KIND == SCAN_NIB8) {
            for (int base = lo; base < hi; base += step) {
                if (base != lo) {
#pragma unroll
                    for (int u = 0; u < PPT; ++u) {
                        int id = base + u * NT + (int)threadIdx.x;
                        id = id < hi ? id : hi - 1;
                        pc[u] = *(const uint2 *)(codes + (size_t)id * 8);
                    }
                }
#pragma unroll
                for (int u = 0; u < PPT; ++u) {
                    if (NT > QUANT_THREADS && base + u * NT >= hi) break;  // (in narrow blocks it costs more than it saves)
                    const int id = base + u * NT + (int)threadIdx.x;
                    const uint32_t sm = sum8(gtab, pc[u].x, pc[u].y);
                    count_key(id < hi ? (sm > (uint32_t)qmax ? (uint32_t)qmax : sm) : 0xffffffffu, id);
                }
            }
        } else if ((KIND == SCAN_W64 || KIND == SCAN_C5) && L->g32ok != 0 && L->ng <= QADC_MAXG_FAST) {
            // group descriptors in registers; 8-byte codes one per load, 5-byte codes four per
            // 20-byte chunk of five dwords (slices start on multiples of 1024 codes)
            const GroupDesc gd = load_group_desc(L);
            for (int base = lo; base < hi; base += step) {
                if (KIND == SCAN_W64) {
                    uint2 w[PPT];
#pragma unroll
                    for (int u = 0; u < PPT; ++u) {
                        int id = base + u * NT + (int)threadIdx.x;
                        id = id < hi ? id : hi - 1;
                        w[u] = *(const uint2 *)(codes + (size_t)id * 8);
                    }
#pragma unroll
                    for (int u = 0; u < PPT; ++u) {
                        if (base + u * NT >= hi) break;
                        const int id = base + u * NT + (int)threadIdx.x;
                        const uint32_t sm = sum_groups_flight(gd, gtab, w[u].x, w[u].y);
                        count_key(id < hi ? (sm > (uint32_t)qmax ? (uint32_t)qmax : sm) : 0xffffffffu, id);
                    }
                } else {
                    uint32_t c5[PPT / 4][5];
#pragma unroll
                    for (int u = 0; u < PPT / 4; ++u) {
                        const int id = base + 4 * (u * NT + (int)threadIdx.x);
#pragma unroll
                        for (int i = 0; i < 5; ++i)  // a chunk not wholly inside is handled code by code
                            c5[u][i] = id + 3 < hi ? ((const uint32_t *)(codes + (size_t)id * 5))[i] : 0u;
                    }
#pragma unroll
                    for (int u = 0; u < PPT / 4; ++u) {
                        const int id = base + 4 * (u * NT + (int)threadIdx.x);
                        uint32_t k4[4];
                        if (id + 3 < hi) {
                            // code v = bits [40v, 40v+40) of the chunk, as (low dword, high byte)
                            const uint32_t l4[4] = {c5[u][0], __builtin_amdgcn_alignbit(c5[u][2], c5[u][1], 8),
                                                    __builtin_amdgcn_alignbit(c5[u][3], c5[u][2], 16),
                                                    __builtin_amdgcn_alignbit(c5[u][4], c5[u][3], 24)};
                            const uint32_t h4[4] = {c5[u][1] & 0xffu, (c5[u][2] >> 8) & 0xffu,
                                                    (c5[u][3] >> 16) & 0xffu, c5[u][4] >> 24};
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const uint32_t sm = sum_groups_flight(gd, gtab, l4[v], h4[v]);
                                k4[v] = sm > (uint32_t)qmax ? (uint32_t)qmax : sm;
                            }
                        } else {
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                k4[v] = id + v < hi ? key_at<KIND, QT>(L, gtab, codes, id + v) : 0xffffffffu;
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v) count_key(k4[v], id + v);
                    }
                }
            }
        } else {
            for (int base = lo; base < hi; base += step) {
                uint32_t key[PPT];
                keys_batch<KIND, QT, PPT>(L, gtab, codes, (int64_t)base + threadIdx.x, NT,
                                        (int64_t)hi, key);
#pragma unroll
                for (int u = 0; u < PPT; ++u) count_key(key[u], base + u * NT + (int)threadIdx.x);
            }
        }
        __syncthreads();
        if constexpr (SHORT) {
            // The codes of as many whole bins from the lowest on as the block's list holds, and how many bins these are: no code outside them
            // is in a lower bin than one inside, so if the R-th of all is within every block's bins, it was found among these.
            if (threadIdx.x < QADC_WAVE) {
                uint4 h4 = *(const uint4 *)&hist[4 * threadIdx.x];
                const uint32_t c4 = h4.x + h4.y + h4.z + h4.w, room = (uint32_t)short_cap, upto = qadc_wave_incl_scan(c4);
                if (threadIdx.x == QADC_WAVE - 1) h4.w = (uint32_t)(hi - lo) - upto;  // (the last bin was not counted)
                uint32_t run = upto - c4;
                uint32_t whole = 0;
                whole += (run += h4.x) <= room ? 1u : 0u;
                whole += (run += h4.y) <= room ? 1u : 0u;
                whole += (run += h4.z) <= room ? 1u : 0u;
                whole += (run += h4.w) <= room ? 1u : 0u;
                whole = (uint32_t)__builtin_amdgcn_readlane((int)qadc_wave_incl_scan(whole), QADC_WAVE - 1);
                if (threadIdx.x == 0) {
                    sel[0] = whole;
                    sel[1] = 0u;
                }
            }
            __syncthreads();
            const uint32_t whole = sel[0];
            ScanHdr *hd = (ScanHdr *)(hdr_out + q * gtab_stride);
            uint32_t *cand = (uint32_t *)(hdr_out + q * gtab_stride + cand_rel) + (size_t)p * short_cap;
            for (int i = threadIdx.x; i < hi - lo; i += NT) {
                const uint32_t key = skey[i];
                if ((key >> shift) < whole) cand[atomicAdd(&sel[1], 1u)] = (key << SHORT_SLICE_BITS) | (uint32_t)i;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                hd->count[p][0] = sel[1];
                hd->count[p][1] = whole;
            }
        } else if (P > 1) {
            // this block's record: cumulative counts over 64 coarse bins, one lane per bin
            if (threadIdx.x < QADC_WAVE) {
                const uint4 h4 = *(const uint4 *)&hist[4 * threadIdx.x];
                const uint32_t c4 = h4.x + h4.y + h4.z + h4.w;
                const uint32_t cum = qadc_wave_incl_scan(c4);
                bound_rec[((size_t)q * QADC_REC_BINS + threadIdx.x) * QADC_REC_SLOTS + p] =
                    (uint16_t)(cum > 65535u ? 65535u : cum);
            }
        } else {
            if (threadIdx.x < QADC_WAVE) qadc_wave_select_bin(hist, (uint32_t)k, 0u, sel);
            __syncthreads();
            bound = sizeof(QT) == 1 ? sel[0] : ((sel[0] << 8) | 255u);
        }
    }
    if (!first) return;
    if (threadIdx.x == 0) {
        pq_qparams_t prm;
        prm.d_min = dmin;
        prm.delta = delta;
        prm.d_max = dmax;
        prm.key_bound = bound;
        qparams[q] = prm;
    }
}

// (64-bit codes of nibbles: narrow blocks hold 80 registers without the bound, six to a CU, and calls of some 1600 to 1800 blocks have a second
// filling: 16 x 4 bits, 85,000 codes, 41 queries 34.9 us a call, 32.9 with seven)
template <int KIND, typename QT, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == QUANT_THREADS && KIND == SCAN_NIB8 ? 7 : 1)))
k_quantize(QUANT_PARAMS) {
    quantize_block<KIND, QT, NT, false>(QUANT_ARGS, 0, 0);
}

// Short lists, a few queries: the blocks that would count a pilot count every code of the list, so the scan's work is done when
// they have, and they leave the codes that can be results, a list per block of (key, place in the slice), for k_short_final.
// (512 threads: 16 x 4 bits, one query over 250,000 codes 17.6 us a call, 20.3 with 256, 17.0 with 1024; 32 queries over 65,537 26.9, 24.6, 45.2.)
#define SHORT_THREADS 512
template <int KIND, typename QT>
__global__ void __launch_bounds__(SHORT_THREADS)
k_quantize_short(QUANT_PARAMS, size_t cand_rel, int short_cap) {
    quantize_block<KIND, QT, SHORT_THREADS, true>(QUANT_ARGS, cand_rel, short_cap);
}

// The pilot of four queries by one block, for batches whose queries have one block each: the same bound as k_quantize's
// own pilot (the largest key of the bin of the k-th smallest key among the first `pilot` codes), from the quantized tables
// that it left.  A code is loaded and split once for the four, whose entries of a group are one 8-byte word of an
// interleaved table; and once a few thousand codes are counted, the bin of the k-th among them bounds the final one from
// above, and only keys up to it are counted from there on.
// What bounds it: the 8-byte LDS reads, eight a code of 64 bits (random entries, about seven clocks a wave).  16 x 4 bits, 65,536 codes, 1000
// queries: 42 us beside 8 of the quantizer that counts nothing; 95 with a block per query counting its own.
#define PILOT4_THREADS 1024
template <int KIND, typename QT>
__global__ void __launch_bounds__(PILOT4_THREADS)
k_pilot4(const DevLayout *__restrict__ L, const uint8_t *__restrict__ codes, int k, int pilot,
         const void *__restrict__ qtables, int T, int gtab_len, int nq, GroupDesc gd, pq_qparams_t *__restrict__ qparams) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NT = PILOT4_THREADS, PC = KIND == SCAN_NIB16 ? 2 : 4 /* codes per thread and round (128 registers) */, shift = sizeof(QT) == 1 ? 0 : 8;
    constexpr bool WIDE = KIND == SCAN_NIB16 || KIND == SCAN_W128;
    uint2 *tab = (uint2 *)smem;  // [gtab_len]
    uint2 *ent = tab + gtab_len;  // [T] quantized entries of the four queries
    uint32_t *hist = (uint32_t *)(ent + T);  // [MQ][256]
    uint32_t *sel = hist + MQ * 256;         // [MQ][2]
    const int q0 = blockIdx.x * MQ, wave = threadIdx.x / QADC_WAVE;
    uint4 c[PC];  // a round's codes
    auto request = [&](int base) {  // codes past the end: the last one again
#pragma unroll
        for (int u = 0; u < PC; ++u) {
            int id = base + u * NT + (int)threadIdx.x;
            id = id < pilot ? id : pilot - 1;
            if (WIDE) {
                c[u] = *(const uint4 *)(codes + (size_t)id * 16);
            } else if (KIND == SCAN_C5) {
                const size_t at = (size_t)id * 5;
                if (id + 1 < pilot) {  // the two aligned dwords that hold the code
                    const uint32_t *p = (const uint32_t *)(codes + (at & ~(size_t)3));
                    const uint64_t w = (((uint64_t)p[1] << 32) | p[0]) >> (8 * ((uint32_t)at & 3u));
                    c[u] = make_uint4((uint32_t)w, (uint32_t)(w >> 32) & 0xffu, 0u, 0u);
                } else {  // (there may be no memory behind the last code)
                    const uint8_t *p = codes + at;
                    c[u] = make_uint4((uint32_t)p[0] | (uint32_t)p[1] << 8 | (uint32_t)p[2] << 16 | (uint32_t)p[3] << 24, p[4], 0u, 0u);
                }
            } else {
                const uint2 w = *(const uint2 *)(codes + (size_t)id * 8);
                c[u] = make_uint4(w.x, w.y, 0u, 0u);
            }
        }
    };
    request(0);
    for (int e = threadIdx.x; e < T; e += NT) {
        uint32_t v[MQ];
#pragma unroll
        for (int j = 0; j < MQ; ++j) v[j] = ((const QT *)qtables)[(size_t)(q0 + j < nq ? q0 + j : q0) * T + e];
        ent[e] = make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
    }
    for (int i = threadIdx.x; i < MQ * 256; i += NT) hist[i] = 0;
    __syncthreads();
    // Group entries as sums of four at a time.  8-bit tables: not saturated (at most 64 addends of 255 stay below 2^16;
    // the key is the smaller of the sum and q_max all the same).
    if constexpr (KIND == SCAN_NIB8 || KIND == SCAN_NIB16) {
        for (int e = threadIdx.x; e < gtab_len; e += NT) {  // group = code byte
            const uint2 *s = ent + 32 * (e >> 8);
            MqAcc<QT> a;
            a.zero();
            a.add(s[e & 15]);
            a.add(s[16 + ((e >> 4) & 15)]);
            tab[e] = make_uint2(a.a, a.b);
        }
    } else {
        const int ng = L->ng;
        for (int g = 0; g < ng; ++g) {
            const int entries = 1 << L->gw[g], first = L->gfirst[g], cnt = L->gcount[g], base = L->gbase[g];
            for (int e = threadIdx.x; e < entries; e += NT) {
                uint32_t rem = (uint32_t)e;
                MqAcc<QT> a;
                a.zero();
                for (int i = 0; i < cnt; ++i) {
                    const int b = L->nbits[first + i];
                    a.add(ent[L->toff[first + i] + (rem & ((1u << b) - 1u))]);
                    rem >>= b;
                }
                tab[base + e] = make_uint2(a.a, a.b);
            }
        }
    }
    __syncthreads();
    uint32_t lim[MQ];  // keys in bins below it are counted (never the last: the selection's answer where there are too few)
#pragma unroll
    for (int j = 0; j < MQ; ++j) lim[j] = 255u << shift;
    const uint32_t three = 3;
    for (int base = 0; base < pilot; base += PC * NT) {
        uint4 w[PC];
#pragma unroll
        for (int u = 0; u < PC; ++u) w[u] = c[u];
        if (base + PC * NT < pilot) request(base + PC * NT);
        MqAcc<QT> acc[PC];
#pragma unroll
        for (int u = 0; u < PC; ++u) {
            acc[u].zero();
            if constexpr (KIND == SCAN_NIB8 || KIND == SCAN_NIB16) {
                const uint32_t d[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
                for (int g = 0; g < (KIND == SCAN_NIB8 ? 8 : 16); g += 4) {
                    acc[u].add(mq_entry<0>(g, d[g >> 2], three));
                    acc[u].add(mq_entry<1>(g + 1, d[g >> 2], three));
                    acc[u].add(mq_entry<2>(g + 2, d[g >> 2], three));
                    acc[u].add(mq_entry<3>(g + 3, d[g >> 2], three));
                }
            } else {
#pragma unroll
                for (int g = 0; g < QADC_MAXG_FAST; ++g)
                    if (g < gd.ng) {
                        const uint32_t off = (uint32_t)(gd.off[g] & 31), wd = (uint32_t)gd.w[g];
                        acc[u].add(tab[gd.base[g] + __builtin_amdgcn_ubfe(gd.off[g] >= 32 ? w[u].y : w[u].x, off, wd)]);
                        if (WIDE) acc[u].add(tab[gd.base2[g] + __builtin_amdgcn_ubfe(gd.off[g] >= 32 ? w[u].w : w[u].z, off, wd)]);
                    }
            }
        }
#pragma unroll
        for (int u = 0; u < PC; ++u) {
            const bool in = base + u * NT + (int)threadIdx.x < pilot;
#pragma unroll
            for (int j = 0; j < MQ; ++j) {
                const uint32_t s = acc[u].sum(j);
                if (in && s < lim[j]) atomicAdd(&hist[j * 256 + (s >> shift)], 1u);
            }
        }
        // after 4,096 and 16,384 codes, and at the end: the bin of the k-th so far
        const int done = base + PC * NT;
        if (done == 4096 || done == 16384 || done >= pilot) {
            __syncthreads();
            if (wave < MQ) qadc_wave_select_bin(hist + wave * 256, (uint32_t)k, 0u, sel + 2 * wave);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < MQ; ++j) lim[j] = min(sel[2 * j] + 1u, 255u) << shift;
        }
    }
    if (threadIdx.x < MQ && q0 + (int)threadIdx.x < nq)
        qparams[q0 + threadIdx.x].key_bound = sizeof(QT) == 1 ? sel[2 * threadIdx.x] : (sel[2 * threadIdx.x] << 8) | 255u;
}

// Pilot codes of a block at least, when several share them (one batch of a block of 256 threads, eight per thread, half of one of a
// wide block), and at most.  A batch's requests beyond the slice ask for its last code again: ending them there cost more
// (16 x 4 bits, 1000 queries, 88 us a call, 93 with an end in the loop).
#define PILOT_BATCH (8 * QUANT_THREADS)
#define PILOT_BLOCK_MAX 65536
int qadc_pilot_blocks_max(int nq) {
    const int64_t cap = qadc_option(PQ_OPT_PILOT_BLOCKS);
    int pmax = 2048 / (nq > 0 ? nq : 1);  // (blocks of 256 threads: a few thousand fill the chip)
    pmax = pmax < 1 ? 1 : (pmax > QADC_REC_SLOTS ? QADC_REC_SLOTS : pmax);
    return cap >= 1 && cap < pmax ? (int)cap : pmax;
}

size_t qadc_pilot_scratch_bytes(int nq) {
    return (size_t)(nq > 0 ? nq : 0) * QADC_REC_BINS * QADC_REC_SLOTS * sizeof(uint16_t);
}

// The pilot of a call: how many codes, split over how many blocks per query.  With scratch
// memory (the fused search) a small batch of queries spreads a large pilot over many
// blocks; without it every query has one block and the pilot stays small.
PilotPlan qadc_pilot_plan(int nq, int64_t n, int t_eff, int R, bool have_scratch, bool cheap_lookups) {
    int64_t multi = qadc_option(PQ_OPT_PILOT_CODES);
    const int64_t single = qadc_option(PQ_OPT_PILOT_CODES_SINGLE);
    PilotPlan pp;
    const int pmax = have_scratch ? qadc_pilot_blocks_max(nq) : 1;
    // The whole sample pays when many blocks share it and a look-up is cheap (m x 4 codes, one
    // query per call: 4096 codes per block; fewer candidates then shorten the scan's appends and
    // the selection by more than the sample costs).  Otherwise half of it, as long as that is
    // not below 262144.
    const int64_t per_block = cheap_lookups ? 4096 : 2048;
    if (multi > 262144 && multi > per_block * pmax) multi = per_block * pmax > 262144 ? per_block * pmax : 262144;
    int64_t want = pmax > 1 ? multi : single;
    // the candidates the scan keeps grow with R / pilot: long result lists get a longer pilot
    if (pmax > 1 && want < pilot_for_results(n, R, nq)) want = pilot_for_results(n, R, nq);
    if (want > (int64_t)pmax * PILOT_BLOCK_MAX) want = (int64_t)pmax * PILOT_BLOCK_MAX;
    if (want < 64 * (int64_t)R) want = 64 * (int64_t)R;
    if (want < t_eff) want = t_eff;
    if (want > n) want = n;
    int64_t P = (want + PILOT_BATCH - 1) / PILOT_BATCH;
    if (P > pmax) P = pmax;
    if (P < 1) P = 1;
    int64_t slice = (want + P - 1) / P;
    slice = (slice + 1023) / 1024 * 1024;
    if (slice < 1024) slice = 1024;
    pp.pilot = (int)want;
    pp.P = (int)P;
    pp.slice = (int)slice;
    return pp;
}

// bits and dimensions of every sub-quantizer if they are all alike, else 0
static void quantize_alike(const DevLayout &h, int &ubits, int &uds) {
    ubits = h.nbits[0];
    uds = h.dsub[0];
    for (int j = 1; j < h.m; ++j) {
        if (h.nbits[j] != ubits) ubits = 0;
        if (h.dsub[j] != uds) uds = 0;
    }
}

static QuantShape quantize_shape(const DevLayout &h) {
    QuantShape s = {h.T, h.m, h.cs, h.qmax, h.d, 0, 0, 0, {}};
    quantize_alike(h, s.ubits, s.uds);
    bool ok = h.ng <= QUANT_MAX_GROUPS && h.gtab_len <= 65536;
    for (int g = 0; g < h.ng && ok; ++g) ok = h.gcount[g] >= 1 && h.gcount[g] <= 3;
    if (ok) {
        s.groups = h.ng;
        for (int g = 0; g < h.ng; ++g) {
            const int f = h.gfirst[g], c = h.gcount[g];
            s.grp[g][0] = (uint32_t)h.gbase[g] | ((uint32_t)h.gw[g] << 16) | ((uint32_t)c << 24);
            s.grp[g][1] = (uint32_t)h.nbits[f] | (uint32_t)(c > 1 ? h.nbits[f + 1] : 0) << 4 | ((uint32_t)h.toff[f] << 16);
        }
    }
    return s;
}

static size_t quantize_lds(const DevLayout &h, int t_eff, size_t esz) {
    const size_t nord = (size_t)((t_eff > h.d ? t_eff : h.d) > 0 ? (t_eff > h.d ? t_eff : h.d) : 1);
    return (((size_t)h.T * 4 + nord * 4 + PQ_MAX_M * 4 + (size_t)h.T * 3 + 15) & ~(size_t)15) +
           (size_t)h.gtab_len * esz;
}

#define PILOT4_LEAST 16384  // codes
static size_t pilot4_lds(const DevLayout &h) { return ((size_t)h.gtab_len + (size_t)h.T) * sizeof(uint2) + MQ * 256 * 4 + MQ * 8; }

// Whether a batch's pilots are counted four queries to a block (k_pilot4) behind a quantizer that counts none.  Stage calls of
// gamma or Gaussian data, d = 128, R = 100, 200,001 codes, us a call, own pilots / four to a block: 16 x 4 bits 256 queries 89 / 105, 257 115 / 105, 512 144 / 134,
// 1000 244 / 202; 32 x 4 257 178 / 159, 1000 422 / 312; {6,6,4} x 4 256 164 / 170, 257 209 / 169, 1000 417 / 315; 40-bit codes 111 / 125,
// 149 / 126, 295 / 227; 8 x 8 134 / 142, 182 / 144, 363 / 263; {6,6,4} x 8 64 queries 229 / 206, 257 499 / 379, 1000 1078 / 792: where a CU would have
// more than one query's pilot.  Short ones lose the second launch: {6,5,5} x 4, 301 codes, 1030 queries 80 / 87; 40-bit, 5000 codes, 1100 114 / 117;
// 16,384 codes, 300 queries: 16 x 4 47.8 / 45.1, 40-bit 67 / 59.
template <int KIND>
static bool pilot4_pays(const DevLayout &h, int nq, const PilotPlan &pp) {
    if (KIND == SCAN_GENERIC || pp.P != 1 || pp.pilot < PILOT4_LEAST) return false;
    if ((KIND == SCAN_W64 || KIND == SCAN_C5) && (h.g32ok == 0 || h.ng > QADC_MAXG_FAST)) return false;
    if (KIND == SCAN_W128 && h.ng / 2 > QADC_MAXG_FAST) return false;
    return nq > 256 && pilot4_lds(h) <= 128 * 1024;
}

// The whole of a short list's scan by the quantizer's blocks, if it is one: blocks per query, codes per block and entries of a block's list.
// Where the pilot would be the whole list anyway, the slices are at most 4096 codes (64 lists a query: 262,144 codes) and a block's list holds the
// results and a quarter more.  us a call of one query, R = 100, pilot and scan / this: 16 x 4 bits 1000 codes 20.2 / 15.2, 50,000 19.2 / 15.3,
// 250,000 19.3 / 17.6; {6,6,4} x 4 33.6 / 21.5, 33.0 / 21.7, 33.2 / 26.0; 32 queries over 65,537: 33.5 / 22.9, 52.0 / 33.5.  None of
// 110 sizes over six layouts was slower.
ShortPlan qadc_short_plan(const pq_index *idx, int nq, int64_t n, int R, int t, const ScanPlan &sp) {
    ShortPlan p = {};
    if (n < 1 || nq < 1) return p;
    const int64_t want = t > 4 * (int64_t)R ? t : 4 * (int64_t)R;
    const PilotPlan pp = qadc_pilot_plan(nq, n, (int)(n < want ? n : want), R, true, idx->h.kind == SCAN_NIB8 || idx->h.kind == SCAN_NIB16);
    if (pp.pilot < n) return p;
    const int64_t least = R + R / 4 + 16, room = (int64_t)QADC_NSUB * sp.cap * 2;
    if (least > SHORT_CAP_MAX || room < least) return p;
    int64_t P = room / least < QADC_NSUB ? room / least : QADC_NSUB;
    // (about two blocks per CU, with more queries longer slices: every block makes its query's tables.  130,001 codes, 16 queries, us a call, up to 1024 / 512
    // blocks: 16 x 4 bits 25.1 / 20.4, {6,6,4} x 4 40.3 / 29.7, 40-bit codes 34.7 / 26.0; 65,537 codes, 32 queries 22.0 / 22.9, 32.2 / 33.5, 28.2 / 28.9)
    const int64_t few = SHORT_BLOCKS / nq, longest = (n + (1 << SHORT_SLICE_BITS) - 1) >> SHORT_SLICE_BITS;
    if (P > few) P = few > longest ? few : (longest < P ? longest : P);
    const int64_t slice = ((n + P - 1) / P + 1023) / 1024 * 1024;
    if (slice > (1 << SHORT_SLICE_BITS)) return p;
    P = (n + slice - 1) / slice;
    if (P * nq > SHORT_MAX_BLOCKS) return p;
    p.use = true;
    p.P = (int)P;
    p.slice = (int)slice;
    p.cap = (int)(room / P < SHORT_CAP_MAX ? room / P : SHORT_CAP_MAX);
    return p;
}

template <int KIND, typename QT>
static int launch_short(const pq_index *idx, const float *queries, int nq, const uint8_t *codes, int n, int t_eff, int k, const ShortPlan &sh,
                        void *qtables, pq_qparams_t *qparams, const ScanPlan &sp, char *ws, hipStream_t s) {
    const size_t lds = ((quantize_lds(idx->h, t_eff, sizeof(QT)) + 15) & ~(size_t)15) + 16 * sizeof(QT) + (size_t)sh.slice * 2;
    const QuantShape shape = quantize_shape(idx->h);
    if (lds > 48 * 1024)
        QADC_HIP_TRY(hipFuncSetAttribute((const void *)k_quantize_short<KIND, QT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((k_quantize_short<KIND, QT>), dim3((unsigned)nq * (unsigned)sh.P), dim3(SHORT_THREADS), lds, s, idx->dev,
                       shape, idx->edesc, idx->codebooks, queries,
                       (const float *)nullptr, (float *)nullptr, codes, t_eff, k, n, sh.slice, sh.P, qtables, qparams, ws + sp.gtab_off,
                       sp.per_query, (size_t)0, ws, (uint16_t *)nullptr, sp.cand_off, sh.cap);
    QADC_LAUNCH_CHECK("k_quantize_short");
    return PQ_OK;
}

int qadc_quantize_short(const pq_index *idx, const float *queries, int nq, const uint8_t *codes, int64_t n, int t, int R, const ShortPlan &sh,
                        void *qtables, pq_qparams_t *qparams, const ScanPlan &sp, char *ws, hipStream_t s) {
    const int64_t want = t > 4 * (int64_t)R ? t : 4 * (int64_t)R;
    const int t_eff = (int)(n < want ? n : want), k = R < t_eff ? R : t_eff;
    const bool u8 = idx->h.acc_bits == 8;
#define QADC_GO(KIND)                                                                                                        \
    return u8 ? launch_short<KIND, uint8_t>(idx, queries, nq, codes, (int)n, t_eff, k, sh, qtables, qparams, sp, ws, s)  \
              : launch_short<KIND, uint16_t>(idx, queries, nq, codes, (int)n, t_eff, k, sh, qtables, qparams, sp, ws, s)
    switch (idx->h.kind) {
        case SCAN_NIB8: QADC_GO(SCAN_NIB8);
        case SCAN_NIB16: QADC_GO(SCAN_NIB16);
        case SCAN_W64: QADC_GO(SCAN_W64);
        case SCAN_C5: QADC_GO(SCAN_C5);
        case SCAN_W128: QADC_GO(SCAN_W128);
        default: QADC_GO(SCAN_GENERIC);
    }
#undef QADC_GO
}

template <int KIND, typename QT>
static int launch_quantize(const pq_index *idx, const float *queries, const float *tables_in,
                           float *tables_out, int nq, const uint8_t *codes, int t_eff, int k,
                           const PilotPlan &plan, void *qtables, pq_qparams_t *qparams, char *gtab_out,
                           size_t gtab_stride, size_t btab_rel, char *hdr_out, uint16_t *bound_rec, hipStream_t s) {
    const bool pilot4 = pilot4_pays<KIND>(idx->h, nq, plan);
    PilotPlan pp = plan;
    if (pilot4) pp.pilot = 0;
    const size_t lds = quantize_lds(idx->h, t_eff, sizeof(QT));
    const QuantShape shape = quantize_shape(idx->h);
#define QADC_QUANT_GO(NT)                                                                                         \
    do {                                                                                                          \
        if (lds > 48 * 1024)                                                                                      \
            QADC_HIP_TRY(hipFuncSetAttribute((const void *)k_quantize<KIND, QT, NT>,                              \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));              \
        hipLaunchKernelGGL((k_quantize<KIND, QT, NT>), dim3((unsigned)nq * (unsigned)pp.P), dim3(NT), lds, s,     \
                           idx->dev, shape, \
                           idx->edesc, idx->codebooks, queries, tables_in, tables_out, codes, t_eff, k, pp.pilot, \
                           pp.slice, pp.P, qtables, qparams, gtab_out, gtab_stride, btab_rel, hdr_out, bound_rec); \
    } while (0)
    if (quantize_wide((int64_t)nq * pp.P, pp.P, t_eff, pp.pilot, KIND == SCAN_NIB8)) QADC_QUANT_GO(QUANT_WIDE); else QADC_QUANT_GO(QUANT_THREADS);
#undef QADC_QUANT_GO
    QADC_LAUNCH_CHECK("k_quantize");
    if constexpr (KIND != SCAN_GENERIC)
        if (pilot4) {
            GroupDesc gd = group_desc_args(idx->h);
            if (KIND == SCAN_W128) gd.ng = idx->h.ng / 2;
            const size_t lds4 = pilot4_lds(idx->h);
            // (mq_entry reads its table from LDS address 0: the kernel must have no static LDS)
            static const bool at_zero = [] {
                hipFuncAttributes a;
                return hipFuncGetAttributes(&a, (const void *)k_pilot4<KIND, QT>) == hipSuccess && a.sharedSizeBytes == 0;
            }();
            if (!at_zero) {
                qadc_set_error("k_pilot4: static LDS (its tables must start at LDS address 0)");
                return PQ_EHIP;
            }
            if (lds4 > 48 * 1024)
                QADC_HIP_TRY(hipFuncSetAttribute((const void *)k_pilot4<KIND, QT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds4));
            hipLaunchKernelGGL((k_pilot4<KIND, QT>), dim3((unsigned)(nq + MQ - 1) / MQ), dim3(PILOT4_THREADS), lds4, s, idx->dev, codes, k,
                               plan.pilot, qtables, idx->h.T, idx->h.gtab_len, nq, gd, qparams);
            QADC_LAUNCH_CHECK("k_pilot4");
        }
    return PQ_OK;
}

// Shared by pq_quantize_tables (queries == null) and the fused search call.  `scratch`
// (qadc_pilot_scratch_bytes(nq) bytes, 256-byte aligned, any contents) lets several blocks
// share a query's pilot; null keeps one block per query.
int qadc_quantize_launch(const pq_index *idx, const float *queries, const float *tables_in,
                         float *tables_out, int nq, const uint8_t *codes, int64_t n, int t, int R,
                         void *qtables, pq_qparams_t *qparams, char *gtab_out, size_t gtab_stride,
                         size_t btab_rel, char *hdr_out, char *scratch, PilotPlan *plan_used, hipStream_t s) {
    const int64_t want = t > 4 * (int64_t)R ? t : 4 * (int64_t)R;
    const int t_eff = (int)(n < want ? n : want);
    const int k = R < t_eff ? R : t_eff;
    PilotPlan pp = qadc_pilot_plan(nq, n, t_eff, R, scratch != nullptr,
                                   idx->h.kind == SCAN_NIB8 || idx->h.kind == SCAN_NIB16);
    if (btab_rel) {
        pp.pilot = 0;
        pp.P = 1;
    }
    if (plan_used) *plan_used = pp;
    uint16_t *bound_rec = (uint16_t *)scratch;
    const bool u8 = idx->h.acc_bits == 8;
#define QADC_GO(KIND, QT)                                                                       \
    return launch_quantize<KIND, QT>(idx, queries, tables_in, tables_out, nq, codes, t_eff, k, \
                                     pp, qtables, qparams, gtab_out, gtab_stride, btab_rel, hdr_out, bound_rec, s)
    switch (idx->h.kind) {
        case SCAN_NIB8:
            if (u8) QADC_GO(SCAN_NIB8, uint8_t); else QADC_GO(SCAN_NIB8, uint16_t);
        case SCAN_NIB16:
            if (u8) QADC_GO(SCAN_NIB16, uint8_t); else QADC_GO(SCAN_NIB16, uint16_t);
        case SCAN_W64:
            if (u8) QADC_GO(SCAN_W64, uint8_t); else QADC_GO(SCAN_W64, uint16_t);
        case SCAN_C5:
            if (u8) QADC_GO(SCAN_C5, uint8_t); else QADC_GO(SCAN_C5, uint16_t);
        case SCAN_W128:
            if (u8) QADC_GO(SCAN_W128, uint8_t); else QADC_GO(SCAN_W128, uint16_t);
        default:
            if (u8) QADC_GO(SCAN_GENERIC, uint8_t); else QADC_GO(SCAN_GENERIC, uint16_t);
    }
#undef QADC_GO
}

extern "C" int pq_quantize_tables(const pq_index_t *idx, const float *tables, int nq,
                                  const uint8_t *codes, int64_t n, int t, int R, void *qtables,
                                  pq_qparams_t *qparams, void *stream) {
    if (!idx || nq < 0 || n < 0) {
        qadc_set_error("pq_quantize_tables: bad handle, nq or n");
        return PQ_EINVAL;
    }
    if (R < 1 || R > PQ_MAX_R || t < 1) {
        qadc_set_error("pq_quantize_tables: need 1<=R<=%d and t>=1 (got R=%d t=%d)", PQ_MAX_R, R, t);
        return PQ_EINVAL;
    }
    const int64_t want = t > 4 * (int64_t)R ? t : 4 * (int64_t)R;
    if (want > PQ_MAX_T_EFF) {
        qadc_set_error("pq_quantize_tables: max(t,4R)=%lld exceeds %d", (long long)want, PQ_MAX_T_EFF);
        return PQ_EINVAL;
    }
    if (nq == 0) return PQ_OK;
    if (!tables || !qtables || !qparams || (n > 0 && !codes)) {
        qadc_set_error("pq_quantize_tables: null pointer");
        return PQ_EINVAL;
    }
    if (n > 0 && ((uintptr_t)codes & 15u) != 0) {
        qadc_set_error("pq_quantize_tables: codes must be 16-byte aligned");
        return PQ_EINVAL;
    }
    return qadc_quantize_launch(idx, nullptr, tables, nullptr, nq, codes, n, t, R, qtables, qparams,
                                nullptr, 0, 0, nullptr, nullptr, nullptr, (hipStream_t)stream);
}
