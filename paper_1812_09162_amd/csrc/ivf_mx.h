#pragma once
// One pass over an inverted list for up to sixteen of the queries that probe it, on the matrix cores
// (Section 2.1.3: every (query, cell) pair has its own tables, but the codes of the cell are the same
// for all).  16 x 4-bit codes over equal sub-spaces, 8-bit tables.
#include "quotient.h"
#include "scan_device.h"

typedef int ivf_v8i __attribute__((ext_vector_type(8)));
typedef float ivf_v4f __attribute__((ext_vector_type(4)));

// A group: up to IVF_COLS (query, probe) pairs of one cell, entries [first, first + k) of the sorted pairs.
#define IVF_COLS 16
struct __align__(16) IvfGroup {
    int32_t cell;
    uint32_t first;
    int32_t k;
    int32_t pad;
};

#define IVF_QCAP 320  // queue entries per wave: 64 are taken off when there are as many, and a tile adds up to 256
template <int DS>
struct IvfMxLds {
    uint2 onehot[16][32];             // row of nibble v, one copy per pair of banks (lane l reads copy l % 32)
    // (what the tables are made with and what the scan uses share their room)
    union __align__(16) {
        union {
            float zres[16 * DS];      // residual of the pair; then, when its tables are in registers,
            uint8_t level[256];       // its entries as 6-bit codes (mx_floor_code)
        } u[IVF_COLS];
        uint32_t queue[4][IVF_QCAP];
    };
    union __align__(16) {
        float pmin[IVF_COLS][20];
        uint32_t bt[IVF_COLS][50];    // 6-bit codes packed, three dwords per sub-quantizer
    };
    __align__(16) uint8_t qt[IVF_COLS][272];  // quantized entries (rows 4 banks apart)
    unsigned long long slot[IVF_COLS];  // slot list of the pair
    uint32_t *counts_out[IVF_COLS];
    float fdelta[IVF_COLS], fdmin[IVF_COLS];
    float thr[IVF_COLS];              // the pair's pruning bound on distances
    float top[IVF_COLS];              // ... and on sums, in the products' units: the largest key within thr; below 0: none, inf: all
    uint32_t count[IVF_COLS];
    int nqueue[4];
};

// A block of four waves serves one group.
//   1. Wave w builds the tables of pairs w, w + 4, ...: eq. (1), the quantizer against the query's d_max
//      (Section 3.4) and the quantized entries, exactly as k_ivf_scan does; and from the query's bound on
//      distances the largest key within it.
//   2. The entries, rounded DOWN to the 6-bit format (exact up to 15, within 1 up to 31 and 3 up to 60), are
//      one operand, the codes as one-hot rows of 4-bit ones the other: two products of K = 128 give the
//      sums of 16 codes for 16 pairs, exact as sums and never above the code's sum of entries.  Codes whose
//      sum is within the bound are queued.
//   3. Queued codes are summed again from the quantized entries; those within the bound on distances, with
//      their exact distance, go to the pair's slot list.  So the lists hold what k_ivf_scan's would.
// What bounds it: vector instructions and, behind them, the chain of loads that starts a block (three deep).  10^8 codes in
// 65,536 lists, 10,000 queries x 64 probes (640,000 pairs in 75,000 groups, 8.7 million tiles of 16 x 16, 6 million
// results within the bounds): the call 1609 us, 1682 with every quotient in fp64 (1240 and 1410 vector instructions a wave), when the
// kernel took 780: 370 to make tables, 250 to form rows and compare, 150 to sum queued codes again; 1544 as a pass per four pairs
// with byte-pair tables in LDS (2048 entries of eight bytes to build per group, and 1.3 random 8-byte reads per code and
// pair).  Seven waves per SIMD: with six 840, with five 920.
template <int DS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DS < 8 ? 7 : 6)))
k_ivf_scan_mx(const float *__restrict__ cb, const float *__restrict__ coarse,
              const int64_t *__restrict__ list_offsets, const uint8_t *__restrict__ list_codes,
              const int32_t *__restrict__ list_ids, const float *__restrict__ queries, int nprobe,
              char *__restrict__ ws, size_t per_query, size_t counts_off, size_t slots_off, int cap_b,
              const IvfGroup *__restrict__ gdesc, const uint32_t *__restrict__ ngroups, const uint32_t *__restrict__ order,
              const float2 *__restrict__ bounds) {
    __shared__ __align__(16) IvfMxLds<DS> S;
    if (blockIdx.x >= *ngroups) return;
    constexpr int d = 16 * DS;
    constexpr uint32_t qmax = 255;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const IvfGroup *gp = gdesc + blockIdx.x;
    const int k = gp->k, c = gp->cell;  // 1..IVF_COLS pairs of cell c, whose list is not empty
    const uint32_t first = gp->first;
    const int64_t lo = list_offsets[c], hi = list_offsets[c + 1];
    const int g = lane >> 4, pl = lane & 15;
    {
        // lane l < 16 knows pair l
        const uint32_t pair = order[first + (uint32_t)(pl < k ? pl : k - 1)];
        const uint32_t q = pair / (uint32_t)nprobe, a = pair - q * (uint32_t)nprobe;
        char *wq = ws + (size_t)q * per_query;
        const float2 bd = bounds[q];
        const float dmax = bd.x, thr0 = bd.y;
        float cv[4][DS];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < DS; ++t) cv[i][t] = cb[(lane + 64 * i) * DS + t];
        const bool two = lane + 64 < d;
        const float c0 = coarse[(size_t)c * d + lane], c1 = two ? coarse[(size_t)c * d + 64 + lane] : 0.0f;
        float z0[4], z1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float *z = queries + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)q, w + 4 * i) * d;
            z0[i] = z[lane];
            z1[i] = two ? z[64 + lane] : 0.0f;
        }
        {
            const uint64_t v = 2ull << (4 * (threadIdx.x >> 4));  // 1.0 of the 4-bit format at value threadIdx.x / 16
            *((uint4 *)&S.onehot[0][0] + threadIdx.x) = make_uint4((uint32_t)v, (uint32_t)(v >> 32), (uint32_t)v, (uint32_t)(v >> 32));
        }
        if (w == 0 && lane < IVF_COLS) {
            S.slot[lane] = (unsigned long long)((uint64_t *)(wq + slots_off) + (size_t)a * cap_b);
            S.counts_out[lane] = (uint32_t *)(wq + counts_off) + a;
            S.count[lane] = 0;
            S.thr[lane] = thr0;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            S.u[w + 4 * i].zres[lane] = __fsub_rn(z0[i], c0);
            if (two) S.u[w + 4 * i].zres[64 + lane] = __fsub_rn(z1[i], c1);
        }
        // (a wave's LDS accesses are in order, and until the barrier it uses its own pairs' rows only)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // eq. (1), terms in ascending dimension order; entry e = lane + 64 r, 16 adjacent lanes hold one sub-quantizer
        float tv[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int col = w + 4 * i;
            if (col < k) {
                float mn[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float *zz = &S.u[col].zres[(g + 4 * r) * DS];
                    float acc = 0.0f;
#pragma unroll
                    for (int t = 0; t < DS; ++t) {
                        const float diff = __fsub_rn(zz[t], cv[r][t]);
                        acc = __fadd_rn(acc, __fmul_rn(diff, diff));
                    }
                    tv[i][r] = acc;
                    mn[r] = acc;
                }
                // minima over 16 lanes (squares: the bit patterns order as integers)
#define IVF_MIN16(CTRL)                                                                                         \
    _Pragma("unroll") for (int r = 0; r < 4; ++r) mn[r] = __uint_as_float(min(__float_as_uint(mn[r]),           \
        (uint32_t)__builtin_amdgcn_update_dpp(0, __float_as_int(mn[r]), CTRL, 0xf, 0xf, true)))
                IVF_MIN16(0xB1);   // quad_perm [1,0,3,2]
                IVF_MIN16(0x4E);   // quad_perm [2,3,0,1]
                IVF_MIN16(0x141);  // row_half_mirror
                IVF_MIN16(0x140);  // row_mirror
#undef IVF_MIN16
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (pl == 0) S.pmin[col][g + 4 * r] = mn[r];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // lane i < 4: d_min (fp64, ascending) and delta of pair w + 4 i
        double dm = 0.0, dl;
        int skip;
        float vinv;
        {
            const int col = w + 4 * (lane & 3);
            const float dmx = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * col, __float_as_int(dmax)));
#pragma unroll
            for (int j = 0; j < 16; j += 4) {
                const float4 v = *(const float4 *)&S.pmin[col][j];
                dm = dm + (double)v.x;
                dm = dm + (double)v.y;
                dm = dm + (double)v.z;
                dm = dm + (double)v.w;
            }
            dl = ((double)dmx - dm) / (double)qmax;
            if (!((dl > 0.0) && isfinite(dl))) dl = 0.0;
            skip = col >= k || dm >= (double)dmx;  // Section 3.4: nothing in this list is closer than d_max
            vinv = dl > 1e-30 && dl < 1e30 ? (float)(1.0 / dl) : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int col = w + 4 * i;
            if (__builtin_amdgcn_readlane(skip, i)) {
                if (lane == 0) S.top[col] = -INFINITY;  // (its operand holds anything, sums below zero too)
                continue;
            }
            const float fdelta = __int_as_float(__builtin_amdgcn_readlane(__float_as_int((float)dl), i));
            const float fdmin = __int_as_float(__builtin_amdgcn_readlane(__float_as_int((float)dm), i));
            const float inv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vinv), i));
            // keys whose distance is within the bound (distances do not decrease with the key)
            const float thr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(thr0), col));
            int within = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) within += (int)__popcll(__ballot(fmaf((float)(lane + 64 * r), fdelta, fdmin) <= thr));
            if (lane == 0) {
                S.fdelta[col] = fdelta;
                S.fdmin[col] = fdmin;
                // (saturated codes have the largest key: if that is within the bound, all codes are)
                S.top[col] = within > (int)qmax ? INFINITY : (float)(within - 1) * 0.125f;
            }
            // floor((p - p_min) / delta) in fp32 where that cannot differ, else (or with a delta not of ordinary size,
            // inv == 0) in fp64, by the whole wave: the reads of a lane's delta want all lanes active
            uint32_t qv[4];
            bool sure = inv > 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = (tv[i][r] - S.pmin[col][g + 4 * r]) * inv;
                qv[r] = (uint32_t)fminf(x, 255.0f);
                sure = sure & quotient_sure(x, QUOTIENT_SLACK);
            }
            if (__ballot(!sure) != 0) {
                const unsigned long long db = (unsigned long long)__double_as_longlong(dl);
                const double delta = __longlong_as_double((long long)(((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(db >> 32), i) << 32) |
                                                                      (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)db, i)));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    qv[r] = 0;
                    if (delta > 0.0) {
                        const double y = floor(((double)tv[i][r] - (double)S.pmin[col][g + 4 * r]) / delta);
                        qv[r] = (y >= (double)qmax) ? qmax : (uint32_t)y;
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                S.qt[col][lane + 64 * r] = (uint8_t)qv[r];
                S.u[col].level[lane + 64 * r] = (uint8_t)mx_floor_code(qv[r]);
            }
        }
    }
    __syncthreads();
    // pack: thread t packs sub-quantizer t % 16 of pair t / 16
    {
        const int col = threadIdx.x >> 4, j = threadIdx.x & 15;
        const uint4 v = *(const uint4 *)&S.u[col].level[16 * j];
        auto four = [](uint32_t x) {  // four bytes of 6 bits to 24 bits
            return (x & 0x3fu) | ((x >> 2) & 0xfc0u) | ((x >> 4) & 0x3f000u) | ((x >> 6) & 0xfc0000u);
        };
        const uint32_t y0 = four(v.x), y1 = four(v.y), y2 = four(v.z), y3 = four(v.w);
        uint32_t *dst = &S.bt[col][3 * j];
        dst[0] = y0 | (y1 << 24);
        dst[1] = (y1 >> 8) | (y2 << 16);
        dst[2] = (y2 >> 16) | (y3 << 8);
    }
    __syncthreads();
    // a lane's part of K: code bytes g and 4 + g; of the results: rows 4 g .. 4 g + 3 of column pl
    const float top = S.top[pl];
    if (__ballot(top >= 0.0f) != 0) {  // (the same for all waves of the block)
        ivf_v8i b0, b1;
        {
            const uint2 *s0 = (const uint2 *)&S.bt[pl][6 * g], *s1 = (const uint2 *)&S.bt[pl][24 + 6 * g];
            const uint2 x0 = s0[0], x1 = s0[1], x2 = s0[2], y0 = s1[0], y1 = s1[1], y2 = s1[2];
            b0 = ivf_v8i{(int)x0.x, (int)x0.y, (int)x1.x, (int)x1.y, (int)x2.x, (int)x2.y, 0, 0};
            b1 = ivf_v8i{(int)y0.x, (int)y0.y, (int)y1.x, (int)y1.y, (int)y2.x, (int)y2.y, 0, 0};
        }
        // The list from its first even position on (16-byte loads), in blocks of 64 codes: row r of tile t is code
        // 4 r + t of the block, so a lane loads four consecutive codes and its 16 results are 16 consecutive ones.
        // Wave w takes blocks w, w + 4, ...  (Spans of 2^28 codes: a code's place in a span fits a queue entry.)
        const uint32_t rot = (uint32_t)(8 * g - 8) & 31u, mine = (uint32_t)(lane & 31) * 8u;
        const char *oh = (const char *)&S.onehot[0][0];
        uint32_t *queue = S.queue[w];
        for (int64_t lo2 = lo & ~(int64_t)1; lo2 < hi; lo2 += (int64_t)1 << 28) {
            const int len = (int)min(hi - lo2, (int64_t)1 << 28);
            const uint8_t *codes = list_codes + lo2 * 8;
            const int32_t *ids = list_ids + lo2;
            const int before = lo2 < lo ? 1 : 0;  // the first code may be the last of the list before
            int nqueue = 0;
            // the code of a queue entry: place in the span << 4 | column
            auto rescore = [&](uint32_t it) {
                const int cl = (int)it & 15, pos = (int)(it >> 4);
                if (pos < before || pos >= len) return;
                const uint2 cw = *(const uint2 *)(codes + (size_t)(uint32_t)pos * 8);
                const uint32_t id = (uint32_t)ids[pos];
                const uint8_t *qt = S.qt[cl];
                uint32_t sum = 0;
#pragma unroll
                for (int j = 0; j < 16; ++j) sum += qt[16 * j + (((j < 8 ? cw.x : cw.y) >> (4 * (j & 7))) & 15u)];
                const float dist = fmaf((float)(sum > qmax ? qmax : sum), S.fdelta[cl], S.fdmin[cl]);
                if (dist <= S.thr[cl]) {
                    const uint32_t at = atomicAdd(&S.count[cl], 1u);
                    if (at < (uint32_t)cap_b) ((uint64_t *)S.slot[cl])[at] = ((uint64_t)qadc_f2ord(dist) << 32) | id;
                }
            };
            auto queue_tile = [&](const ivf_v4f &acc, uint32_t item) {
                bool hit[4];
                uint64_t have[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    hit[i] = acc[i] <= top;
                    have[i] = __ballot(hit[i]);
                }
                if ((have[0] | have[1] | have[2] | have[3]) != 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (have[i] != 0) {
                            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(have[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)have[i], (uint32_t)nqueue));
                            if (hit[i]) queue[at] = item + (uint32_t)i * (4u << 4);
                            nqueue += (int)__popcll(have[i]);
                        }
                    while (nqueue >= 64) {
                        nqueue -= 64;
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        rescore(queue[nqueue + lane]);
                    }
                }
            };
            auto process = [&](const uint4 &x, const uint4 &y, int blk) {
                const uint32_t w0[4] = {x.x, x.z, y.x, y.z}, w1[4] = {x.y, x.w, y.y, y.w};
                const uint32_t item = ((uint32_t)(blk * 64 + 16 * g) << 4) | (uint32_t)pl;
                ivf_v4f acc[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    auto row = [&](uint32_t word) {
                        const uint32_t r = __builtin_amdgcn_alignbit(word, word, rot);  // byte g at bits 8..15
                        const uint2 l = *(const uint2 *)(oh + ((r & 0xf00u) | mine)), h = *(const uint2 *)(oh + (((r >> 4) & 0xf00u) | mine));
                        return ivf_v8i{(int)l.x, (int)l.y, (int)h.x, (int)h.y, 0, 0, 0, 0};
                    };
                    const ivf_v4f zero = {0.f, 0.f, 0.f, 0.f};
                    // formats: 4 = 4 bits (rows), 2 = 6 bits e2m3 (entries)
                    acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(row(w0[t]), b0, zero, 4, 2, 0, 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(row(w1[t]), b1, acc[t], 4, 2, 0, 0, 0, 0);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) queue_tile(acc[t], item + ((uint32_t)t << 4));
            };
            // whole blocks, the next one requested before a block is multiplied; then the last block if it is not whole,
            // codes past the end read as the last one (dropped when queued)
            const int whole = len >> 6;
            const uint8_t *base = codes + 32u * (uint32_t)pl;
            if (w < whole) {
                uint4 x = *(const uint4 *)(base + (size_t)w * 512), y = *(const uint4 *)(base + (size_t)w * 512 + 16);
                for (int blk = w; blk < whole; blk += 4) {
                    const uint8_t *next = base + (size_t)(uint32_t)(blk + 4 < whole ? blk + 4 : blk) * 512;
                    const uint4 nx = *(const uint4 *)next, ny = *(const uint4 *)(next + 16);
                    process(x, y, blk);
                    x = nx;
                    y = ny;
                }
            }
            if ((whole & 3) == w && (len & 63) != 0) {
                uint2 v[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = *(const uint2 *)(codes + (size_t)(uint32_t)min(whole * 64 + 4 * pl + t, len - 1) * 8);
                process(make_uint4(v[0].x, v[0].y, v[1].x, v[1].y), make_uint4(v[2].x, v[2].y, v[3].x, v[3].y), whole);
            }
            // what the four queues hold, by all waves together
            if (lane == 0) S.nqueue[w] = nqueue;
            __syncthreads();
            const int n0 = S.nqueue[0], n1 = n0 + S.nqueue[1], n2 = n1 + S.nqueue[2], n3 = n2 + S.nqueue[3];
            for (int i = threadIdx.x; i < n3; i += 256) {
                const int wq = (i >= n0 ? 1 : 0) + (i >= n1 ? 1 : 0) + (i >= n2 ? 1 : 0);
                rescore(S.queue[wq][i - (wq == 0 ? 0 : (wq == 1 ? n0 : (wq == 2 ? n1 : n2)))]);
            }
            __syncthreads();
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < k) *S.counts_out[threadIdx.x] = S.count[threadIdx.x];  // uncapped, as in k_ivf_scan
}
