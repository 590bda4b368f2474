#pragma once
// Batched exhaustive scan on the matrix cores (eq. (2) for many queries at once).
//
// The sum of a code's table entries is a row of zeros and ones (the code's sub-codes, one-hot)
// times a column of table entries, so a batch of queries over a list of codes is a matrix product
// [codes x K] x [K x queries], K = the table length.  The one-hot rows cost a shift or two per
// sub-code and the product runs at the full rate of the 4- and 6-bit formats.  The entries are held
// in the 6-bit format e2m3 (32 values, 0..60 in units of 1/8), rounded DOWN, of the quantized
// entry's level: entries and keys are scaled, per query, by a factor (mx_level) that leaves the range of the
// keys 255 levels or, where the R-th key is expected near its top, brings that key to 160.  Small entries, which
// is what codes near the result have, lose little, the sum is exact, and it bounds the level of the code's
// unsaturated sum, its key unless that is q_max, from below.
//
//   k_scan_mx  writes, per query, the smallest such sum of every group of 64 codes (one byte; sums
//              above 255 as 255) and nothing else: no bound, no compare, no atomic.
//   k_pick     one block per query: the R-th smallest group minimum names about R groups; the exact
//              keys of their codes give an upper bound on the R-th key, and every code that could
//              be within it lies in a group whose minimum is within it.  Those codes' exact keys are
//              computed from the group tables, and the R smallest (key, id) are written.
//
// What bounds it: the matrix cores, and beside them the vector units (minima, row addresses), which overlap them in part
// where both alternate in a wave's stream.  16 x 4 bits, K = 256: four products of 64 (32 clocks each) and eight
// three-operand minima per 32 x 32 results.  10^7 codes, 256 queries, by counters: matrix cores busy 312,400 of the 423,800 cycles in which a CU has
// waves (74 %), vector instructions (37.8 million besides the products) 148,000.  Kernel times from a trace of 12 calls: 236 us, of which the uneven
// end of 2442 blocks, two to a CU, is a tenth (940 us as look-ups in LDS, k_scan_mq); back to back the whole call takes 235.  32 queries:
// 41 and 165 us; {6,6,4} x 4, 32 queries: 69 and 230 us (81 with the minima behind all products of a tile; 110 with the one-hot
// rows shifted together on the vector units).  k_pick: 16 us for
// 32 queries, 24 for 256 (it replaces the quantizer's pilot and k_final: 95 + 16 us at 256 queries).
#include <string.h>

#include "scan_device.h"

typedef int mx_v8i __attribute__((ext_vector_type(8)));
typedef float mx_v16f __attribute__((ext_vector_type(16)));

// The fields of every product step, by value (uniform).
struct MxDesc {
    int32_t type[MX_MAX_STEPS], off[MX_MAX_STEPS][2], off2[MX_MAX_STEPS][2];
};

// byte N of w times 16 (the byte offset of a 16-byte table entry), as one instruction
template <int N>
__device__ __forceinline__ uint32_t mx_byte_x16(uint32_t w, uint32_t four) {
    uint32_t r;
    if (N == 0)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(four), "v"(w));
    else if (N == 1)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(four), "v"(w));
    else if (N == 2)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(four), "v"(w));
    else
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(four), "v"(w));
    return r;
}

// A lane's half of the one-hot row: 32 values of 4 bits, the value 1.0 being the bit pattern 2.
struct MxRow {
    uint64_t lo, hi;
};
// two nibbles, as shift amounts 4 * nibble (the hardware takes the low six bits of an amount)
__device__ __forceinline__ MxRow mx_row_nibbles(uint32_t amt0, uint32_t amt1) {
    MxRow r;
    r.lo = 2ull << (amt0 & 63u);
    r.hi = 2ull << (amt1 & 63u);
    return r;
}
// a 5-bit field: 1.0 at value x & 31, z = 2 (or 0: an empty row)
__device__ __forceinline__ MxRow mx_row_five(uint32_t x, uint64_t z) {
    const uint64_t y = z << ((x << 2) & 63u);
    const uint32_t m = (uint32_t)((int32_t)(x << 27) >> 31);  // all ones if bit 4 is set
    const uint32_t y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
    MxRow r;
    r.lo = ((uint64_t)(y1 & ~m) << 32) | (y0 & ~m);
    r.hi = ((uint64_t)(y1 & m) << 32) | (y0 & m);
    return r;
}

// The codes of a lane for four tiles (row c of tile t is code base + 4 c + t), as each kind needs
// them: NIB8 one dword per code (the half's four bytes), NIB16 two, the irregular kinds whole codes.
template <int KIND>
struct MxCodes {
    static constexpr int W = KIND == SCAN_NIB8 ? 1 : (KIND == SCAN_W128 ? 4 : 2);
    uint32_t w[4][W];
    // requested first, arranged when used: the request alone must not wait
    uint4 raw[KIND == SCAN_NIB8 ? 2 : (KIND == SCAN_C5 ? 2 : (KIND == SCAN_W64 ? 2 : (KIND == SCAN_NIB16 ? 2 : 4)))];
    __device__ __forceinline__ void request(const uint8_t *__restrict__ codes, int64_t first, int h) {
        if (KIND == SCAN_NIB8 || KIND == SCAN_W64) {
            const uint4 *p = (const uint4 *)(codes + first * 8);
            raw[0] = p[0];
            raw[1] = p[1];
        } else if (KIND == SCAN_NIB16) {
            const uint2 *p = (const uint2 *)(codes + first * 16) + h;
            const uint2 a = p[0], b = p[2], c = p[4], d = p[6];
            raw[0] = make_uint4(a.x, a.y, b.x, b.y);
            raw[1] = make_uint4(c.x, c.y, d.x, d.y);
        } else if (KIND == SCAN_C5) {
            const uint32_t *p = (const uint32_t *)(codes + first * 5);
            raw[0] = make_uint4(p[0], p[1], p[2], p[3]);
            raw[1].x = p[4];
        } else {
            const uint4 *p = (const uint4 *)(codes + first * 16);
#pragma unroll
            for (int t = 0; t < 4; ++t) raw[KIND == SCAN_W128 ? t : 0] = p[t];
        }
    }
    __device__ __forceinline__ void arrange(int h) {
        if constexpr (KIND == SCAN_NIB8) {
            w[0][0] = h ? raw[0].y : raw[0].x;
            w[1][0] = h ? raw[0].w : raw[0].z;
            w[2][0] = h ? raw[1].y : raw[1].x;
            w[3][0] = h ? raw[1].w : raw[1].z;
        } else if constexpr (KIND == SCAN_W64 || KIND == SCAN_NIB16) {
            w[0][0] = raw[0].x; w[0][1] = raw[0].y; w[1][0] = raw[0].z; w[1][1] = raw[0].w;
            w[2][0] = raw[1].x; w[2][1] = raw[1].y; w[3][0] = raw[1].z; w[3][1] = raw[1].w;
        } else if constexpr (KIND == SCAN_C5) {
            // code t = bits [40 t, 40 t + 40) of the 20 bytes
            w[0][0] = raw[0].x;
            w[0][1] = raw[0].y & 0xffu;
            w[1][0] = __builtin_amdgcn_alignbit(raw[0].z, raw[0].y, 8);
            w[1][1] = (raw[0].z >> 8) & 0xffu;
            w[2][0] = __builtin_amdgcn_alignbit(raw[0].w, raw[0].z, 16);
            w[2][1] = (raw[0].w >> 16) & 0xffu;
            w[3][0] = __builtin_amdgcn_alignbit(raw[1].x, raw[0].w, 24);
            w[3][1] = raw[1].x >> 24;
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                w[t][0] = raw[t].x; w[t][1] = raw[t].y; w[t][2] = raw[t].z; w[t][3] = raw[t].w;
            }
        }
    }
};

// ------------------------------------------------------------- k_scan_mx ---
// A wave scans a chunk of gpc * nb * 128 codes against 32 * NCOL queries (blockIdx.y): the queries'
// tables stay in its registers, the codes stream through in blocks of 128 (four tiles of 32 rows,
// four consecutive codes per row), the next block requested before the current one is multiplied.
// Lane (c, h) of a 32 x 32 result holds 16 codes of query column c; their minimum over nb blocks is
// one group.  A chunk's gpc group minima of a lane are stored together: row of query q = [chunk]
// [h][gpc] bytes.  S product steps of 64 table entries; a lane half holds 32 of them.
// PAT: the kinds of the steps (of each 64-bit word) at compile time, 100 N6 + 10 N5 + N4: N6 steps of
// 6-bit fields, then N5 of 5-bit ones, then N4 of nibbles; 0: read from the descriptors.
// Three query tiles of 16 x 4-bit codes: minima are stored four at a time, not sixteen, whose nine registers
// would leave a SIMD two waves instead of three (2 * 10^7 codes, us a call: 96 queries 191, held 194; 192 342 and 349.
// One, two and four tiles keep their waves either way, and are up to 3 % slower with more stores).
constexpr bool mx_each(int kind, int ncol) { return kind == SCAN_NIB8 && ncol == 3; }
template <int KIND, int S, int NCOL, int PAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KIND == SCAN_W128 ? 1 : (mx_each(KIND, NCOL) ? 3 : 2))))
k_scan_mx(const uint8_t *__restrict__ codes, int nchunks, int gpc, int nb, char *__restrict__ ws,
          size_t per_query, size_t btab_off, size_t min_off, int nq, MxDesc md) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / QADC_WAVE), l = threadIdx.x % QADC_WAVE;
    const int c = l & 31, h = l >> 5;
    const int q0 = blockIdx.y * (32 * NCOL);
    uint32_t b[NCOL][S][6];
#pragma unroll
    for (int ct = 0; ct < NCOL; ++ct) {
        const int q = q0 + ct * 32 + c < nq ? q0 + ct * 32 + c : nq - 1;  // (columns past the batch are not stored)
        const uint2 *src = (const uint2 *)(ws + (size_t)q * per_query + btab_off) + 3 * h;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const uint2 v = src[s * 6 + i];
                b[ct][s][2 * i] = v.x;
                b[ct][s][2 * i + 1] = v.y;
            }
    }
    // One-hot rows from tables in LDS (16 bytes per entry; the reads run beside the products, which
    // shifts and selects on the vector units do not): m x 4: a byte's two nibbles; irregular kinds of
    // known pattern: a 6-bit field's half h (entries 64 h + field), which for fields below 32 is also a
    // 5-bit field's row.
    constexpr bool NIB = KIND == SCAN_NIB8 || KIND == SCAN_NIB16;
    constexpr bool LUT = NIB || PAT != 0;
    __shared__ __align__(16) uint4 lut[NIB ? 256 : (LUT ? 128 : 1)];
    if constexpr (NIB) {
        const uint64_t a = 2ull << (4 * (threadIdx.x & 15u)), d = 2ull << (4 * (threadIdx.x >> 4));
        lut[threadIdx.x] = make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)d, (uint32_t)(d >> 32));
        __syncthreads();
    } else if constexpr (LUT) {
        if (threadIdx.x < 128) {
            const uint32_t x = threadIdx.x & 63u;
            const uint64_t y = (x >> 5) == (threadIdx.x >> 6) ? 2ull << (4 * (x & 15u)) : 0ull;
            const bool up = (x & 16u) != 0;
            lut[threadIdx.x] = make_uint4(up ? 0u : (uint32_t)y, up ? 0u : (uint32_t)(y >> 32), up ? (uint32_t)y : 0u, up ? (uint32_t)(y >> 32) : 0u);
        }
        __syncthreads();
    }
    const uint32_t four = 4, hbase = h ? 1024u : 0u;
    const int nblk = gpc * nb;
    const uint32_t hz = h ? 0u : 2u;
    // irregular kinds: bit offset of the half's field | offset of its second nibble << 6; of fields read
    // through the table: the rotation that brings them to bit 4
    uint32_t offs[S];
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (PAT != 0 && s % (KIND == SCAN_W128 ? S / 2 : S) < PAT / 100 + PAT / 10 % 10)
            offs[s] = (uint32_t)((h ? md.off[s][1] : md.off[s][0]) + 28) & 31u;
        else
            offs[s] = h ? (uint32_t)(md.off[s][1] | md.off2[s][1] << 6) : (uint32_t)(md.off[s][0] | md.off2[s][0] << 6);
    // A lane's row of product step s for tile t of a block of codes.
    auto row_of = [&](const MxCodes<KIND> &cd, int t, int s) {
        const uint32_t *w = cd.w[t];
        if constexpr (NIB) {
            const uint32_t x = w[s >> 2];
            uint32_t at;
            switch (s & 3) {
                case 0: at = mx_byte_x16<0>(x, four); break;
                case 1: at = mx_byte_x16<1>(x, four); break;
                case 2: at = mx_byte_x16<2>(x, four); break;
                default: at = mx_byte_x16<3>(x, four); break;
            }
            return *(const uint4 *)((const char *)lut + at);
        } else {
            // (128-bit codes: the steps of the upper word follow those of the lower)
            constexpr int HS = KIND == SCAN_W128 ? S / 2 : S;
            constexpr int W0 = MxCodes<KIND>::W - 2;
            const uint32_t lo = s < HS ? w[0] : w[W0], hi = s < HS ? w[1] : w[W0 + 1];
            constexpr int N6 = PAT / 100, N5 = PAT / 10 % 10;
            const int sw = s % HS;
            if (PAT != 0 && sw < N6 + N5) {
                // the field, rotated to bit 4 of its dword: the steps of a kind are in the order of
                // the code, half of them in each dword (40-bit codes: all in the lower)
                const bool upper = KIND != SCAN_C5 && (sw < N6 ? 2 * sw >= N6 : 2 * (sw - N6) >= N5);
                const uint32_t x = upper ? hi : lo;
                const uint32_t r = __builtin_amdgcn_alignbit(x, x, offs[s]);
                const uint32_t at = sw < N6 ? ((r & 0x3f0u) | hbase) : (r & 0x1f0u);
                return *(const uint4 *)((const char *)lut + at);
            } else {
                const uint64_t v = ((uint64_t)hi << 32) | lo;
                const int type = PAT == 0 ? md.type[s] : MX_NIBBLES;
                const uint32_t x = (uint32_t)(v >> (offs[s] & 63u));
                MxRow y;
                if (type == MX_SIX)
                    y = mx_row_five(x, ((x >> 4) & 2u) ^ hz);
                else if (type == MX_FIVE)
                    y = mx_row_five(x, 2);
                else
                    y = mx_row_nibbles(x << 2, (uint32_t)(v >> ((offs[s] >> 6) & 63u)) << 2);
                return make_uint4((uint32_t)y.lo, (uint32_t)(y.lo >> 32), (uint32_t)y.hi, (uint32_t)(y.hi >> 32));
            }
        }
    };
    auto minima_of = [&](int ct, int ch) {  // this lane's part of a chunk: gpc bytes of query column ct * 32 + c
        return ws + (size_t)(q0 + ct * 32 + c) * per_query + min_off + (size_t)ch * (2 * gpc) + h * gpc;
    };
    // Rows held: a tile's, which every query tile multiplies; with one query tile and many steps only the next eight, as the
    // others' registers would leave a SIMD one wave ({6,6,4} x 8, 2 * 10^7 codes, 32 queries, us a call: 382, with all of a tile's 430).
    constexpr int H = NCOL == 1 && S > 16 ? 8 : S;
    static_assert(4 * S % H == 0, "a block of codes starts with the first of the rows held");
    for (int ch = blockIdx.x * 4 + wave; ch < nchunks; ch += gridDim.x * 4) {
        const int64_t first = (int64_t)ch * nblk * 128 + 4 * c;
        MxCodes<KIND> cur, nxt;
        cur.request(codes, first, h);
        uint32_t mn[NCOL], pk[NCOL][4];
#pragma unroll
        for (int ct = 0; ct < NCOL; ++ct) {
            mn[ct] = 0x7f7fffffu;
#pragma unroll
            for (int i = 0; i < 4; ++i) pk[ct][i] = 0;
        }
        int inb = 0, gi = 0;
        cur.arrange(h);
        uint4 row[H];
#pragma unroll
        for (int s = 0; s < H; ++s) row[s] = row_of(cur, 0, s);
        for (int blk = 0; blk < nblk; ++blk) {
            nxt.request(codes, first + (int64_t)(blk + 1 < nblk ? blk + 1 : blk) * 128, h);
            // Units (tile, query tile) in turn on two accumulators: between the products of one, the minima of the
            // one before (sums are >= 0: their bit patterns order as integers) and, in a tile's last unit, the
            // rows H steps on: those of the next tile.  Products and vector instructions overlap on this chip where they alternate in
            // a wave's stream (four products 131 clocks, 32 minima 140, alternating 175, one after the other 271).
            mx_v16f acc[2];
            auto minima = [&](const mx_v16f &a, uint32_t &m, int p) {
                m = min(m, min(__float_as_uint(a[2 * p]), __float_as_uint(a[2 * p + 1])));
            };
#pragma unroll
            for (int u = 0; u < 4 * NCOL; ++u) {
                const int t = u / NCOL, ct = u % NCOL, before = (u + NCOL - 1) % NCOL;
                if (t == 3 && ct == NCOL - 1) nxt.arrange(h);
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    uint4 &r = row[(t * S + s) % H];
                    const mx_v8i a = {(int)r.x, (int)r.y, (int)r.z, (int)r.w, 0, 0, 0, 0};
                    const uint32_t *bs = b[ct][s];
                    const mx_v8i bv = {(int)bs[0], (int)bs[1], (int)bs[2], (int)bs[3], (int)bs[4], (int)bs[5], 0, 0};
                    const mx_v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    // formats: 4 = 4 bits (one-hot rows), 2 = 6 bits e2m3 (tables)
                    acc[u & 1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, bv, s == 0 ? zero : acc[u & 1], 4, 2, 0, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (ct == NCOL - 1) {
                        if (s + H < S) r = row_of(cur, t, s + H);
                        else r = t < 3 ? row_of(cur, t + 1, s + H - S) : row_of(nxt, 0, s + H - S);
                    }
                    if (u > 0 && s > 0) {  // (the last product of the unit before needs a step or two to finish)
#pragma unroll
                        for (int p = 8 * (s - 1) / (S - 1); p < 8 * s / (S - 1); ++p) minima(acc[(u + 1) & 1], mn[before], p);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int p = 0; p < 8; ++p) minima(acc[1], mn[NCOL - 1], p);
            if (++inb == nb) {
                inb = 0;
#pragma unroll
                for (int ct = 0; ct < NCOL; ++ct) {
                    const uint32_t u = (uint32_t)fminf(__uint_as_float(mn[ct]) * 8.0f, 255.0f);
                    pk[ct][3] = (pk[ct][3] >> 8) | (u << 24);
                    mn[ct] = 0x7f7fffffu;
                }
                if constexpr (mx_each(KIND, NCOL)) {
                    if ((++gi & 3) == 0) {
#pragma unroll
                        for (int ct = 0; ct < NCOL; ++ct)
                            if (q0 + ct * 32 + c < nq) *(uint32_t *)(minima_of(ct, ch) + gi - 4) = pk[ct][3];
                    }
                } else if ((++gi & 3) == 0 && gi < gpc) {
#pragma unroll
                    for (int ct = 0; ct < NCOL; ++ct) {
                        pk[ct][0] = pk[ct][1];
                        pk[ct][1] = pk[ct][2];
                        pk[ct][2] = pk[ct][3];
                    }
                }
            }
            cur = nxt;
        }
        if constexpr (!mx_each(KIND, NCOL)) {
#pragma unroll
            for (int ct = 0; ct < NCOL; ++ct)
                if (q0 + ct * 32 + c < nq) {
                    if (gpc == 16)
                        *(uint4 *)minima_of(ct, ch) = make_uint4(pk[ct][0], pk[ct][1], pk[ct][2], pk[ct][3]);
                    else
                        *(uint32_t *)minima_of(ct, ch) = pk[ct][3];
                }
        }
    }
}

// ---------------------------------------------------------------- k_pick ---
// smallest byte of a dword pair-wise: the two 16-bit halves hold the minima of the even and odd bytes
typedef unsigned short mx_u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pick_min_bytes(uint32_t x, uint32_t m) {
    const mx_u16x2 e = __builtin_bit_cast(mx_u16x2, x & 0x00ff00ffu), o = __builtin_bit_cast(mx_u16x2, (x >> 8) & 0x00ff00ffu);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_elementwise_min(e, o), __builtin_bit_cast(mx_u16x2, m)));
}

// Exact key of code id from the group tables in LDS.  Irregular kinds with at most eight groups (per
// 64-bit half) take the group descriptors as kernel arguments; gd.ng == 0: from the layout.
template <int KIND, typename QT>
__device__ __forceinline__ uint32_t pick_key(const DevLayout *L, const GroupDesc &gd, const QT *gtab,
                                             const uint8_t *__restrict__ codes, int64_t id, int64_t n) {
    constexpr uint32_t qmax = sizeof(QT) == 1 ? 255u : 65535u;
    if constexpr (KIND == SCAN_W64 || KIND == SCAN_C5 || KIND == SCAN_W128) {
        if (gd.ng > 0) {
            uint32_t s;
            if constexpr (KIND == SCAN_W64) {
                const uint2 w = *(const uint2 *)(codes + id * 8);
                s = sum_groups_flight(gd, gtab, w.x, w.y);
            } else if constexpr (KIND == SCAN_C5) {
                // the two aligned dwords that hold the code (the last code of the array: byte by byte)
                if (id + 1 >= n) return key_at<KIND, QT>(L, gtab, codes, id);
                const int64_t at = id * 5;
                const uint32_t *p = (const uint32_t *)(codes + (at & ~(int64_t)3));
                const uint64_t w = (((uint64_t)p[1] << 32) | p[0]) >> (8 * ((uint32_t)at & 3u));
                // (five groups as eight cost more than they gained: 2 * 10^6 codes, 20 queries 47.2 us a call with a branch per group, 48.7 as eight, 44.9)
                const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32) & 0xffu;
                s = gd.ng <= 5 ? sum_groups_flight<5>(gd, gtab, lo, hi) : sum_groups_flight(gd, gtab, lo, hi);
            } else {
                const uint4 w = *(const uint4 *)(codes + id * 16);
                s = sum_groups_flight(gd, gtab, w.x, w.y) + sum_groups_flight(gd, gtab, w.z, w.w, true);
            }
            return s > qmax ? qmax : s;
        }
    }
    return key_at<KIND, QT>(L, gtab, codes, id);
}

// A block's time is a chain of memory round trips and barriers: a query's minima are read once, UB
// 16-byte units per thread in flight (their smallest bytes stay in registers when that is all of
// them), and the exact keys are computed once, of the groups a little above the bound; only when
// these do not hold R codes within that margin are they computed again around an exact bound.
template <int KIND, typename QT, int NT, int ACAP>
__global__ void __launch_bounds__(NT)
k_pick(const DevLayout *__restrict__ L, const pq_qparams_t *__restrict__ qparams,
       const uint8_t *__restrict__ codes, int64_t n, int R, const char *__restrict__ ws, size_t per_query,
       size_t gtab_off, size_t min_off, int lgpc, int lnb, int nmin, int margin, int gtab_len, GroupDesc gd,
       int32_t *__restrict__ out_ids, uint16_t *__restrict__ out_keys, float *__restrict__ out_dist) {
    extern __shared__ __align__(16) unsigned char smem[];
    typedef SelectLds<NT, ACAP> Lds;
    Lds &S = *(Lds *)smem;
    QT *gtab = (QT *)(smem + sizeof(Lds));
    // until the ranking, the room of its histograms lists groups, and that of
    // its order the 16-byte units of minima they come from
    constexpr int LIST = NT / 64 * 256, ULIST = ACAP / 2;
    uint32_t *list = &S.whist[0][0], *ulist = (uint32_t *)S.order;
    constexpr int SEG = LIST / 16 < ULIST ? LIST / 16 : ULIST;  // units whose groups the lists surely hold
    const size_t q = blockIdx.x;
    const char *wq = ws + q * per_query;
    constexpr int shift = sizeof(QT) == 1 ? 0 : 8;  // (key bins of the ranking)
    const uint32_t qmax = sizeof(QT) == 1 ? 255u : 65535u;
    const uint32_t scale = ((const ScanHdr *)wq)->scale;
    // the largest key of a level (level 255 stands for all above as well)
    auto last_key = [scale, qmax](uint32_t level) { return level >= 255u ? qmax : min((((level + 1) << 16) - 1u) / scale, qmax); };
    const uint4 *row = (const uint4 *)(wq + min_off);
    const int units = (nmin + 15) >> 4;
    constexpr int UB = 10;
    uint32_t um[UB];  // smallest minimum of unit u0 + thread + k * NT; units at or beyond u1: none
    auto load_units = [&](int u0, int u1) {
        uint4 v[UB];
#pragma unroll
        for (int k = 0; k < UB; ++k) {
            const int u = u0 + k * NT + (int)threadIdx.x;
            v[k] = u < u1 ? row[u] : make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
            if (u == units - 1 && (nmin & 15) != 0) v[k].z = v[k].w = 0xffffffffu;  // (nmin is a multiple of 8)
        }
#pragma unroll
        for (int k = 0; k < UB; ++k) {
            uint32_t m = pick_min_bytes(v[k].x, 0xffffffffu);
            m = pick_min_bytes(v[k].y, m);
            m = pick_min_bytes(v[k].z, m);
            m = pick_min_bytes(v[k].w, m);
            um[k] = u0 + k * NT + (int)threadIdx.x < u1 ? min(m & 0xffffu, m >> 16) : 0xffffffffu;
        }
    };
    const bool kept = units <= UB * NT;  // all units' minima are in the registers, for good
    const pq_qparams_t prm = qparams[q];
    {
        const int n16 = (gtab_len * (int)sizeof(QT) + 15) >> 4;
        for (int i = threadIdx.x; i < n16; i += NT) ((uint4 *)gtab)[i] = ((const uint4 *)(wq + gtab_off))[i];
    }
    load_units(0, units);
    for (int i = threadIdx.x; i < 256; i += NT) S.hist[i] = 0;
    if (threadIdx.x < 4) S.sh[threadIdx.x] = 0;  // 0: entries in A, 1: overflow of A, 2: groups listed, 3: units listed
    __syncthreads();
    // the bin of the kk-th smallest counted value (255 if fewer were counted), and in S.sh[5] how many
    // values lie in the bins below it
    auto select_bin = [&](uint32_t kk) {
        __syncthreads();
        if (threadIdx.x < QADC_WAVE) qadc_wave_select_bin(S.hist, kk, 0u, S.sh + 4);
        __syncthreads();
        return S.sh[4];
    };
    // 1. the R-th smallest of the units' minima: an upper bound on the R-th smallest group minimum (and
    //    close to it: the few groups within it are spread over many more units).  With few units for
    //    the R results the groups' minima are counted themselves.
    if (units < 4 * R) {
        for (int g = threadIdx.x; g < nmin; g += NT) atomicAdd(&S.hist[((const uint8_t *)row)[g]], 1u);
    } else {
        for (int u0 = 0; u0 < units; u0 += UB * NT) {
            if (u0) load_units(u0, units);
#pragma unroll
            for (int k = 0; k < UB; ++k)
                if (um[k] <= 255u) atomicAdd(&S.hist[um[k]], 1u);
        }
    }
    const uint32_t b0 = select_bin((uint32_t)R);
    const int64_t tail0 = (int64_t)(nmin / 2) << (7 + lnb);  // codes behind the last whole chunk
    // f(id, key) for every code of the groups with a minimum within thr, and of the tail
    auto each_code = [&](uint32_t thr, auto f) {
        bool whole = true;
        for (int ua = 0; ua < units;) {
            // all units at once, or (a crowd of equal minima) as many as the lists surely hold
            const int ub = whole || ua + SEG > units ? units : ua + SEG;
            __syncthreads();
            if (threadIdx.x < 2) S.sh[2 + threadIdx.x] = 0;
            __syncthreads();
            for (int u0 = ua; u0 < ub; u0 += UB * NT) {
                if (!kept) load_units(u0, ub);
#pragma unroll
                for (int k = 0; k < UB; ++k) {
                    const int u = (kept ? 0 : u0) + k * NT + (int)threadIdx.x;
                    if (um[k] <= thr && u >= ua && u < ub) {
                        const int pos = (int)atomicAdd(&S.sh[3], 1u);
                        if (pos < ULIST) ulist[pos] = (uint32_t)u;
                    }
                }
                if (kept) break;
            }
            __syncthreads();
            const int nu = (int)S.sh[3];
            if (nu <= ULIST)
                for (int i = threadIdx.x; i < 16 * nu; i += NT) {
                    const uint32_t g = ulist[i >> 4] * 16u + (uint32_t)(i & 15);
                    const uint32_t m = (int)g < nmin ? (uint32_t)((const uint8_t *)row)[g] : 0xffffffffu;
                    if (m <= thr) {
                        const int pos = (int)atomicAdd(&S.sh[2], 1u);
                        if (pos < LIST) list[pos] = g;
                    }
                }
            __syncthreads();
            const int cnt = (int)S.sh[2];
            if (nu > ULIST || cnt > LIST) {
                whole = false;
                continue;
            }
            const int total = cnt << (6 + lnb);
            constexpr int U = KIND == SCAN_NIB16 || KIND == SCAN_W128 ? 4 : 6;  // codes per thread in flight
            for (int e0 = threadIdx.x; e0 < total; e0 += U * NT) {
                int64_t id[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * NT < total ? e0 + u * NT : total - 1;
                    const int g = (int)list[e >> (6 + lnb)], blk = (e >> 6) & ((1 << lnb) - 1), j = e & 63;
                    const int chunk = g >> (lgpc + 1), hh = (g >> lgpc) & 1, i = g & ((1 << lgpc) - 1);
                    id[u] = ((((int64_t)chunk << lgpc) + i) << (7 + lnb)) + blk * 128 + 16 * (2 * (j >> 4) + hh) + (j & 15);
                }
                uint32_t key[U];
#pragma unroll
                for (int u = 0; u < U; ++u) key[u] = pick_key<KIND, QT>(L, gd, gtab, codes, id[u], n);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (e0 + u * NT < total) f((uint32_t)id[u], key[u]);
            }
            ua = ub;
        }
        for (int64_t id = tail0 + threadIdx.x; id < n; id += NT) f((uint32_t)id, pick_key<KIND, QT>(L, gd, gtab, codes, id, n));
    };
    auto keep = [&](uint32_t id, uint32_t key) {
        const uint32_t pos = atomicAdd(&S.sh[0], 1u);
        if (pos < (uint32_t)ACAP) S.A[pos] = ((uint64_t)key << 32) | id; else S.sh[1] = 1u;
    };
    // 2. the codes within a margin above that minimum.  Every code whose unsaturated sum's level is within
    //    `top` is in a group whose minimum is.  A key below q_max is that sum.  A saturated code's sum can be
    //    larger than its key, and where entries are scaled so that q_max has a level below 255, its sum of levels
    //    too: such codes are left out here, and if R are found without them the result is among those.
    const uint32_t most = mx_level(qmax, scale) < 255u ? qmax - 1u : qmax;  // the largest key that a minimum bounds
    const uint32_t top = min(b0 + (b0 >> 5) + (uint32_t)(scale == 65536u ? 1 : margin), 255u);
    uint32_t bound = min(min(last_key(top), most), prm.key_bound);
    each_code(top, [&](uint32_t id, uint32_t key) { if (key <= bound) keep(id, key); });
    __syncthreads();
    int na = (int)S.sh[0];
    bool over = S.sh[1] != 0;
    if (na < R || over) {
        // 3. exactly: the R-th smallest key among the groups up to the R-th bounds the R-th key
        __syncthreads();
        for (int i = threadIdx.x; i < 256; i += NT) S.hist[i] = 0;
        if (threadIdx.x < 2) S.sh[threadIdx.x] = 0;
        each_code(b0, [&](uint32_t, uint32_t key) { atomicAdd(&S.hist[min(mx_level(key, scale), 255u)], 1u); });
        const uint32_t bin = select_bin((uint32_t)R);
        bound = last_key(bin);
        const uint32_t lo = bin > 0 ? last_key(bin - 1) + 1u : 0u, width = bound - lo + 1u;
        if (width > 1) {  // a level is many keys, and where keys are close together many codes: 256 parts of it
            const uint32_t kk = (uint32_t)R - S.sh[5];
            __syncthreads();
            for (int i = threadIdx.x; i < 256; i += NT) S.hist[i] = 0;
            each_code(b0, [&](uint32_t, uint32_t key) {
                if (key >= lo && key <= bound) atomicAdd(&S.hist[((key - lo) << 8) / width], 1u);
            });
            const uint32_t part = select_bin(kk);
            bound = lo + (uint32_t)(((uint64_t)(part + 1) * width - 1u) >> 8);
        }
        bound = min(bound, prm.key_bound);
        over = bound > most;  // the R-th key may be a saturated one: the lowest ids of any group belong to it
        if (!over) {
            each_code(bin, [&](uint32_t id, uint32_t key) { if (key <= bound) keep(id, key); });
            __syncthreads();
            na = (int)S.sh[0];
            over = S.sh[1] != 0;
        }
        if (over) {  // ... or more equal keys than the block can rank
            __syncthreads();
            exact_select<KIND, QT>(L, gtab, codes, n, R, S.A, S.hist, S.sh);
            __syncthreads();
            na = (int)S.sh[2];
            __syncthreads();
        }
    }
    FinalOut o;
    o.ids = out_ids + q * R;
    o.keys = out_keys + q * R;
    o.dist = out_dist + q * R;
    rank_and_write<NT, ACAP>(S, na, R, prm, qmax, o, shift);
}

// ------------------------------------------------------------------ host ---
// 32-query tiles a wave's registers hold
static constexpr int mx_most(int kind, bool known_pattern) {
    return kind == SCAN_NIB8 ? 4 : (kind == SCAN_NIB16 ? 2 : (!known_pattern ? 1 : (kind == SCAN_C5 ? 3 : 2)));
}
template <int KIND, int S, int NCOL, int PAT>
static void mx_go(const DevLayout &h, const MxPlan &p, int nq, const uint8_t *codes, char *ws, size_t per_query, hipStream_t s) {
    MxDesc md;
    memcpy(md.type, h.mx_type, sizeof(md.type));
    memcpy(md.off, h.mx_off, sizeof(md.off));
    memcpy(md.off2, h.mx_off2, sizeof(md.off2));
    const int cpw = p.gpc == 16 ? 1 : 4;  // chunks per wave
    const unsigned gx = (unsigned)((p.nchunks + 4 * cpw - 1) / (4 * cpw));
    hipLaunchKernelGGL((k_scan_mx<KIND, S, NCOL, PAT>), dim3(gx, p.groups), dim3(256), 0, s, codes, p.nchunks, p.gpc, p.nb, ws,
                       per_query, p.btab_off, p.min_off, nq, md);
}

template <int KIND, int S, int PAT = 0>
static void mx_cols(const DevLayout &h, const MxPlan &p, int nq, const uint8_t *codes, char *ws, size_t per_query, hipStream_t s) {
    constexpr int most = mx_most(KIND, PAT != 0);
    if constexpr (most >= 4)
        if (p.ncol == 4) return mx_go<KIND, S, 4, PAT>(h, p, nq, codes, ws, per_query, s);
    if constexpr (most >= 3)
        if (p.ncol == 3) return mx_go<KIND, S, 3, PAT>(h, p, nq, codes, ws, per_query, s);
    if constexpr (most >= 2)
        if (p.ncol == 2) return mx_go<KIND, S, 2, PAT>(h, p, nq, codes, ws, per_query, s);
    mx_go<KIND, S, 1, PAT>(h, p, nq, codes, ws, per_query, s);
}

template <int KIND>
static void mx_steps(const DevLayout &h, const MxPlan &p, int nq, const uint8_t *codes, char *ws, size_t per_query, hipStream_t s) {
    const int pat = h.mx_pat;
    (void)pat;
#define MX_COLS(S, PAT) return mx_cols<KIND, S, PAT>(h, p, nq, codes, ws, per_query, s)
    if constexpr (KIND == SCAN_NIB8) MX_COLS(4, 0);
    else if constexpr (KIND == SCAN_NIB16) MX_COLS(8, 0);
    else if constexpr (KIND == SCAN_C5) {
        if (pat == 221) MX_COLS(5, 221);
        if (h.mx_steps == 5) MX_COLS(5, 0);
        MX_COLS(6, 0);
    } else if constexpr (KIND == SCAN_W64) {
        if (pat == 801) MX_COLS(9, 801);
        if (pat == 440) MX_COLS(8, 440);
        MX_COLS(10, 0);
    } else {
        if (pat == 801) MX_COLS(18, 801);
        if (pat == 440) MX_COLS(16, 440);
        MX_COLS(20, 0);
    }
#undef MX_COLS
}

template <int KIND, typename QT>
int mx_launch(const pq_index *idx, const pq_qparams_t *qparams, int nq, const uint8_t *codes, int64_t n, int R,
                     int32_t *out_ids, uint16_t *out_keys, float *out_dist, char *ws, const ScanPlan &sp, const MxPlan &p,
                     hipStream_t s) {
    const DevLayout &h = idx->h;
    mx_steps<KIND>(h, p, nq, codes, ws, sp.per_query, s);
    QADC_LAUNCH_CHECK("k_scan_mx");
    const size_t gtab_bytes = ((size_t)h.gtab_len * sizeof(QT) + 15) & ~(size_t)15;
    GroupDesc gd = group_desc_args(h);
    if ((KIND == SCAN_W64 || KIND == SCAN_C5) && (h.g32ok == 0 || h.ng > QADC_MAXG_FAST)) gd.ng = 0;
    if (KIND == SCAN_W128) gd.ng = h.ng / 2;
    // levels the sums fall short by: about half a level per sub-quantizer where entries are scaled
    const int margin = 1 + 3 * h.m / 8;
    const int lgpc = p.gpc == 16 ? 4 : 2, lnb = __builtin_ctz((unsigned)p.nb);
#define QADC_PICK_GO(NT, CAP)                                                                                   \
    do {                                                                                                        \
        const size_t lds = sizeof(SelectLds<NT, CAP>) + gtab_bytes;                                             \
        if (lds > 48 * 1024)                                                                                    \
            QADC_HIP_TRY(hipFuncSetAttribute((const void *)k_pick<KIND, QT, NT, CAP>,                           \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));            \
        hipLaunchKernelGGL((k_pick<KIND, QT, NT, CAP>), dim3(nq), dim3(NT), lds, s, idx->dev, qparams, codes, n, R, \
                           (const char *)ws, sp.per_query, sp.gtab_off, p.min_off, lgpc, lnb, p.nmin, margin,   \
                           h.gtab_len, gd, out_ids, out_keys, out_dist);                                            \
    } while (0)
    // many queries with short results: small blocks, of which a CU holds eight; else large ones, of
    // which a query's latency profits
    if (R <= FUSED_R && nq > 512) QADC_PICK_GO(256, FUSED_CAP);
    else if (R <= FINAL_SMALL_R) QADC_PICK_GO(1024, FINAL_SMALL_CAP);
    else QADC_PICK_GO(1024, FINAL_CAP);
#undef QADC_PICK_GO
    QADC_LAUNCH_CHECK("k_pick");
    return PQ_OK;
}
