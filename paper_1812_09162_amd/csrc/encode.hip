// pq_encode: vectors -> packed codes (Section 2.1.2: each sub-vector is replaced by the index of
// its nearest centroid; Section 2.1.1: behind an inverted index the residual x - centroid is
// encoded; Section 3.3: the sub-codes are packed as a little-endian bit stream).
//
// The distance of sub-vector j to centroid i is the table entry D^j[i] of eq. (1) for z = x:
// fp32, dimensions ascending, separate subtract / multiply / add.  Sub-code j is the index of
// the smallest distance, the lowest index among equals.
//
// A block of 256 threads encodes tiles of 64 vectors, staged (minus the shift) in LDS; wave w takes the
// sub-quantizers w, w+4, ... and lane v the vector v, so that centroid values are uniform across a wave:
// codebooks of up to 16 KB are read from memory with scalar loads (they stay in the scalar cache), larger
// ones are staged in LDS when they fit (one word broadcast to 64 lanes).  A second step packs.
//
// 16 and 32 sub-quantizers of 4 bits over equal sub-spaces have a kernel of their own on the matrix cores
// (k_encode_mx); what follows is about the rest.
//
// Bound by the vector units: eq. (1) term by term is three operations per dimension and centroid.  Where
// it pays (enc_form) the nearest centroid of a sub-space of up to 8 dimensions is found from ||x||^2 + ||c||^2 - 2 x.c, one fused
// multiply-add per dimension; the distances of eq. (1) themselves are computed only in waves that hold a
// vector whose two smallest values are closer than the rounding of both forms can account for, and then
// decide.  The norms are taken once per block, which runs over many tiles; tiles are staged with 16-byte
// loads and without a division per value.  10^7 vectors, d = 96, 16 x 4 bits: 1.23 ms (2.12 term by
// term; 1.37 without the next tile requested ahead).
#include <type_traits>

#include "qadc_device.h"

#define ENC_VB 64  // vectors per tile
#define ENC_MX_BLOCKS 3  // of a CU, which run over the tiles (matrix form)
#define ENC_PF 8   // 16-byte pieces of a tile a thread holds: d <= 128
typedef float enc_f4 __attribute__((ext_vector_type(4)));

// Nearest of kj centroids of DS dimensions (rows of c) to the sub-vector xv: eq. (1) term by
// term, the lowest index among equal distances.
template <int DS>
__device__ __forceinline__ void enc_nearest(const float *xv, const float *c, int kj, float &best,
                                            int &besti) {
    float xr[DS];
#pragma unroll
    for (int l = 0; l < DS; ++l) xr[l] = xv[l];
#pragma unroll 4
    for (int i = 0; i < kj; ++i) {
        float acc = 0.0f;
#pragma unroll
        for (int l = 0; l < DS; ++l) {
            const float diff = __fsub_rn(xr[l], c[i * DS + l]);
            acc = __fadd_rn(acc, __fmul_rn(diff, diff));
        }
        if (i == 0 || acc < best) {
            best = acc;
            besti = i;
        }
    }
}

// The same index for a wave from the expanded form (nrm: the centroids' squared norms in LDS, kj of them,
// a multiple of four; nmax: the largest).  Values carry their index in the low `nb` bits.
template <int DS>
__device__ __forceinline__ int enc_nearest_fast(const float *xv, const float *c, const float *nrm, float nmax, int nb) {
    float y[DS], xx = 0.0f;
#pragma unroll
    for (int l = 0; l < DS; ++l) {
        const float x = xv[l];
        xx = __fmaf_rn(x, x, xx);
        y[l] = -2.0f * x;
    }
    // S bounds |2 x.c| and half of any distance.  The offset keeps every value above zero, so that its
    // bits order as an integer.
    const float S = xx + nmax, off = __fmaf_rn(S, 1.0f / 65536.0f, xx);
    const int kj = 1 << nb;
    const uint32_t keep = ~((1u << nb) - 1u);
    uint32_t m1 = 0xffffffffu, m2 = 0xffffffffu;  // the two smallest
    for (int i0 = 0; i0 < kj; i0 += 4) {  // (four independent chains at a time)
        const float4 n4 = *(const float4 *)(nrm + i0);
        float v[4] = {n4.x + off, n4.y + off, n4.z + off, n4.w + off};
#pragma unroll
        for (int l = 0; l < DS; ++l)
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = __fmaf_rn(c[(i0 + u) * DS + l], y[l], v[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t key = (__float_as_uint(v[u]) & keep) | (uint32_t)(i0 + u);
            m2 = min(m2, max(m1, key));
            m1 = min(m1, key);
        }
    }
    // Roundings: at most DS + 3 of the expanded form and DS + 2 of eq. (1), each 2^-24 of at most 2 S, for
    // two values: below 2^-17 S; the dropped bits: 2^(nb - 23) of a value.  (Sums near the smallest
    // normal numbers round otherwise: S > 1e-30.)
    const float f1 = __uint_as_float(m1 & keep), f2 = __uint_as_float(m2 & keep);
    const bool clear = S > 1e-30f && f2 - f1 > __fmaf_rn(f2, ldexpf(1.0f, nb - 22), S * (1.0f / 131072.0f));
    int besti = (int)(m1 & ~keep);
    if (__ballot(!clear) != 0) {
        float best = INFINITY;
        int e = 0;
        enc_nearest<DS>(xv, c, kj, best, e);
        besti = clear ? besti : e;
    }
    return besti;
}

template <bool FAST, bool AHEAD>
__global__ void __launch_bounds__(256)
k_encode(const DevLayout *__restrict__ L, const EntryDesc *__restrict__ edesc, const float *__restrict__ cb,
         const float *__restrict__ x, int64_t n, const float *__restrict__ shift_rows,
         const int32_t *__restrict__ shift_ids, uint8_t *__restrict__ codes, int cb_floats, int nrm_words,
         int64_t ntiles, int vec, int nib) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int d = L->d, m = L->m, cs = L->cs, T = L->T;
    const int ldx = d | 1;  // odd row stride: lanes of a wave (consecutive vectors) hit distinct banks
    // FAST: squared norms [T], and the largest norm per sub-quantizer (bits) [m]
    float *nrm = (float *)smem;
    uint32_t *nmax = (uint32_t *)nrm + ((T + 3) & ~3);
    float *xs = nrm + nrm_words;                           // [ENC_VB][ldx]
    float *cbs = xs + (size_t)ENC_VB * ldx;                // [cb_floats] (0 if they do not fit)
    uint8_t *sub = (uint8_t *)(cbs + cb_floats);           // [ENC_VB][m]
    if constexpr (FAST)
        for (int i = threadIdx.x; i < m; i += 256) nmax[i] = 0;
    for (int e = threadIdx.x; e < cb_floats; e += 256) cbs[e] = cb[e];
    if constexpr (FAST) {
        __syncthreads();
        for (int e = threadIdx.x; e < T; e += 256) {
            const EntryDesc ed = edesc[e];
            const float *c = cb + ed.cb_off;
            float s = 0.0f;
            for (int l = 0; l < ed.ds; ++l) s = __fmaf_rn(c[l], c[l], s);
            atomicMax(&nmax[ed.j], __float_as_uint(s));
            nrm[e] = s;
        }
    }
    // this thread's first 16-byte piece of a tile: vector sv, piece sl of its d4; the next is 256 further on
    const int d4 = vec ? d >> 2 : 1, dv = 256 / d4, dl = 256 - dv * d4;
    const int sv = (int)threadIdx.x / d4, sl = (int)threadIdx.x - sv * d4;
    enc_f4 nx[AHEAD ? ENC_PF : 1];
    auto request = [&](int64_t t) {  // (pieces past the end: the last one again)
        const int64_t left = n - t * ENC_VB;
        const int last = (int)(left < ENC_VB ? left : ENC_VB) * d4 - 1;
        const enc_f4 *src = (const enc_f4 *)(x + (size_t)t * ENC_VB * d);
#pragma unroll
        for (int i = 0; i < (AHEAD ? ENC_PF : 1); ++i) {
            const int e = i * 256 + (int)threadIdx.x;
            nx[i] = __builtin_nontemporal_load(src + (e < last ? e : last));
        }
    };
    if constexpr (AHEAD) request(blockIdx.x);
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t v0 = tile * ENC_VB;
        const int nv = n - v0 < ENC_VB ? (int)(n - v0) : ENC_VB;
        __syncthreads();  // the previous tile has been packed
        if constexpr (AHEAD) {
            // the tile is in registers already; the next one is requested before this one is encoded
            int v = sv, l4 = sl;
#pragma unroll
            for (int i = 0; i < ENC_PF; ++i) {
                if (i * 256 + (int)threadIdx.x < nv * d4) {
                    enc_f4 val = nx[i];
                    if (shift_rows) {
                        const enc_f4 s = *(const enc_f4 *)(shift_rows + (size_t)shift_ids[v0 + v] * d + 4 * l4);
                        val.x = __fsub_rn(val.x, s.x);
                        val.y = __fsub_rn(val.y, s.y);
                        val.z = __fsub_rn(val.z, s.z);
                        val.w = __fsub_rn(val.w, s.w);
                    }
                    float *dst = xs + v * ldx + 4 * l4;
                    dst[0] = val.x;
                    dst[1] = val.y;
                    dst[2] = val.z;
                    dst[3] = val.w;
                    v += dv;
                    l4 += dl;
                    if (l4 >= d4) l4 -= d4, ++v;
                }
            }
            if (tile + gridDim.x < ntiles) request(tile + gridDim.x);
        } else if (vec) {
            int v = sv, l4 = sl;
            const float4 *src = (const float4 *)(x + (size_t)v0 * d);
            for (int e = threadIdx.x; e < nv * d4; e += 256) {
                float4 val = src[e];
                if (shift_rows) {
                    const float4 s = *(const float4 *)(shift_rows + (size_t)shift_ids[v0 + v] * d + 4 * l4);
                    val.x = __fsub_rn(val.x, s.x);
                    val.y = __fsub_rn(val.y, s.y);
                    val.z = __fsub_rn(val.z, s.z);
                    val.w = __fsub_rn(val.w, s.w);
                }
                float *dst = xs + v * ldx + 4 * l4;
                dst[0] = val.x;
                dst[1] = val.y;
                dst[2] = val.z;
                dst[3] = val.w;
                v += dv;
                l4 += dl;
                if (l4 >= d4) l4 -= d4, ++v;
            }
        } else {
            for (int e = threadIdx.x; e < nv * d; e += 256) {
                const int v = e / d, l = e - v * d;
                float val = x[(size_t)v0 * d + e];
                if (shift_rows) val = __fsub_rn(val, shift_rows[(size_t)shift_ids[v0 + v] * d + l]);
                xs[v * ldx + l] = val;
            }
        }
        __syncthreads();

        // the wave index as a scalar: sub-quantizer, widths and codebook addresses are then uniform
        // values, and codebook entries read from memory come through the scalar cache
        const int v = threadIdx.x % ENC_VB, w = __builtin_amdgcn_readfirstlane(threadIdx.x / ENC_VB);
        // `c0` = the codebooks, in LDS or in memory: one instance of the loop for each, so that the
        // reads are plain LDS reads or (uniform addresses) scalar loads, not generic-pointer loads
        auto assign = [&](const float *c0) {
            for (int j = w; j < m; j += 4) {
                const int ds = L->dsub[j], nb = L->nbits[j];
                const float *c = c0 + L->cboff[j];
                const float *xv = xs + (v < nv ? v : 0) * ldx + L->dimoff[j];
                const float *nj = nrm + L->toff[j];
                const float mx = FAST ? __uint_as_float(__builtin_amdgcn_readfirstlane(nmax[j])) : 0.0f;
                float best = INFINITY;
                int besti = 0;
                // (four centroids at a time: tables that begin on a multiple of four entries)
                const bool fast = FAST && (L->toff[j] & 3) == 0 && nb >= 2;
                auto nearest = [&](auto width) {
                    constexpr int DS = decltype(width)::value;
                    if constexpr (FAST) {
                        besti = enc_nearest_fast<DS>(xv, c, nj, mx, nb);
                    } else {
                        enc_nearest<DS>(xv, c, 1 << nb, best, besti);
                    }
                };
                switch (!FAST || fast ? ds : 0) {  // uniform over the wave; widths up to 8 are unrolled without predicates
                    case 1: nearest(std::integral_constant<int, 1>()); break;
                    case 2: nearest(std::integral_constant<int, 2>()); break;
                    case 3: nearest(std::integral_constant<int, 3>()); break;
                    case 4: nearest(std::integral_constant<int, 4>()); break;
                    case 5: nearest(std::integral_constant<int, 5>()); break;
                    case 6: nearest(std::integral_constant<int, 6>()); break;
                    case 7: nearest(std::integral_constant<int, 7>()); break;
                    case 8: nearest(std::integral_constant<int, 8>()); break;
                    default:
                        for (int i = 0; i < (1 << nb); ++i) {
                            float acc = 0.0f;
                            for (int l = 0; l < ds; ++l) {
                                const float diff = __fsub_rn(xv[l], c[i * ds + l]);
                                acc = __fadd_rn(acc, __fmul_rn(diff, diff));
                            }
                            if (i == 0 || acc < best) {
                                best = acc;
                                besti = i;
                            }
                        }
                }
                if (v < nv) sub[v * m + j] = (uint8_t)besti;
            }
        };
        if (cb_floats)
            assign(cbs);
        else
            assign(cb);
        __syncthreads();

        if (nib) {  // four code bytes = eight sub-codes per thread and round (codes of 8 or 16 bytes)
            const int c4 = cs >> 2;
            for (int e = threadIdx.x; e < nv * c4; e += 256) {
                const uint2 s = *(const uint2 *)(sub + 8 * e);  // (m = 2 cs: the sub-codes of dword e)
                const uint32_t lo = s.x | (s.x >> 4), hi = s.y | (s.y >> 4);
                ((uint32_t *)(codes + (size_t)v0 * cs))[e] = (lo & 255u) | ((lo >> 8) & 0xff00u) | ((hi & 255u) << 16) | ((hi << 8) & 0xff000000u);
            }
        } else {
            // pack: one output byte per thread and round
            for (int e = threadIdx.x; e < nv * cs; e += 256) {
                const int vv = e / cs, b = e - vv * cs;
                uint32_t byte = 0;
                for (int j = 0; j < m; ++j) {
                    const int off = L->bitoff[j], nb = L->nbits[j];
                    if (off + nb <= 8 * b || off >= 8 * b + 8) continue;
                    const uint32_t val = sub[vv * m + j];
                    const int rel = off - 8 * b;  // position of the sub-code's bit 0 relative to this byte
                    byte |= rel >= 0 ? (val << rel) : (val >> (-rel));
                }
                codes[(size_t)v0 * cs + e] = (uint8_t)(byte & 255u);
            }
        }
    }
}

// ------------------------------------------------------- on the matrix cores ---
// M sub-quantizers of 4 bits over DS dimensions each.  The expanded form's products are a matrix product of a
// sub-quantizer's 16 centroids and 16 vectors, which the fp32 matrix instruction takes four dimensions at a time (a
// chain of fused multiply-adds in ascending order).  A wave encodes tiles of 16 vectors by itself, staged in rows of
// its own in LDS and read as lane (vector l % 16, dimension l / 16 of four); the centroids stay in its registers
// (times -2).  A lane gets ||c||^2 - 2 x.c of four centroids for one vector; with their index in the low four bits the two
// smallest of the 16 take six minima, maxima and medians and, for four sub-quantizers together, fifteen operations across
// lanes, which leave lane (v, g) with vector v and sub-quantizer {0, 2, 1, 3}[g] of the four.  Near ties are decided
// by eq. (1) as in enc_nearest_fast, within a margin of the sub-space's own norms (sub-spaces may differ in size by any
// factor); values may be below zero here, so that no offset has to be the same for all lanes of a vector.
// What bounds it: memory; behind it minima and packing on the vector units (106 instructions a wave per 1024 distances, 52 % of the
// time) and the products (31 %).  10^7 vectors, d = 96, 16 x 4 bits: 912 us
// (4.3 TB/s; a copy of this card's memory runs at 4.8), 1193 with the expanded form on the vector units; 969 with values made
// positive by the whole vector's norm and margins of that size, which also took every small sub-space of uneven vectors for
// a near tie: 10^6 vectors of variance i^-4 97 us, 207 so, 133 on the vector units.
typedef float enc_v4f __attribute__((ext_vector_type(4)));
template <int M, int DS>
struct EncMxLds {
    static constexpr int D = M * DS, ROW = D + 4;  // a row is an odd multiple of four floats: no bank conflicts
    static constexpr int CB = 16 * DS + 4;         // (four sub-quantizers' centroids, read at a time, too)
    float xs[4][16][ROW];
    float cb[M * CB];
    float nrm[M][16];
    uint32_t nmax[M];
};
template <int M, int DS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ENC_MX_BLOCKS)))
k_encode_mx(const float *__restrict__ cb, const float *__restrict__ x, int64_t n, const float *__restrict__ shift_rows,
            const int32_t *__restrict__ shift_ids, uint8_t *__restrict__ codes, int64_t ntiles) {
    constexpr int KK = (DS + 3) / 4, D = M * DS, D4 = D / 4, PF = D4 * 16 / 64;
    static_assert(D % 16 == 0 && M % 4 == 0 && M <= 32, "rows of whole 16-byte pieces, groups of four sub-quantizers");
    typedef EncMxLds<M, DS> Lds;
    __shared__ __align__(16) Lds S;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int v = lane & 15, g = lane >> 4;
    for (int e = threadIdx.x; e < M * 16 * DS; e += 256) S.cb[e + e / (16 * DS) * 4] = cb[e];
    if (threadIdx.x < M) S.nmax[threadIdx.x] = 0;
    __syncthreads();
    for (int e = threadIdx.x; e < M * 16; e += 256) {
        const float *c = &S.cb[(e >> 4) * Lds::CB + (e & 15) * DS];
        float s = 0.0f;
#pragma unroll
        for (int l = 0; l < DS; ++l) s = __fmaf_rn(c[l], c[l], s);
        (&S.nrm[0][0])[e] = s;
        atomicMax(&S.nmax[e >> 4], __float_as_uint(s));
    }
    float a[M][KK];
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) a[j][kk] = 4 * kk + g < DS ? -2.0f * S.cb[j * Lds::CB + v * DS + 4 * kk + g] : 0.0f;
    __syncthreads();
    float (*xs)[Lds::ROW] = S.xs[w];
    enc_f4 nx[PF];
    auto request = [&](int64_t tile) {  // (rows past the end: the last one again)
        const int64_t left = n - tile * 16;
        const int rows = left < 16 ? (int)left : 16;
        const enc_f4 *src = (const enc_f4 *)(x + (size_t)tile * 16 * D);
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const int e = i * 64 + lane;
            nx[i] = __builtin_nontemporal_load(src + (rows == 16 ? e : min(e / D4, rows - 1) * D4 + e % D4));
        }
    };
    // Minima and maxima as medians with an infinity that the compiler does not see: it makes both arguments of a minimum
    // quiet first, an operation each.  (Of a NaN it is no minimum; where there is one, none is used.)
    float inf = INFINITY;
    asm("" : "+s"(inf));
    auto least = [inf](float p, float q) { return __builtin_amdgcn_fmed3f(p, q, -inf); };
    const int64_t stride = (int64_t)gridDim.x * 4;
    int64_t tile = (int64_t)blockIdx.x * 4 + w;
    if (tile < ntiles) request(tile);
    const uint32_t idx0 = 4u * (uint32_t)g;
    const int sub = g == 1 ? 2 : (g == 2 ? 1 : g);  // of a group of four: the one this lane ends up with
    const uint32_t own = 4 * (KK - 1) + g < DS ? ~0u : 0u;  // of a sub-quantizer's last four dimensions: those it has
    for (; tile < ntiles; tile += stride) {
        const int64_t v0 = tile * 16;
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const int e = i * 64 + lane, r = e / D4, l4 = e % D4;
            enc_f4 val = nx[i];
            if (shift_rows) {
                const int64_t row = v0 + r < n ? v0 + r : n - 1;
                const enc_f4 s = *(const enc_f4 *)(shift_rows + (size_t)shift_ids[row] * D + 4 * l4);
                val.x = __fsub_rn(val.x, s.x);
                val.y = __fsub_rn(val.y, s.y);
                val.z = __fsub_rn(val.z, s.z);
                val.w = __fsub_rn(val.w, s.w);
            }
            *(enc_f4 *)&xs[r][4 * l4] = val;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (the rows are this wave's own)
        if (tile + stride < ntiles) request(tile + stride);
        float b[M][KK];
#pragma unroll
        for (int j = 0; j < M; ++j)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                b[j][kk] = xs[v][j * DS + 4 * kk + g];
                if (kk == KK - 1 && DS % 4 != 0) b[j][kk] = __uint_as_float(__float_as_uint(b[j][kk]) & own);
            }
        uint32_t word[M / 8];
#pragma unroll
        for (int i = 0; i < M / 8; ++i) word[i] = 0;
#pragma unroll
        for (int q = 0; q < M / 4; ++q) {
            float m1[4], m2[4], xx[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = 4 * q + u;
                enc_v4f acc = *(const enc_v4f *)&S.nrm[j][4 * g];
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j][kk], b[j][kk], acc, 0, 0, 0);
                float k[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) k[i] = __uint_as_float((__float_as_uint(acc[i]) & ~15u) | (idx0 + (uint32_t)i));
                m1[u] = least(k[0], k[1]);
                m2[u] = __builtin_amdgcn_fmed3f(k[0], k[1], inf);
#pragma unroll
                for (int i = 2; i < 4; ++i) {
                    m2[u] = __builtin_amdgcn_fmed3f(m1[u], m2[u], k[i]);
                    m1[u] = least(m1[u], k[i]);
                }
                xx[u] = b[j][0] * b[j][0];
#pragma unroll
                for (int kk = 1; kk < KK; ++kk) xx[u] = __fmaf_rn(b[j][kk], b[j][kk], xx[u]);
            }
            // two lists of two smallest, the second's at least its first: their two smallest
            auto merge = [least](float p1, float p2, float q1, float q2, float &r1, float &r2) {
                r2 = __builtin_amdgcn_fmed3f(p1, q1, least(p2, q2));
                r1 = least(p1, q1);
            };
            auto swap32 = [](float &p, float &q) {
                const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(q), false, false);
                p = __uint_as_float(r[0]);
                q = __uint_as_float(r[1]);
            };
            auto swap16 = [](float &p, float &q) {
                const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(q), false, false);
                p = __uint_as_float(r[0]);
                q = __uint_as_float(r[1]);
            };
#pragma unroll
            for (int u = 0; u < 4; u += 2) {
                swap32(m1[u], m1[u + 1]);
                swap32(m2[u], m2[u + 1]);
                swap32(xx[u], xx[u + 1]);
                merge(m1[u], m2[u], m1[u + 1], m2[u + 1], m1[u], m2[u]);
                xx[u] += xx[u + 1];
            }
            swap16(m1[0], m1[2]);
            swap16(m2[0], m2[2]);
            swap16(xx[0], xx[2]);
            float s1, s2;
            merge(m1[0], m2[0], m1[2], m2[2], s1, s2);
            // S bounds |2 x.c| and half of any distance in this lane's sub-space.  Roundings: at most DS + 3 of the expanded
            // form and DS + 2 of eq. (1), each 2^-24 of at most 2 S (one more for the roundings of S itself), for two
            // values; the dropped bits: 2^-19 of a value.  (Sums near the smallest normal numbers round otherwise, and
            // near the largest they overflow: S within [1e-30, 1e38], which infinities and NaN are not.)
            constexpr float ROUND = (2 * DS + 6) * 4 / 16777216.0f;
            const float Sb = (xx[0] + xx[2]) + __uint_as_float(S.nmax[4 * q + sub]);
            const uint32_t k1 = __float_as_uint(s1);
            const float f1 = __uint_as_float(k1 & ~15u), f2 = __uint_as_float(__float_as_uint(s2) & ~15u);
            const bool clear = Sb > 1e-30f && Sb < 1e38f && f2 - f1 > __fmaf_rn(fabsf(f1) + fabsf(f2), 1.0f / 262144.0f, Sb * ROUND);
            int besti = (int)(k1 & 15u);
            if (__ballot(!clear) != 0) {
                if (!clear) {
                    float best = INFINITY;
                    enc_nearest<DS>(&xs[v][(4 * q + sub) * DS], &S.cb[(4 * q + sub) * Lds::CB], 16, best, besti);
                }
            }
            word[q >> 1] |= (uint32_t)besti << (16 * (q & 1) + 4 * sub);
        }
        // a vector's words, from its four lanes; lane (v, g) stores word g (and g + 4)
#pragma unroll
        for (int i = 0; i < M / 8; ++i) {
            auto r = __builtin_amdgcn_permlane32_swap(word[i], word[i], false, false);
            word[i] = (uint32_t)r[0] | (uint32_t)r[1];
            r = __builtin_amdgcn_permlane16_swap(word[i], word[i], false, false);
            word[i] = (uint32_t)r[0] | (uint32_t)r[1];
        }
        if (v0 + v < n) {
            uint32_t *dst = (uint32_t *)(codes + (size_t)(v0 + v) * (M / 2));
#pragma unroll
            for (int i = 0; i < M / 8; ++i)
                if (i == g) dst[i] = word[i];
        }
    }
}

// The matrix form takes 16 or 32 sub-quantizers of 4 bits over equal sub-spaces; vectors and shifts are read in
// 16-byte pieces.  At every size and on every kind of data timed it was the faster one, us for 10^6 vectors, expanded form on the vector
// units / here: 16 x 4 bits, d = 64 98 / 73, d = 96 129 / 96, d = 128 150 / 102; 32 x 4 bits, d = 96 193 / 145, d = 128 191 / 141;
// integer-valued data (near ties) 129 / 93, 144 / 96 and 189 / 152; variance falling as i^-1.5 to i^-4 or one sub-space a hundred
// times as large 130 to 137 / 97 to 99 (d = 96); one dimension a hundred or a thousand standard deviations off the origin, which makes
// near ties of one sub-space in sixteen, 139 and 142 / 114 and 124; 1000 vectors 10.8 / 9.5.
static int enc_mx_width(const pq_index *idx, bool vec, bool nib) {
    const DevLayout &h = idx->h;
    if (!vec || !nib || h.ds_uniform == 0 || h.d != h.m * h.ds_uniform) return 0;
    if (h.kind == SCAN_NIB8 && (h.ds_uniform == 4 || h.ds_uniform == 6 || h.ds_uniform == 8)) return h.ds_uniform;
    if (h.kind == SCAN_NIB16 && (h.ds_uniform == 3 || h.ds_uniform == 4)) return h.ds_uniform;
    return 0;
}

// Which form a call takes: FAST = the expanded form (its norms are taken once per block, of up to 4096 that
// run over the tiles); AHEAD = a tile requested while the one before is encoded (32 registers, which halve the
// wavefronts of a SIMD to four).  Without both every tile has a block of its own.  Times in us, of 10^6
// vectors unless said, FAST + AHEAD / AHEAD / neither:
//   16 x 4 bits, d = 96 (where vectors or codes are not aligned for the matrix form): 129 / 132 / 140 (232 with loads of
//   one value each); d = 128: 148 / 159 / 209
//   {6,6,4} x 8, d = 128: 915 / 1009 / 1130; 2 * 10^5 vectors: 238 / 241 / 241
//   16 x 8 bits, d = 128: 2000 / 2177 / 3190; d = 96: 1759 / 1742 / 1464
//   8 x 8 bits (sub-spaces of 12 and 16 dimensions), d = 96: 5041 / 5230 / 4099; d = 128: 8273 / 6818 / 6441
//   {6,5,5,6,5,5,4,4}, d = 96: 1016 / 1057 / 778; d = 128: 2640 / 1915 / 1955
//   64 x 4 bits, d = 96: 1268 / 1230 / 1055
struct EncForm {
    bool fast, ahead;
};
static EncForm enc_form(const DevLayout &h, int64_t tiles, size_t lds, size_t norms, bool vec) {
    EncForm f;
    int64_t cb = 0;
    bool narrow = true;  // all sub-spaces within what the expanded form is unrolled for
    for (int j = 0; j < h.m; ++j) {
        cb += ((int64_t)1 << h.nbits[j]) * h.dsub[j];
        narrow = narrow && h.dsub[j] <= 8;
    }
    const int64_t most = 160 * 1024, per_cu = most / (int64_t)lds, with_norms = most / (int64_t)(lds + norms);
    // The expanded form: wide sub-spaces (it saves one operation in three per dimension and adds some per
    // centroid) of 16 centroids and more; enough tiles per block to pay for the norms, or so few that the
    // latency of a block counts; and norms that do not cost a CU too many of its blocks.
    if (!narrow || h.T < 16 * h.m || with_norms < 1)
        f.fast = false;
    else if (tiles <= 256)
        f.fast = cb >= 5 * (int64_t)h.T;
    else
        f.fast = tiles >= 3 * (int64_t)h.T &&
                 (with_norms == per_cu ? cb >= 4 * (int64_t)h.T : 4 * with_norms >= 3 * per_cu && cb >= 6 * (int64_t)h.T);
    // The tile ahead: its registers cost nothing where LDS allows no more than four blocks of a CU.  (Sub-spaces
    // of two dimensions have too little to do per tile: 64 x 4 bits, d = 128, 1000 vectors 73 us, 69 without.)
    f.ahead = vec && h.d <= 4 * 4 * ENC_PF && (f.fast || (per_cu <= 4 && cb >= 3 * (int64_t)h.T));
    return f;
}

extern "C" int pq_encode(const pq_index_t *idx, const float *vectors, int64_t n,
                         const float *shift_rows, const int32_t *shift_ids, uint8_t *codes,
                         void *stream) {
    if (!idx || n < 0) {
        qadc_set_error("pq_encode: bad handle or n");
        return PQ_EINVAL;
    }
    if (n == 0) return PQ_OK;
    if (!vectors || !codes || ((shift_rows == nullptr) != (shift_ids == nullptr))) {
        qadc_set_error("pq_encode: null pointer (shift_rows and shift_ids go together)");
        return PQ_EINVAL;
    }
    const DevLayout &h = idx->h;
    const int64_t blocks = n / ENC_VB + (n % ENC_VB != 0);
    if (blocks > 0x7fffffffLL) {
        qadc_set_error("pq_encode: n=%lld too large for one call", (long long)n);
        return PQ_EINVAL;
    }
    const int vec = h.d % 4 == 0 && (((uintptr_t)vectors | (uintptr_t)shift_rows) & 15u) == 0;
    const int nib = (h.kind == SCAN_NIB8 || h.kind == SCAN_NIB16) && ((uintptr_t)codes & 3u) == 0;
    if (const int ds = enc_mx_width(idx, vec != 0, nib != 0)) {
        const int64_t tiles = (n + 15) / 16, most = 256 * ENC_MX_BLOCKS;
        const unsigned grid = (unsigned)((tiles + 3) / 4 < most ? (tiles + 3) / 4 : most);
#define ENC_MX_GO(M, DS)                                                                                         \
    hipLaunchKernelGGL((k_encode_mx<M, DS>), dim3(grid), dim3(256), 0, (hipStream_t)stream, idx->codebooks,       \
                       vectors, n, shift_rows, shift_ids, codes, tiles)
        if (h.kind == SCAN_NIB8) {
            if (ds == 4) ENC_MX_GO(16, 4); else if (ds == 6) ENC_MX_GO(16, 6); else ENC_MX_GO(16, 8);
        } else {
            if (ds == 3) ENC_MX_GO(32, 3); else ENC_MX_GO(32, 4);
        }
#undef ENC_MX_GO
        QADC_LAUNCH_CHECK("k_encode_mx");
        return PQ_OK;
    }
    size_t cbf = 0;  // codebook floats
    for (int j = 0; j < h.m; ++j) cbf += ((size_t)1 << h.nbits[j]) * (size_t)h.dsub[j];
    const size_t base_lds = (size_t)ENC_VB * (size_t)(h.d | 1) * sizeof(float) + (size_t)ENC_VB * (size_t)h.m;
    if (cbf * sizeof(float) > 48 * 1024 || base_lds + cbf * sizeof(float) > 96 * 1024) cbf = 0;
    // small codebooks are read through the scalar cache instead (faster than LDS reads)
    if (cbf * sizeof(float) <= 16 * 1024) cbf = 0;
    size_t lds = base_lds + cbf * sizeof(float);
    size_t nrm_words = (size_t)((h.T + 3) & ~3) + (size_t)((h.m + 3) & ~3);
    const EncForm f = enc_form(h, blocks, lds, nrm_words * sizeof(float), vec != 0);
    if (!f.fast) nrm_words = 0;
    lds += nrm_words * sizeof(float);
    if (lds > 160 * 1024) {
        qadc_set_error("pq_encode: d=%d needs %zu bytes of LDS per block, more than 163840", h.d, lds);
        return PQ_EINVAL;
    }
    const int64_t grid = f.fast || f.ahead ? (blocks < 256 * 16 ? blocks : 256 * 16) : blocks;
#define ENC_GO(FAST, AHEAD)                                                                                       \
    do {                                                                                                          \
        if (lds > 48 * 1024)                                                                                      \
            QADC_HIP_TRY(hipFuncSetAttribute((const void *)k_encode<FAST, AHEAD>,                                 \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));              \
        hipLaunchKernelGGL((k_encode<FAST, AHEAD>), dim3((unsigned)grid), dim3(256), lds, (hipStream_t)stream,    \
                           idx->dev, idx->edesc, idx->codebooks, vectors, n, shift_rows, shift_ids, codes, (int)cbf, \
                           (int)nrm_words, blocks, vec, nib);                                                     \
    } while (0)
    if (f.fast && f.ahead) ENC_GO(true, true);
    else if (f.fast) ENC_GO(true, false);
    else if (f.ahead) ENC_GO(false, true);
    else ENC_GO(false, false);
#undef ENC_GO
    QADC_LAUNCH_CHECK("k_encode");
    return PQ_OK;
}
