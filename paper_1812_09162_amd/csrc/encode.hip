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

// Which form a call takes: FAST = the expanded form (its norms are taken once per block, of up to 4096 that
// run over the tiles); AHEAD = a tile requested while the one before is encoded (32 registers, which halve the
// wavefronts of a SIMD to four).  Without both every tile has a block of its own.  Times in us, of 10^6
// vectors unless said, FAST + AHEAD / AHEAD / neither:
//   16 x 4 bits, d = 96: 129 / 132 / 140 (232 with loads of one value each); d = 128: 148 / 159 / 209
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
    size_t cbf = 0;  // codebook floats
    for (int j = 0; j < h.m; ++j) cbf += ((size_t)1 << h.nbits[j]) * (size_t)h.dsub[j];
    const size_t base_lds = (size_t)ENC_VB * (size_t)(h.d | 1) * sizeof(float) + (size_t)ENC_VB * (size_t)h.m;
    if (cbf * sizeof(float) > 48 * 1024 || base_lds + cbf * sizeof(float) > 96 * 1024) cbf = 0;
    // small codebooks are read through the scalar cache instead (faster than LDS reads)
    if (cbf * sizeof(float) <= 16 * 1024) cbf = 0;
    size_t lds = base_lds + cbf * sizeof(float);
    const int64_t blocks = (n + ENC_VB - 1) / ENC_VB;
    if (blocks > 0x7fffffffLL) {
        qadc_set_error("pq_encode: n=%lld too large for one call", (long long)n);
        return PQ_EINVAL;
    }
    const int vec = h.d % 4 == 0 && (((uintptr_t)vectors | (uintptr_t)shift_rows) & 15u) == 0;
    size_t nrm_words = (size_t)((h.T + 3) & ~3) + (size_t)((h.m + 3) & ~3);
    const EncForm f = enc_form(h, blocks, lds, nrm_words * sizeof(float), vec != 0);
    if (!f.fast) nrm_words = 0;
    lds += nrm_words * sizeof(float);
    if (lds > 160 * 1024) {
        qadc_set_error("pq_encode: d=%d needs %zu bytes of LDS per block, more than 163840", h.d, lds);
        return PQ_EINVAL;
    }
    const int nib = (h.kind == SCAN_NIB8 || h.kind == SCAN_NIB16) && ((uintptr_t)codes & 3u) == 0;
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
