// Coarse search of a batch with half-precision products and exact re-scoring.
//
// The scores' definition is a chain of fp32 fused multiply-adds, which the matrix cores evaluate at
// 1/16 of their half-precision rate.  Here every cell gets an approximate score from fp16 products
// (fp32 sums) whose distance from the exact one is bounded, E per query; whatever the bound cannot
// rule out, a few cells more than nprobe, is scored again exactly.  The result is the same.
//
//   k_cstat    exact norms ||c||^2 (the chain), and per 256 cells the largest component and norm
//   k_cprep    cells as fp16 rows (-c, then an eighth of the norm in three pieces), scaled by one power
//              of two for all so that the largest component is in [16, 32), in the order the products read
//              (and a constant column)
//   k_qprep    the queries likewise (z, then 4 4 4, then an offset that keeps v from being negative, so
//              that its bits order as integers), and the bound E
//   k_cscan    v = ||c||^2 / 2 - z.c + offset (scaled) for all cells.  PILOT: the smallest of every 16
//              cells of the first P; their nprobe-th smallest (k_cbound) + 2 E is a bound no result
//              exceeds.  Otherwise: 16 cells that hold one within the bound go, with their values, to a
//              list of their own per (query, 1024 cells, half of the wave): no atomics, one test per lane and
//              32 x 32 results.
//   k_cpick    gathers a query's lists, takes the cells within the nprobe-th smallest + 2 E, scores them
//              exactly and ranks them by (score, id)
//
// E, in units of v, bounds |v - exact / 2|: u = 2^-11 is the rounding of fp16, so the products are off
// by at most (2 u + u^2) |z||c|; values below the fp16 normals by 2^-14 each (should the products take
// them as zero); the sums here and the chains of the definition by less than 2^-14 (|z||c| + |c|^2) for
// d <= 256.  The chains also round where they underflow, each sum by 2^-150 or d 2^-150 in all, and end
// at infinity where they overflow.  With the cells' largest component in [2^-50, 2^51) the first is
// nothing beside the terms above (2^-34 in units of v against 2^-6), and the second cannot be (|z||c| of
// a query within the fp16 range is below 2^111); other cells take the exact form.
#include "coarse.h"

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16h __attribute__((ext_vector_type(16)));

#define CH_PICK 2048   // cells within the bound that a k_cpick block holds
#define CH_MAX_D 256

// ------------------------------------------------------------------ k_cstat ---
// A block's 256 cells pass through LDS in pieces of 32 dimensions (coalesced loads; every thread runs
// the chain of one cell).  65,536 x 96: 8 us; one thread per cell reading its row from memory 20 us.
__global__ void __launch_bounds__(256)
k_cstat(const float *__restrict__ centroids, int K, int d, float *__restrict__ cnorm, float *__restrict__ bmax,
        float *__restrict__ bnorm) {
    __shared__ float t[256 * 33];
    __shared__ float s_m[4], s_n[4];
    const int64_t c0 = (int64_t)blockIdx.x * 256;
    const int nc = K - c0 < 256 ? (int)(K - c0) : 256;
    const float *base = centroids + c0 * d;
    float acc = 0.0f, mx = 0.0f;
    for (int k0 = 0; k0 < d; k0 += 32) {
        const int kl = threadIdx.x & 31, r0 = threadIdx.x >> 5;
        float v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const int r = r0 + 8 * i;
            v[i] = (r < nc && k0 + kl < d) ? base[(size_t)r * d + k0 + kl] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 32; ++i) t[(r0 + 8 * i) * 33 + kl] = v[i];
        __syncthreads();
        const int kn = d - k0 < 32 ? d - k0 : 32;
        for (int k = 0; k < kn; ++k) {
            const float x = t[threadIdx.x * 33 + k];
            acc = __fmaf_rn(x, x, acc);
            mx = fmaxf(mx, fabsf(x));
        }
    }
    if ((int)threadIdx.x < nc) cnorm[c0 + threadIdx.x] = acc;
    if (bmax == nullptr) return;
    const uint32_t wm = qadc_wave_max(__float_as_uint(mx)), wn = qadc_wave_max(__float_as_uint(acc));
    if (threadIdx.x % QADC_WAVE == 0) {
        s_m[threadIdx.x / QADC_WAVE] = __uint_as_float(wm);
        s_n[threadIdx.x / QADC_WAVE] = __uint_as_float(wn);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        bmax[blockIdx.x] = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
        bnorm[blockIdx.x] = fmaxf(fmaxf(s_n[0], s_n[1]), fmaxf(s_n[2], s_n[3]));
    }
}

// ---------------------------------------------------------------- k_cdirect ---
// A few queries: norms and scores of 64 cells per block of one wave, straight from the chains of the
// definition (every thread those of one cell).  The cells are read once, in pieces of 32 dimensions
// through LDS, the next piece requested before the current one is used; a call is bound by that read
// and by its launches, of which this form has two instead of seven.
template <int NQ>
__global__ void __launch_bounds__(64)
k_cdirect(const float *__restrict__ queries, int nq, const float *__restrict__ centroids, int K, int d,
          float *__restrict__ scores, size_t ld, float *__restrict__ minima) {
    __shared__ float t[64 * 33];
    __shared__ __align__(16) float zs[32 * NQ];  // [dimension][query]
    const int l = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * 64;
    const int nc = K - c0 < 64 ? (int)(K - c0) : 64;
    const float *base = centroids + c0 * d;
    const int kl = l & 31, r0 = l >> 5;
    float v[32], acc[NQ], norm = 0.0f;
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = (r0 + 2 * i < nc && kl < d) ? base[(size_t)(r0 + 2 * i) * d + kl] : 0.0f;
    for (int k0 = 0; k0 < d; k0 += 32) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 32; ++i) t[(r0 + 2 * i) * 33 + kl] = v[i];
        for (int i = l; i < 32 * NQ; i += 64) {
            const int q = i / 32, k = k0 + (i & 31);
            zs[(i & 31) * NQ + q] = q < nq && k < d ? queries[(size_t)q * d + k] : 0.0f;
        }
        __syncthreads();
        if (k0 + 32 < d)
#pragma unroll
            for (int i = 0; i < 32; ++i)
                v[i] = (r0 + 2 * i < nc && k0 + 32 + kl < d) ? base[(size_t)(r0 + 2 * i) * d + k0 + 32 + kl] : 0.0f;
        const int kn = d - k0 < 32 ? d - k0 : 32;
        for (int k = 0; k < kn; ++k) {
            const float x = t[l * 33 + k];
            norm = __fmaf_rn(x, x, norm);
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q] = __fmaf_rn(zs[k * NQ + q], x, acc[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q >= nq) break;
        const float sc = __fmaf_rn(-2.0f, acc[q], norm);
        if (l < nc) scores[(size_t)q * ld + c0 + l] = sc;
        const uint32_t m = qadc_wave_min(l < nc ? qadc_f2ord(sc) : 0xffffffffu);
        if (l == 0) minima[(size_t)q * ld + blockIdx.x] = qadc_ord2f(m);  // the block's smallest, for the selection
    }
}

int qadc_coarse_direct(const float *queries, int nq, const float *centroids, int K, int d, float *scores, size_t ld,
                       float *minima, hipStream_t s) {
#define CH_DIRECT(NQ) \
    hipLaunchKernelGGL(k_cdirect<NQ>, dim3((K + 63) / 64), dim3(64), 0, s, queries, nq, centroids, K, d, scores, ld, minima)
    if (nq == 1) CH_DIRECT(1); else if (nq <= 4) CH_DIRECT(4); else if (nq <= 8) CH_DIRECT(8); else CH_DIRECT(QADC_DIRECT_NQ);
    QADC_LAUNCH_CHECK("k_cdirect");
    return PQ_OK;
}

// the scale, a power of two, from the blocks' largest components (256 threads; LDS word s: the largest of all)
__device__ __forceinline__ float ch_scale(const float *__restrict__ bmax, int nb, uint32_t *s) {
    uint32_t m = 0;
    for (int i = threadIdx.x; i < nb; i += 256) m = max(m, __float_as_uint(bmax[i]));
    m = qadc_wave_max(m);
    if (threadIdx.x == 0) *s = 0;
    __syncthreads();
    if (threadIdx.x % QADC_WAVE == 0) atomicMax(s, m);
    __syncthreads();
    const float mx = __uint_as_float(*s);
    const int e = mx > 0.0f ? ilogbf(mx) : 0;
    return ldexpf(1.0f, 4 - (e < -90 ? -90 : (e > 90 ? 90 : e)));
}

// ------------------------------------------------------------------ k_cprep ---
// 16 bytes per thread: lane l of step s of a tile of 32 cells = row l % 32, columns 16 s + 8 (l / 32) ..
__global__ void __launch_bounds__(256)
k_cprep(const float *__restrict__ centroids, int K, int d, int S, const float *__restrict__ cnorm,
        const float *__restrict__ bmax, int nb, uint4 *__restrict__ out, int ntiles) {
    __shared__ uint32_t s;
    const float g = ch_scale(bmax, nb, &s);
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
    for (int r = threadIdx.x; r < S * 64; r += 256) {
        const int st = r >> 6, l = r & 63;
        const int64_t c = (int64_t)tile * 32 + (l & 31);
        const int k0 = 16 * st + 8 * (l >> 5);
        h8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = k0 + j;
            float x = 0.0f;
            if (c < K && k < d) {
                x = -g * centroids[c * d + k];
            } else if (k >= d && k < d + 3) {
                // an eighth of the scaled norm in three pieces of eleven bits; rows past the end: out of reach
                const float n = c < K ? (g * cnorm[c]) * g * 0.125f : 60000.0f;
                const float n1 = (float)(_Float16)n, n2 = (float)(_Float16)(n - n1);
                x = k == d ? n1 : (k == d + 1 ? n2 : (n - n1) - n2);
            } else if (k == d + 3) {
                x = 8.0f;
            }
            v[j] = (_Float16)x;
        }
        out[(size_t)tile * (S * 64) + r] = __builtin_bit_cast(uint4, v);
    }
}

// ------------------------------------------------------------------ k_qprep ---
// One block per 32 queries.
__global__ void __launch_bounds__(256)
k_qprep(const float *__restrict__ queries, int nqc, int d, int S, const float *__restrict__ bmax,
        const float *__restrict__ bnorm, int nb, uint4 *__restrict__ out, float *__restrict__ err) {
    __shared__ uint32_t s, s2;
    const float g = ch_scale(bmax, nb, &s);
    uint32_t m = 0;
    for (int i = threadIdx.x; i < nb; i += 256) m = max(m, __float_as_uint(bnorm[i]));
    m = qadc_wave_max(m);
    if (threadIdx.x == 0) s2 = 0;
    __syncthreads();
    if (threadIdx.x % QADC_WAVE == 0) atomicMax(&s2, m);
    __syncthreads();
    const float cmax2 = (g * __uint_as_float(s2)) * g * 1.0001f, cmax = sqrtf(cmax2);
    const float mx = __uint_as_float(s);  // the cells' largest component (ch_scale)
    const bool in_range = mx == 0.0f || (mx >= 0x1p-50f && mx < 0x1p51f);
    const int q0 = blockIdx.x * 32;
    __shared__ float s_off[32];
    // eight lanes per query: norm and largest component
    {
        const int q = q0 + (threadIdx.x >> 3), part = threadIdx.x & 7;
        float z2 = 0.0f, zm = 0.0f;
        if (q < nqc)
            for (int k = part; k < d; k += 8) {
                const float x = g * queries[(size_t)q * d + k];
                z2 += x * x;
                zm = fmaxf(zm, fabsf(x));
            }
#pragma unroll
        for (int sft = 1; sft < 8; sft <<= 1) {
            z2 += __shfl_xor(z2, sft, QADC_WAVE);
            zm = fmaxf(zm, __shfl_xor(zm, sft, QADC_WAVE));
        }
        const float zn = sqrtf(z2 * 1.0001f);
        const float u = 1.0f / 2048.0f;
        const float e = (2.01f * u + 1.0f / 16384.0f) * zn * cmax + cmax2 * (1.0f / 16384.0f) +
                        (zn + cmax + 1.0f) * (sqrtf((float)d) * ldexpf(1.0f, -13));
        const float off = (1.01f * zn * cmax + 2.0f * e) * 0.125f;  // (the cells' column holds 8)
        if (part == 0) {
            s_off[threadIdx.x >> 3] = off;
            // (components or sums beyond the fp16 range, cells outside the bound's, or nothing comparable: the
            // exact form takes the pass)
            if (q < nqc) err[q] = in_range && zm < 16384.0f && off < 60000.0f ? e : INFINITY;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < S * 64; i += 256) {
        const int st = i >> 6, l = i & 63, q = q0 + (l & 31), k0 = 16 * st + 8 * (l >> 5);
        h8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = k0 + j;
            float x = 0.0f;
            if (q < nqc && k < d) x = g * queries[(size_t)q * d + k];
            else if (k >= d && k < d + 3) x = 4.0f;
            else if (k == d + 3) x = s_off[l & 31];
            v[j] = (_Float16)x;
        }
        out[(size_t)blockIdx.x * (S * 64) + i] = __builtin_bit_cast(uint4, v);
    }
}

// ------------------------------------------------------------------ k_cscan ---
// A wave has 32 NCOL queries in registers (S steps of 16 columns) and runs over `tiles` tiles of 32
// cells; the four waves of a block take consecutive groups of queries and the same cells, so that these
// come from memory once for all four.  Lane (c, h) of a result: query column c, cells 8 g + 4 h + i.
// 65,536 cells x 4096 queries, d = 96 (7 steps): 90 us (490 us for the fp32 products of k_scores), of
// which the products alone are 30; the rest is the minima (their time adds to the products') and the
// listing.  Cells read by every wave for itself instead of staged in LDS: 101 us.
// a thread's pieces of the stage that begins with tile t (tiles at or past t1: the last one again)
template <int S, int PER>
__device__ __forceinline__ void ch_request(const u32x4 *__restrict__ cells, int t, int t1, u32x4 (&nx)[PER]) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int at = i * 256 + (int)threadIdx.x, tt = t + at / (S * 64);
        nx[i] = cells[(size_t)(tt < t1 ? tt : t1 - 1) * (S * 64) + at % (S * 64)];
    }
}

template <int S, int NCOL, bool PILOT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_cscan(const u32x4 *__restrict__ cells, int ntiles, int tiles, const uint4 *__restrict__ qs, int nqc,
        const float2 *__restrict__ bounds, uint32_t *__restrict__ minima, int mld, uint4 *__restrict__ ent, uint32_t *__restrict__ ids, uint32_t *__restrict__ counts, int nslots, int cap) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / QADC_WAVE), l = threadIdx.x % QADC_WAVE;
    const int c = l & 31, h = l >> 5;
    const int qt0 = (blockIdx.y * 4 + wave) * NCOL;  // first query tile of this wave
    const int nqt = (nqc + 31) / 32;
    const bool idle = qt0 >= nqt;  // (a wave without queries only helps to stage the cells)
    h8 b[NCOL][S];
    uint32_t bound[NCOL], cnt[NCOL];
#pragma unroll
    for (int ct = 0; ct < NCOL; ++ct) {
        const int qt = qt0 + ct < nqt ? qt0 + ct : nqt - 1;
#pragma unroll
        for (int s = 0; s < S; ++s) b[ct][s] = __builtin_bit_cast(h8, qs[((size_t)qt * S + s) * 64 + l]);
        const int q = (qt0 + ct) * 32 + c;
        cnt[ct] = 0;
        bound[ct] = !PILOT && q < nqc ? __float_as_uint(bounds[q].y) : 0u;
    }
    // this lane's list of column ct starts at entry base0 + ct * bstep (32 bits: K x queries of a pass <= 2^28)
    const uint32_t base0 = ((uint32_t)(qt0 * 32 + c) * (uint32_t)nslots + (uint32_t)(blockIdx.x * 2 + h)) * (uint32_t)cap;
    const uint32_t bstep = 32u * (uint32_t)nslots * (uint32_t)cap;
    uint4 keep[PILOT ? NCOL : 1];  // the last four minima
    const int t0 = blockIdx.x * tiles, t1 = t0 + tiles < ntiles ? t0 + tiles : ntiles;
    // Stages of TS tiles pass through LDS, read from memory once for the four waves; the next stage is
    // requested before the current one is multiplied and stored behind it in the other half.
    constexpr int TS = S <= 9 ? 4 : 2, PER = TS * S / 4;  // 16-byte pieces per thread and stage
    static_assert(TS * S % 4 == 0, "whole pieces per thread");
    __shared__ u32x4 stage[2][TS * S * 64];
    u32x4 nx[PER];
    ch_request<S, PER>(cells, t0, t1, nx);
    int half = 0;
    for (int ts = t0; ts < t1; ts += TS) {
#pragma unroll
        for (int i = 0; i < PER; ++i) stage[half][i * 256 + threadIdx.x] = nx[i];
        __syncthreads();
        if (ts + TS < t1) ch_request<S, PER>(cells, ts + TS, t1, nx);
        const u32x4 *cur = stage[half];
        half ^= 1;
        if (idle) continue;
    for (int t = ts; t < ts + TS && t < t1; ++t) {
        f32x16h acc[NCOL];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const h8 a = __builtin_bit_cast(h8, cur[((t - ts) * S + s) * 64 + l]);
#pragma unroll
            for (int ct = 0; ct < NCOL; ++ct) {
                const f32x16h zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b[ct][s], s == 0 ? zero : acc[ct], 0, 0, 0);
            }
        }
#pragma unroll
        for (int ct = 0; ct < NCOL; ++ct) {
            uint32_t u[16], m = 0xffffffffu;  // (values are >= 0: their bits order as integers)
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = __float_as_uint(acc[ct][r]);
#pragma unroll
            for (int r = 0; r < 16; r += 2) m = min(m, min(u[r], u[r + 1]));
            const int q = (qt0 + ct) * 32 + c;
            if (PILOT) {  // (the order of a row's minima does not matter: four tiles, one store)
                uint4 &kp = keep[PILOT ? ct : 0];
                kp = make_uint4(kp.y, kp.z, kp.w, m);
                if ((t & 3) == 3 && q < nqc) *(uint4 *)(minima + (size_t)q * mld + (2 * (t >> 2) + h) * 4) = kp;
            } else if (m <= bound[ct]) {
                // (a full list keeps counting: the last entry is overwritten and the count tells)
                const uint32_t at = base0 + ct * bstep + min(cnt[ct], (uint32_t)cap - 1u);
                uint4 *e = ent + 4 * (size_t)at;
#pragma unroll
                for (int g = 0; g < 4; ++g) e[g] = make_uint4(u[4 * g], u[4 * g + 1], u[4 * g + 2], u[4 * g + 3]);
                ids[at] = (uint32_t)(t * 32 + 4 * h);
                ++cnt[ct];
            }
        }
    }
    }
    if (idle) return;
    if (!PILOT) {
#pragma unroll
        for (int ct = 0; ct < NCOL; ++ct) {
            const int q = (qt0 + ct) * 32 + c;
            if (q < nqc) counts[(size_t)q * nslots + blockIdx.x * 2 + h] = cnt[ct];  // uncapped
        }
    }
}

// ----------------------------------------------------------------- k_cbound ---
// One wave per query: an upper bound, close by, of the nprobe-th smallest of its pilot minima (NV per
// lane, in registers) by twelve halvings of their range, and from it the bound on v.  (The general
// selection, which ranks them, took 30 us per 4096 queries.)  Clears *flag.
template <int NV>
__global__ void __launch_bounds__(256)
k_cbound(const float *__restrict__ minima, int n, int nq, int nprobe, const float *__restrict__ err,
         float2 *__restrict__ bounds, int *__restrict__ flag) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *flag = 0;
    const int q = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / QADC_WAVE), l = threadIdx.x % QADC_WAVE;
    if (q >= nq) return;
    const float4 *row = (const float4 *)(minima + (size_t)q * n);  // n is a multiple of 128
    float v[NV];
    uint32_t lo_o = 0xffffffffu, hi_o = 0u;
#pragma unroll
    for (int i = 0; i < NV / 4; ++i) {
        const int at = i * QADC_WAVE + l;
        const float4 x = 4 * at < n ? row[at] : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
        v[4 * i] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
        if (4 * at < n)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lo_o = min(lo_o, qadc_f2ord(v[4 * i + j]));
                hi_o = max(hi_o, qadc_f2ord(v[4 * i + j]));
            }
    }
    float lo = qadc_ord2f(qadc_wave_min(lo_o)), hi = qadc_ord2f(qadc_wave_max(hi_o));
    const float first = lo;
    for (int it = 0; it < 12; ++it) {  // at least nprobe values are <= hi
        const float mid = 0.5f * lo + 0.5f * hi;
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) cnt += (int)__popcll(__ballot(v[i] <= mid));
        if (cnt >= nprobe) hi = mid; else lo = mid;
    }
    if (l == 0) bounds[q] = make_float2(first, hi + 2.0f * err[q]);
}

// ------------------------------------------------------------------ k_cpick ---
__global__ void __launch_bounds__(256)
k_cpick(const float *__restrict__ queries, const float *__restrict__ centroids, int K, int d, int nprobe,
        const float *__restrict__ cnorm, const float4 *__restrict__ ent, const uint32_t *__restrict__ ids,
        const uint32_t *__restrict__ counts, int nslots, int cap, const float2 *__restrict__ bounds,
        const float *__restrict__ err, int vec, int32_t *__restrict__ probe_ids, float *__restrict__ probe_scores,
        int *__restrict__ flag) {
    __shared__ uint64_t A[CH_PICK];  // first (ordered v, cell), then (ordered exact score, cell)
    __shared__ uint32_t hist[256], sel[2];
    __shared__ uint32_t s_n, s_m, s_over;
    __shared__ float zs[CH_MAX_D];
    __shared__ uint32_t cand[CS_MAX_NPROBE + 512];
    const size_t q = blockIdx.x;
    const int k = nprobe < K ? nprobe : K;
    const float e = err[q], lo = bounds[q].x, bound = bounds[q].y;
    for (int i = threadIdx.x; i < d; i += 256) zs[i] = queries[q * d + i];
    for (int i = threadIdx.x; i < 256; i += 256) hist[i] = 0;
    if (threadIdx.x == 0) s_n = s_m = s_over = 0;
    __syncthreads();
    if (!(e < 1e30f) || !(bound < 1e30f)) {
        if (threadIdx.x == 0) atomicOr(flag, 1);
        return;
    }
    // four adjacent threads per list: most have a few entries
    const float span = bound - lo;  // (lo: the pilot's smallest value; smaller ones share its bin)
    const float scale = span > 0.0f ? 255.0f / span : 0.0f;
    auto bin_of = [lo, scale](float v) {
        const float x = (v - lo) * scale;
        return x >= 255.0f ? 255u : (x > 0.0f ? (uint32_t)x : 0u);
    };
    const int g = threadIdx.x & 3;  // this thread's four cells of each of a list's entries
    auto take = [&](const float4 &v4, uint32_t c0) {
        const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (v[j] <= bound && (int)(c0 + 8 * g + j) < K) {
                const uint32_t pos = atomicAdd(&s_n, 1u);
                if (pos < CH_PICK) A[pos] = ((uint64_t)__float_as_uint(v[j]) << 32) | (c0 + 8 * g + j);
                atomicAdd(&hist[bin_of(v[j])], 1u);
            }
    };
    for (int s0 = threadIdx.x >> 2; s0 < nslots; s0 += 128) {
        // two lists' lengths and first entries are requested together (entries beyond a list's length
        // are read and ignored)
        constexpr int E = 4;
        uint32_t n[2], c0[2][E];
        float4 v[2][E];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const size_t list = q * nslots + (s0 + 64 * r < nslots ? s0 + 64 * r : s0);
            n[r] = counts[list];
#pragma unroll
            for (int i = 0; i < E; ++i) {
                v[r][i] = ent[4 * (list * cap + i) + g];
                c0[r][i] = ids[list * cap + i];
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (s0 + 64 * r >= nslots) break;
            if (n[r] > (uint32_t)cap) {
                s_over = 1;
                continue;
            }
#pragma unroll
            for (int i = 0; i < E; ++i)
                if ((uint32_t)i < n[r]) take(v[r][i], c0[r][i]);
            for (uint32_t i = E; i < n[r]; ++i) {
                const size_t at = (q * nslots + s0 + 64 * r) * cap + i;
                take(ent[4 * at + g], ids[at]);
            }
        }
    }
    __syncthreads();
    const int na = (int)s_n;
    if (s_over != 0 || na > CH_PICK || na < k) {
        if (threadIdx.x == 0) atomicOr(flag, 1);
        return;
    }
    if (threadIdx.x < QADC_WAVE) qadc_wave_select_bin(hist, (uint32_t)k, 0u, sel);
    __syncthreads();
    // the k-th smallest lies in bin sel[0]: nothing within it exceeds `top`
    const float top = (sel[0] >= 255u ? bound : fminf(bound, lo + (float)(sel[0] + 1) / scale * 1.0001f + fabsf(lo) * 1e-6f)) + 2.0f * e;
    for (int i = threadIdx.x; i < na; i += 256)
        if (__uint_as_float((uint32_t)(A[i] >> 32)) <= top) {
            const uint32_t pos = atomicAdd(&s_m, 1u);
            if (pos < CS_MAX_NPROBE + 512) cand[pos] = (uint32_t)A[i];
        }
    __syncthreads();
    const int nc = (int)s_m;
    if (nc > CS_MAX_NPROBE + 512) {
        if (threadIdx.x == 0) atomicOr(flag, 1);
        return;
    }
    // exact scores: the chain of the definition, one cell per thread
    for (int i = threadIdx.x; i < nc; i += 256) {
        const uint32_t c = cand[i];
        const float *p = centroids + (size_t)c * d;
        float acc = 0.0f;
        int t = 0;
        if (vec) {  // rows on 16-byte boundaries
            for (; t + 32 <= d; t += 32) {
                float4 v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = *(const float4 *)(p + t + 4 * j);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    acc = __fmaf_rn(zs[t + 4 * j], v[j].x, acc);
                    acc = __fmaf_rn(zs[t + 4 * j + 1], v[j].y, acc);
                    acc = __fmaf_rn(zs[t + 4 * j + 2], v[j].z, acc);
                    acc = __fmaf_rn(zs[t + 4 * j + 3], v[j].w, acc);
                }
            }
        }
        for (; t < d; ++t) acc = __fmaf_rn(zs[t], p[t], acc);
        A[i] = ((uint64_t)qadc_f2ord(__fmaf_rn(-2.0f, acc, cnorm[c])) << 32) | c;
    }
    __syncthreads();
    cs_rank_and_write(A, nc, k, nprobe, probe_ids + q * nprobe, probe_scores ? probe_scores + q * nprobe : nullptr);
}

// -------------------------------------------------------------------- host ---
#define CH_TILES 32   // tiles of 32 cells per k_cscan block and candidate list
#define CH_CAP 16     // entries (16 cells each) per list
#define CH_MAX_S 18   // steps of 16 columns: d <= CH_MAX_D and four more
static int ch_steps(int d) { return d + 4 <= 7 * 16 ? 7 : (d + 4 <= 9 * 16 ? 9 : CH_MAX_S); }

static int64_t ch_pilot_most(int K) { return (K / 4 < 65536 ? K / 4 : 65536) & ~2047; }

// The score matrix is idle until the exact form has to take a pass over, so what only one pass needs lies
// in it (about half of it: a list's entries are 2 bytes per query and cell, the matrix 4).  The cells'
// operand outlives a pass; it follows the lists where there is a single one, and else the matrix.
// 65,536 cells, d = 96, 4096 queries: 14 MB behind the matrix of 1 GiB (0.6 GB with all of it there).
static void ch_layout(CoarseHalf &p, int nq, int qc, int K, size_t matrix_bytes) {
    const size_t q = (size_t)qc;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t r = at;
        at += cs_up256(bytes);
        return r;
    };
    p.minima = take(q * (size_t)(p.P / 16) * 4);
    p.qs = take((q + 31) / 32 * (size_t)p.S * 1024);
    p.err = take(q * 4);
    p.bounds = take(q * 8);
    p.ent = take(q * (size_t)p.nslots * CH_CAP * 64);
    p.ids = take(q * (size_t)p.nslots * CH_CAP * 4);
    p.counts = take(q * (size_t)p.nslots * 4);
    if (nq > qc && at < matrix_bytes) at = matrix_bytes;
    p.cells = take((size_t)p.ntiles * (size_t)p.S * 1024);
    if (at < matrix_bytes) at = matrix_bytes;  // (read by the exact form's kernels, or by the next pass)
    p.bmax = take(((size_t)K / 256 + 1) * 4);
    p.bnorm = take(((size_t)K / 256 + 1) * 4);
    p.flag = take(4);
    p.total = at;
}

// When it wins over the fp32 forms; figures in us, those / this one.  It costs the conversion of all cells,
// which a batch has to pay for, and its steps are made for 108, 140 and 252 dimensions, whatever d is:
// `fill` of 100 columns are used.  The fp32 products take tiles of 128 queries, one or many.
//   up to 128 queries     d = 96, nprobe 20: 16,384 cells 63 / 54, 32,768: 64 / 58; nprobe 64: 65,536 cells 72 / 76,
//                         262,144: 137 / 156
//   129 .. 256            65,536 cells, nprobe 64, 160 queries: d = 96 84 / 76, d = 64 69 / 71, d = 144 117 / 114
//   from 257 on           65,536 cells, 512 queries: d = 64 101 / 74, d = 144 175 / 119, d = 32 77 / 66, but with 32,768
//                         cells and d = 32 no gain (1.01); 1000 queries 117 / 78
// Few dimensions over many cells: the error bound takes in so many cells that the lists overflow and the
// exact form follows (byte-range data, d = 16, 10^6 cells: 12 times the time of the fp32 form).
static bool ch_sizes(int nq, int K) {
    return nq >= 64 && K >= 16384 && K <= (nq <= 128 ? 32768 : (1 << 20));
}
static bool ch_pays(int nq, int K, int d) {
    const int fill = 100 * d / (16 * ch_steps(d));
    if (!ch_sizes(nq, K)) return false;
    if (nq <= 256) return fill >= 65;
    return fill >= 40 || (d >= 16 && nq >= 1000 && K <= 131072);
}

CoarseHalf qadc_coarse_half_plan(int nq, int qc, int K, int d, int nprobe, size_t matrix_bytes, size_t room) {
    CoarseHalf p = {};
    if (qadc_option(PQ_OPT_COARSE_FILTER) == 0 || d > CH_MAX_D || !ch_pays(nq, K, d)) return p;
    // The pilot: 256 cells per result, at most a quarter of all.  Fewer than 192 per result and the lists
    // (16 entries, about 512 nprobe / P of them used on average) overflow now and then, which costs the
    // pass the exact form: 16,384 cells, nprobe 64 (P = 4096), 4000 queries: 459 us, exact form at once 260.
    // Over all cells about nprobe K / P lie within its bound; k_cpick holds 2048, so the pilot grows with K,
    // for a quarter of that, or five eighths where it cannot (262,144 cells, nprobe 300, 1000 queries: 301 us, fp32
    // 704; 10^6 cells, nprobe 64, 1000 queries: P = 16,384 left
    // 3900, and every pass went to the exact form as well: 5970 us, fp32 2620, with P = 65,536 1140).
    int64_t P = 256 * (int64_t)nprobe > 16384 ? 256 * (int64_t)nprobe : 16384;
    const int64_t near = nprobe * (int64_t)K;
    if (P * (CH_PICK / 4) < near) P = (near / (CH_PICK / 4) + 2047) & ~(int64_t)2047;
    if (P > ch_pilot_most(K)) P = ch_pilot_most(K);
    P &= ~(int64_t)2047;
    if (P < 192 * (int64_t)nprobe || P * (CH_PICK / 8 * 5) < near) return p;
    p.S = ch_steps(d);
    p.P = (int)P;
    p.ntiles = (K + 31) / 32;
    p.nslots = 2 * ((p.ntiles + CH_TILES - 1) / CH_TILES);
    ch_layout(p, nq, qc, K, matrix_bytes);
    p.use = p.total <= room;
    return p;
}

size_t qadc_coarse_half_bytes(int nq, int qc, int K, size_t matrix_bytes) {
    if (!ch_sizes(nq, K)) return 0;
    CoarseHalf p = {};
    p.S = CH_MAX_S;
    p.P = (int)ch_pilot_most(K);
    p.ntiles = (K + 31) / 32;
    p.nslots = 2 * ((p.ntiles + CH_TILES - 1) / CH_TILES);
    ch_layout(p, nq, qc, K, matrix_bytes);
    return p.total;
}

int qadc_coarse_cells(const float *centroids, int K, int d, const CoarseHalf &hp, float *cnorm, char *base, hipStream_t s) {
    const int nb = (K + 255) / 256;
    float *bmax = hp.use ? (float *)(base + hp.bmax) : nullptr, *bnorm = hp.use ? (float *)(base + hp.bnorm) : nullptr;
    hipLaunchKernelGGL(k_cstat, dim3(nb), dim3(256), 0, s, centroids, K, d, cnorm, bmax, bnorm);
    QADC_LAUNCH_CHECK("k_cstat");
    if (!hp.use) return PQ_OK;
    hipLaunchKernelGGL(k_cprep, dim3(hp.ntiles < 2048 ? hp.ntiles : 2048), dim3(256), 0, s, centroids, K, d, hp.S, (const float *)cnorm,
                       (const float *)bmax, nb, (uint4 *)(base + hp.cells), hp.ntiles);
    QADC_LAUNCH_CHECK("k_cprep");
    return PQ_OK;
}

int qadc_coarse_half_pass(const float *queries, int nqc, const float *centroids, int K, int d, int nprobe,
                          const CoarseHalf &hp, const float *cnorm, char *base, int32_t *probe_ids,
                          float *probe_scores, hipStream_t s) {
    const int nb = (K + 255) / 256, nqt = (nqc + 31) / 32;
    float *minima = (float *)(base + hp.minima);
    int *flag = (int *)(base + hp.flag);
    const u32x4 *cells = (const u32x4 *)(base + hp.cells);
    uint4 *qs = (uint4 *)(base + hp.qs);
    float *err = (float *)(base + hp.err);
    float2 *bounds = (float2 *)(base + hp.bounds);
    uint4 *ent = (uint4 *)(base + hp.ent);
    uint32_t *ids = (uint32_t *)(base + hp.ids), *counts = (uint32_t *)(base + hp.counts);
    hipLaunchKernelGGL(k_qprep, dim3(nqt), dim3(256), 0, s, queries, nqc, d, hp.S, (const float *)(base + hp.bmax),
                       (const float *)(base + hp.bnorm), nb, qs, err);
    QADC_LAUNCH_CHECK("k_qprep");
#define CH_SCAN(SV, NCOLV, PILOTV, NT, TILES)                                                                            \
    hipLaunchKernelGGL((k_cscan<SV, NCOLV, PILOTV>), dim3(((NT) + (TILES) - 1) / (TILES), (nqt + 4 * NCOLV - 1) / (4 * NCOLV)), \
                       dim3(256), 0, s, cells, NT, TILES, (const uint4 *)qs, nqc, (const float2 *)bounds,               \
                       (uint32_t *)minima, hp.P / 16, ent, ids, counts, hp.nslots, CH_CAP)
    // as many query tiles per wave as leave two waves per SIMD
#define CH_SCAN_S(SV, MOST, PILOTV, NT, TILES)                                                                  \
    do {                                                                                                        \
        const int blocks1 = (((NT) + (TILES) - 1) / (TILES)) * ((nqt + 3) / 4);                                 \
        if (MOST >= 4 && blocks1 >= 2048) CH_SCAN(SV, (MOST >= 4 ? 4 : 1), PILOTV, NT, TILES);                   \
        else if (MOST >= 2 && blocks1 >= 1024) CH_SCAN(SV, (MOST >= 2 ? 2 : 1), PILOTV, NT, TILES);              \
        else CH_SCAN(SV, 1, PILOTV, NT, TILES);                                                                 \
    } while (0)
#define CH_SCAN_ANY(PILOTV, NT, TILES)                                  \
    do {                                                                \
        if (hp.S == 7) CH_SCAN_S(7, 4, PILOTV, NT, TILES);              \
        else if (hp.S == 9) CH_SCAN_S(9, 2, PILOTV, NT, TILES);         \
        else CH_SCAN_S(CH_MAX_S, 1, PILOTV, NT, TILES);                 \
    } while (0)
    CH_SCAN_ANY(true, hp.P / 32, 8);
    QADC_LAUNCH_CHECK("k_cscan (pilot)");
#define CH_BOUND(NV)                                                                                             \
    hipLaunchKernelGGL(k_cbound<NV>, dim3((nqc + 3) / 4), dim3(256), 0, s, (const float *)minima, hp.P / 16, nqc, nprobe, \
                       (const float *)err, bounds, flag)
    if (hp.P <= 8192) CH_BOUND(8); else if (hp.P <= 16384) CH_BOUND(16); else if (hp.P <= 32768) CH_BOUND(32); else CH_BOUND(64);
    QADC_LAUNCH_CHECK("k_cbound");
    CH_SCAN_ANY(false, hp.ntiles, CH_TILES);
    QADC_LAUNCH_CHECK("k_cscan");
    const int vec = (d % 4 == 0) && ((uintptr_t)centroids & 15u) == 0;
    hipLaunchKernelGGL(k_cpick, dim3(nqc), dim3(256), 0, s, queries, centroids, K, d, nprobe, cnorm, (const float4 *)ent,
                       (const uint32_t *)ids, (const uint32_t *)counts, hp.nslots, CH_CAP, (const float2 *)bounds,
                       (const float *)err, vec, probe_ids, probe_scores, flag);
    QADC_LAUNCH_CHECK("k_cpick");
    return PQ_OK;
}
