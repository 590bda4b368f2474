#pragma once
// The search with a bound that tightens from list to list (see k_ivf_tight in ivf.hip) for the fixed shape: 16 x 4 bits over
// equal sub-spaces of DS dimensions, 8-bit tables, up to 64 NR results.
//
// A query's lists are a chain (each is quantized against the bound that the ones before left), so what counts is the length of
// a list's steps.  A block of eight waves serves a query:
//   - Tables two lists at a time, without LDS: wave w holds sub-quantizers 2 w and 2 w + 1, the 32 entries of code byte w, of one list in its lower and of
//     the next in its upper half; centroids are requested a pair ahead.  Only the minima go through LDS, to d_min.
//   - Quantized entries meet by lane moves in the byte-indexed table of the wave's code byte.
//   - The R smallest distances are kept in order in the registers of one wave; a new one is inserted by a shift and a minimum and a
//     maximum.  Words (distance, id) of all candidates gather in LDS and are ranked once at the end.  A candidate's id is not needed
//     before that, so its load is taken up only behind the next list's set-up.
//   - Three barriers a list: tables ready, codes scanned, bound known (with the next list's quantizer and the next pair's minima).
// One wave keeps the bound and makes the quantizers: every wave for itself, the fp64 sums and division cost more than the tables.  Nothing
// may spill: a register read back from scratch memory waits for every load before it, the next list's codes among them.
// What bounds it: LDS reads of the codes (eight a code; 16 lanes a clock less conflicts: 160 us of them) and, as all queries are served at
// once, the block with the longest lists.  1000 queries x 64 probes over 10^8 codes in 65,536 lists, d = 96, R = 100: the kernel 490 -> 385 us,
// coarse search and calibration included 610 -> 510; a block's time (stamps, average of all) 353 -> 288 us, of which scans 204 -> 111, tables and
// quantizers 96 -> 90, candidates 53 -> 58, waiting 0 -> 41; one query, 128 probes, 2.9 * 10^6 codes 2333 -> 1486 (1677 where the compiler
// waits for every other read of a code).
#include "fill_level.h"
#include "quotient.h"
#include "scan_device.h"

#define TIGHTF_THREADS 512
#define TIGHTF_CAP 2048     // candidate words; a list segment that overflows them is scanned again in batches, between which they are cut back
#define TIGHTF_INSERT 48    // distances that a list inserts one by one at most (up to a wave's 64); beyond, the order is made anew
#define TIGHTF_SEGMENT 4096  // codes between two looks at the fill level
#define TIGHTF_U 4          // codes per thread and round
#define TIGHTF_PC 64        // probes whose cells and list bounds are fetched together, one per lane

// What a list is quantized and scanned with, made by the leading wave.
struct __align__(8) TightList {
    double delta;
    float fdelta, fdmin;
    uint32_t skip, pad;
};

template <int DS, int NR>
struct TightLds {
    uint64_t A[TIGHTF_CAP];       // ordered distance << 32 | id (of the newest list: place in the list)
    __align__(16) uint32_t gtab[512];
    __align__(16) float pmin[2][2][16];
    __align__(16) float cb[256 * DS], z[16 * DS], cen[2][16 * DS];
    __align__(16) uint32_t hist[256];
    uint32_t kmem[QADC_KTH_MEM], sel[8];
    uint32_t order[64 * NR];      // the R smallest distances in ascending order; none: all ones
    int64_t plo[TIGHTF_PC];
    int32_t plen[TIGHTF_PC], pcell[TIGHTF_PC];
    TightList list[2];
    uint32_t na, thr, cnt;
    int nlists;
};
struct TightHi {  // the distances of the words, as the selection wants them
    const uint64_t *A;
    __device__ __forceinline__ uint32_t operator[](int i) const { return (uint32_t)(A[i] >> 32); }
};

template <int DS, int NR>
__global__ void __launch_bounds__(TIGHTF_THREADS) __attribute__((amdgpu_waves_per_eu(8)))
k_ivf_tight_fix(const float *__restrict__ cb, const float *__restrict__ coarse, const int64_t *__restrict__ list_offsets,
                const uint8_t *__restrict__ list_codes, const int32_t *__restrict__ list_ids, const float *__restrict__ queries,
                const int32_t *__restrict__ probe_ids, int nprobe, int K, int R, const char *__restrict__ ws, size_t per_query,
                int32_t *__restrict__ out_ids, float *__restrict__ out_dist) {
    constexpr int NT = TIGHTF_THREADS, CAP = TIGHTF_CAP, U = TIGHTF_U, d = 16 * DS;
    __shared__ TightLds<DS, NR> S;
    static_assert(64 * NR <= QADC_KTH_MEM, "the smaller ones lie in the room of the selection's members");
    const size_t q = blockIdx.x;
    const int32_t *probes = probe_ids + q * nprobe;
    const int tid0 = (int)threadIdx.x, lane0 = tid0 % QADC_WAVE, wave = __builtin_amdgcn_readfirstlane(tid0 / QADC_WAVE);
    // The thread, its lane, and a lane's list of the pair, entry and sub-quantizer; addresses that hang on them are worked out anew in every
    // part of the loop, as the compiler would otherwise hold them all, and 64 registers are few.
#define TIGHTF_THREAD                 \
    int tid = tid0, lane = lane0;     \
    asm volatile("" : "+v"(tid), "+v"(lane)); \
    (void)tid, (void)lane
#define TIGHTF_LANE                                                     \
    TIGHTF_THREAD;                                                      \
    const int par = lane >> 5, e = lane & 31, j = 2 * wave + (e >> 4);  \
    (void)par, (void)e, (void)j
    float cur = ((const IvfState *)(ws + q * per_query))->dmax;
    const int tid = tid0, lane = lane0;
    for (int i = tid; i < 256 * DS; i += NT) S.cb[i] = cb[i];
    if (tid < d) S.z[tid] = queries[q * d + tid];
    if (tid < 64 * NR) S.order[tid] = 0xffffffffu;
    const int leader = (int)(blockIdx.x >> 8) & 7;  // the wave that keeps the bound: another one for each of a CU's blocks, so that they spread over its SIMDs
    int na = 0;                  // words in A
    int pend_at = -1;            // a word of A whose id is on its way
    int32_t pend_id = 0;
    if (tid == 0) {
        S.na = 0;
        S.thr = 0xffffffffu;
    }
    auto take_pending = [&] {
        if (pend_at >= 0) ((uint32_t *)&S.A[pend_at])[0] = (uint32_t)pend_id;
        pend_at = -1;
    };
    // the order from all words (all threads)
    auto reorder = [&] {
        TIGHTF_THREAD;
        const int k = na < R ? na : R;
        const TightHi hi{S.A};
        const uint32_t kth = qadc_block_kth_f32(hi, na, k, S.hist, S.sel, S.kmem);
        if (tid == 0) S.cnt = 0;
        __syncthreads();
        for (int i = tid; i < na; i += NT)
            if (hi[i] < kth) S.kmem[atomicAdd(&S.cnt, 1u)] = hi[i];  // (fewer than k <= 64 NR)
        __syncthreads();
        const int nb = (int)S.cnt;
        for (int i = tid; i < 64 * NR; i += NT) {
            if (i < nb) {
                const uint32_t mine = S.kmem[i];
                int rank = 0;
                for (int k2 = 0; k2 < nb; ++k2) rank += (S.kmem[k2] < mine || (S.kmem[k2] == mine && k2 < i)) ? 1 : 0;
                S.order[rank] = mine;
            } else {
                S.order[i] = i < k ? kth : 0xffffffffu;
            }
        }
        __syncthreads();
    };
    for (int a0 = 0; a0 < nprobe; a0 += TIGHTF_PC) {
        __syncthreads();  // the previous chunk's entries have been used
        if (wave == 0) {  // the lists that hold codes, in probe order
            TIGHTF_THREAD;
            const int a = a0 + lane, c = a < nprobe ? probes[a] : -1;
            const bool valid = c >= 0 && c < K;
            const int64_t lo = valid ? list_offsets[c] : 0, hi = valid ? list_offsets[c + 1] : 0;
            const uint64_t m = __ballot(hi > lo);
            if (hi > lo) {
                const int at = __popcll(m & ((1ull << lane) - 1ull));
                S.pcell[at] = c;
                S.plo[at] = lo;
                S.plen[at] = (int32_t)(hi - lo);  // a list is shorter than 2^31 codes
            }
            if (lane == 0) S.nlists = __popcll(m);
        }
        __syncthreads();
        const int nl = S.nlists;
        if (nl == 0) continue;
        // the centroids of lists a and a + 1, on their way in a register of the first 2 d threads
        float cc = 0.0f;
        auto request_centroids = [&](int a) {  // (a < nl)
            TIGHTF_THREAD;
            if (tid < 2 * d) cc = coarse[(size_t)S.pcell[tid < d || a + 1 >= nl ? a : a + 1] * d + (tid < d ? tid : tid - d)];
        };
        auto put_centroids = [&] {
            TIGHTF_THREAD;
            if (tid < 2 * d) (&S.cen[0][0])[tid] = cc;
        };
        uint2 wn[U];
        auto request = [&](int a, int base) {  // codes past the end: the last one again
            TIGHTF_THREAD;
            const uint8_t *p = list_codes + S.plo[a] * 8;
            const int last = S.plen[a] - 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = base + u * NT + tid;
                wn[u] = *(const uint2 *)(p + (size_t)(uint32_t)(i < last ? i : last) * 8);
            }
        };
        float tv, pm, tv2 = 0.0f, pm2 = 0.0f;  // this pair's entry and minimum, and the next one's
        // eq. (1) for lists a and a + 1, terms in ascending order, and the sub-quantizers' minima (squares: the bit patterns order as integers)
        auto tables = [&](int a, float &to, float &min_to) {
            TIGHTF_LANE;
            float acc = 0.0f;
#pragma unroll
            for (int t = 0; t < DS; ++t) {
                const float diff = __fsub_rn(__fsub_rn(S.z[j * DS + t], S.cen[par][j * DS + t]), S.cb[(j * 16 + (e & 15)) * DS + t]);
                acc = __fadd_rn(acc, __fmul_rn(diff, diff));
            }
            uint32_t mb = __float_as_uint(acc);
            mb = min(mb, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mb, 0xB1, 0xf, 0xf, true));   // quad_perm [1,0,3,2]
            mb = min(mb, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mb, 0x4E, 0xf, 0xf, true));   // quad_perm [2,3,0,1]
            mb = min(mb, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mb, 0x141, 0xf, 0xf, true));  // row_half_mirror
            mb = min(mb, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mb, 0x140, 0xf, 0xf, true));  // row_mirror
            to = acc;
            min_to = __uint_as_float(mb);
            if ((e & 15) == 0) S.pmin[(a >> 1) & 1][par][j] = min_to;
        };
        // the leader: the quantizer of list a against the bound
        double dm = 0.0;  // d_min of the pair's lists, each in its half of the lanes
        auto quantizer = [&](int a) {
            TIGHTF_LANE;
            if ((a & 1) == 0) {  // fp64, ascending
                const float4 *v = (const float4 *)S.pmin[(a >> 1) & 1][par];
                dm = 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 x = v[i];
                    dm = dm + (double)x.x;
                    dm = dm + (double)x.y;
                    dm = dm + (double)x.z;
                    dm = dm + (double)x.w;
                }
            }
            const unsigned long long db = (unsigned long long)__double_as_longlong(dm);
            const double dmin = __longlong_as_double((long long)(((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(db >> 32), 32 * (a & 1)) << 32) |
                                                                 (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)db, 32 * (a & 1))));
            double delta = ((double)cur - dmin) / 255.0;
            if (!((delta > 0.0) && isfinite(delta))) delta = 0.0;
            if (lane == 0) S.list[a & 1] = TightList{delta, (float)delta, (float)dmin, dmin >= (double)cur ? 1u : 0u, 0u};  // Section 3.4: nothing in a list from d_min on is closer
        };
        request_centroids(0);
        request(0, 0);
        put_centroids();
        __syncthreads();
        tables(0, tv, pm);
        if (nl > 2) request_centroids(2);
        __syncthreads();
        if (wave == leader) quantizer(0);
        __syncthreads();
        for (int ai = 0; ai < nl; ++ai) {
            const int p = ai & 1;
            const TightList li = S.list[p];
            const bool skip = __builtin_amdgcn_readfirstlane((int)li.skip) != 0;
            if (p == 0 && ai + 2 < nl) put_centroids();  // (the pair before has been read before the last barrier)
            if (skip) {
                if (ai + 1 < nl) request(ai + 1, 0);
                if (p == 0 && ai + 2 < nl) __syncthreads();
            } else {
                TIGHTF_LANE;
                // floor((p - p_min) / delta) in fp32 where that cannot differ, else (or with a delta not of ordinary size) in fp64
                const float x32 = (tv - pm) * __builtin_amdgcn_rcpf(li.fdelta);
                uint32_t qv = (uint32_t)fminf(x32, 255.0f);
                if (par == p && !(li.fdelta > 1e-30f && li.fdelta < 1e30f && quotient_sure(x32, QUOTIENT_SLACK_RCP))) {
                    qv = 0;
                    if (li.delta > 0.0) {
                        const double x = floor(((double)tv - (double)pm) / li.delta);
                        qv = x >= 255.0 ? 255u : (uint32_t)x;
                    }
                }
                // entries 4 lane .. 4 lane + 3 of code byte `wave`: four of the lower nibble's, side by side, and one of the upper's
                uint32_t lq = qv << (8 * (lane & 3));
                lq |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lq, 0xB1, 0xf, 0xf, true);
                lq |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lq, 0x4E, 0xf, 0xf, true);
                lq = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (32 * p + 4 * (lane & 3)), (int)lq);
                const uint32_t hq = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (32 * p + 16 + (lane >> 2)), (int)qv) * 0x10001u;
                const mq_u16x2 most = {255, 255};
                const uint32_t ev = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(mq_u16x2, (lq & 0x00ff00ffu) + hq), most));
                const uint32_t od = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(mq_u16x2, ((lq >> 8) & 0x00ff00ffu) + hq), most));
                S.gtab[64 * wave + lane] = ev | (od << 8);
                __syncthreads();
                take_pending();
                const int len = __builtin_amdgcn_readfirstlane(S.plen[ai]);
                const int64_t lo = S.plo[ai];
                const uint8_t *gtab = (const uint8_t *)S.gtab;
                const float fdelta = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(li.fdelta)));
                const float fdmin = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(li.fdmin)));
                auto append = [&](uint32_t sum, int i) {
                    const uint32_t at = atomicAdd(&S.na, 1u);
                    if (at < (uint32_t)CAP) S.A[at] = ((uint64_t)qadc_f2ord(fmaf((float)sum, fdelta, fdmin)) << 32) | (uint32_t)i;
                };
                const int before = na;
                int known = na;       // words up to here have their ids
                uint32_t lim = 255u;  // keys below it are candidates
                bool again = false;   // the order is made anew
                // In segments, behind which a list that adds many candidates is cut back to the R smallest.
                for (int s0 = 0; s0 < len;) {
                    const int s1 = len - s0 > TIGHTF_SEGMENT ? s0 + TIGHTF_SEGMENT : len;
                    for (int base = s0; base < s1; base += U * NT) {
                        TIGHTF_THREAD;
                        uint2 w[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) w[u] = make_uint2(qadc_move(wn[u].x), qadc_move(wn[u].y));
                        if (len - base > U * NT) request(ai, base + U * NT);
                        else if (ai + 1 < nl) request(ai + 1, 0);
#pragma unroll
                        for (int u = 0; u < U; u += 2)
                            if (base + u * NT + wave * QADC_WAVE < len) {
                                uint32_t sum[2];
                                sum8_pair(gtab, gtab, w[u], w[u + 1], sum);
                                const int i = base + u * NT + tid;
                                const bool one = i < len && sum[0] < lim, two = i < len - NT && sum[1] < lim;
                                if (__ballot(one || two) != 0) {
                                    if (one) append(sum[0], i);
                                    if (two) append(sum[1], i + NT);
                                }
                            }
                        if (base > 0x7fffffff - U * NT) break;
                    }
                    int total = (int)fill_level([&] { return S.na; }, s1 < len, [] { __syncthreads(); });
                    const bool over = total > CAP;
                    if (!over && (s1 == len || total <= CAP / 2)) {
                        na = total;
                        s0 = s1;
                        continue;
                    }
                    // the words' ids, and the R smallest of them
                    TIGHTF_THREAD;
                    if (over) total = na;  // what the segment has added is dropped, and it is scanned again below
                    for (int i = known + tid; i < total; i += NT) ((uint32_t *)&S.A[i])[0] = (uint32_t)list_ids[lo + (uint32_t)S.A[i]];
                    __syncthreads();
                    if (tid == 0) S.na = (uint32_t)total;
                    na = total;
                    uint64_t most = ~0ull;
                    __syncthreads();
                    for (int base = over ? s0 : s1; base < s1; base += NT) {  // in batches that surely fit
                        if (na + NT > CAP) {  // na > R here
                            most = ivf_keep<CAP, NT>(S.A, na, R, S.hist, S.sel, &S.na);
                            na = R;
                        }
                        const int i = base + tid;
                        if (i < s1) {
                            const uint2 w = *(const uint2 *)(list_codes + (lo + i) * 8);
                            const uint32_t sum = sum8(gtab, w.x, w.y);
                            if (sum < lim) {
                                const uint64_t word = ((uint64_t)qadc_f2ord(fmaf((float)sum, fdelta, fdmin)) << 32) | (uint32_t)list_ids[lo + i];
                                if (word <= most) S.A[atomicAdd(&S.na, 1u)] = word;
                            }
                        }
                        __syncthreads();
                        na = (int)S.na;
                        __syncthreads();
                        if (base > 0x7fffffff - NT) break;
                    }
                    if (na > R) {
                        most = ivf_keep<CAP, NT>(S.A, na, R, S.hist, S.sel, &S.na);
                        na = R;
                    }
                    known = na;
                    again = true;
                    // keys whose distance is within the R-th (distances do not decrease with the key)
                    lim = 0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int k = lane + 64 * r;
                        lim += (uint32_t)__popcll(__ballot(k < 255 && qadc_f2ord(fmaf((float)k, fdelta, fdmin)) <= (uint32_t)(most >> 32)));
                    }
                    s0 = s1;
                }
                // the ids of the new words: up to one per thread of the other waves on its way, the rest at once
                if (wave != leader) {
                    TIGHTF_THREAD;
                    int i = known + ((tid - QADC_WAVE * (leader + 1)) & (NT - 1));
                    if (i < na) {
                        pend_id = list_ids[lo + (uint32_t)S.A[i]];
                        pend_at = i;
                    }
                    for (i += NT - QADC_WAVE; i < na; i += NT - QADC_WAVE)
                        ((uint32_t *)&S.A[i])[0] = (uint32_t)list_ids[lo + (uint32_t)S.A[i]];
                }
                again = again || na - before > TIGHTF_INSERT;
                if (again) reorder();
                if (wave == leader) {
                    TIGHTF_THREAD;
                    uint32_t D[NR];  // place 64 r + lane in D[r]
#pragma unroll
                    for (int r = 0; r < NR; ++r) D[r] = S.order[64 * r + lane];
                    if (!again && na > before) {
                        const uint32_t x = lane < na - before ? (uint32_t)(S.A[before + lane] >> 32) : 0xffffffffu;
                        for (int i = 0; i < na - before; ++i) {  // the places above the new one move up
                            const uint32_t xs = (uint32_t)__builtin_amdgcn_readlane((int)x, i);
#pragma unroll
                            for (int r = NR - 1; r >= 0; --r) {
                                const uint32_t first = r > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)D[r > 0 ? r - 1 : 0], 63) : 0u;
                                const uint32_t under = (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)D[r], 0x138, 0xf, 0xf, false);  // wave_shr:1
                                D[r] = max(under, min(xs, D[r]));
                            }
                        }
#pragma unroll
                        for (int r = 0; r < NR; ++r) S.order[64 * r + lane] = D[r];
                    }
                    uint32_t thr = 0;  // the R-th
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        if (r == (R - 1) / 64) thr = (uint32_t)__builtin_amdgcn_readlane((int)D[r], (R - 1) & 63);
                    if (lane == 0) S.thr = thr;
                    if (thr != 0xffffffffu) {
                        const float worst = qadc_ord2f(thr);
                        cur = worst < cur ? worst : cur;
                    }
                }
            }
            // (the pair after this one's tables during its first list, so that their minima are there when its second's bound is known)
            if (p == 0 && ai + 2 < nl) tables(ai + 2, tv2, pm2);
            if (p == 1 && ai + 3 < nl) request_centroids(ai + 3);
            if (p == 1) {
                tv = tv2;
                pm = pm2;
            }
            if (wave == leader && ai + 1 < nl) quantizer(ai + 1);
            __syncthreads();
        }
        take_pending();
    }
    const uint32_t thr = S.thr;
    // the words up to the R-th distance, and of these the R smallest by (distance, id)
    __syncthreads();
    {
    TIGHTF_THREAD;
    constexpr int PER = CAP / NT;
    uint64_t mine[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) mine[u] = tid + u * NT < na ? S.A[tid + u * NT] : ~0ull;
    if (tid == 0) S.cnt = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (tid + u * NT < na && (uint32_t)(mine[u] >> 32) <= thr) S.A[atomicAdd(&S.cnt, 1u)] = mine[u];
    __syncthreads();
    // (equal words, which repeated ids give, in the order of their places)
    const int nf = (int)S.cnt;
    for (int i = tid; i < nf; i += NT) {
        const uint64_t w = S.A[i];
        int rank = 0;
#pragma unroll 4
        for (int k = 0; k < nf; ++k) rank += (S.A[k] < w || (S.A[k] == w && k < i)) ? 1 : 0;
        if (rank < R) {
            out_ids[q * R + rank] = (int32_t)(uint32_t)w;
            out_dist[q * R + rank] = qadc_ord2f((uint32_t)(w >> 32));
        }
    }
    for (int r = (nf < R ? nf : R) + tid; r < R; r += NT) {
        out_ids[q * R + r] = -1;
        out_dist[q * R + r] = INFINITY;
    }
    }
}
