#pragma once
// Size rules of the quantizer, the scan and the inverted-list search.  Plain C++, so that the lines can be checked without a GPU.
#include <stdint.h>

// Whether k_quantize runs blocks of 1024 threads: a block's time is a chain of dependent steps, each shorter with more
// threads, but a wide block waits for half of a CU to become free, beside other streams' scans and beside other
// blocks of its own.  us a call, 256 / 1024 threads, one stream and per call on four (8 x 8: m x 8 bits):
//   one block does a query's whole work (batches for the matrix cores, no scratch memory), 2 * 10^6 codes, R = 100: 16 x 4 bits, 192
//     queries 62.7 / 62.0 and 48.5 / 49.8; 320: 101 / 105 and 81 / 84; {6,6,4} x 4, 256: 139 / 134 and
//     117 / 118; 320: 184 / 189 and 147 / 153 (k_quantize itself, 32 queries: 22 / 15.2): up to one block per CU
//   ... and counts a pilot too (tables quantized for inspection; since then k_pilot4 has taken over above 256 queries what its kinds of codes and
//     16,384 codes of pilot allow), 10^6 codes: 300 queries 16 x 4 59 / 52, 40-bit 117 / 77, 8 x 8 145 / 98, {6,6,4} x 8
//     279 / 209; 256: 53 / 28, 112 / 40, 139 / 51, 240 / 107: up to two
//   one query over 128 blocks, R = 100: 16 x 4 bits, 10^7 codes 34.9 / 32.6 and 12.7 / 15.3: not with short calibrations
//   ... more than 1024 calibration codes: one query, 10^6 codes, R = 257: 16 x 4 bits 30.2 / 27.1 and 16.8 / 15.7, 40-bit codes 41.2 / 32.3
//     and 21.9 / 17.7; two: 37.8 / 35.3 and 23.2 / 24.1, 52.2 / 43.3 and 30.9 / 30.6, 8 x 8 55.8 / 48.5 and 33.7 / 35.5; four: 43.0 / 47.5
//     and 27.6 / 34.4, 57.2 / 60.9 and 34.0 / 44.2: up to one block per CU
//   ... R = 1000, four queries (two blocks per CU), 10^6 codes: 40-bit 87.2 / 77.3 and 61.0 / 60.3, 32 x 4 68.0 / 66.3 and 54.0 / 50.1; 16 x 4
//     55.4 / 55.8 and 36.9 / 41.5; R = 2000: 128.7 / 105.7 and 106 / 84, 95.3 / 88.8 and 72.4 / 66.5, 74.4 / 72.4 and 54.2 / 53.0: long
//     calibrations, whose chain outweighs it (later where look-ups are cheap)
inline bool quantize_wide(int64_t blocks, int blocks_per_query, int calibration, int pilot, bool cheap_lookups) {
    if (blocks_per_query == 1) return blocks <= (pilot > 0 ? 512 : 256);
    return calibration > 1024 && blocks <= (calibration > (cheap_lookups ? 4096 : 2048) ? 512 : 256);
}

// Threads of k_ivf_calib's blocks, one query each (the pilot's look-ups and the selections shorten with them): 1024 up to one block per CU,
// 512 up to two, else 256.  us a call with 256 / 512 / 1024 threads (- : not taken), one stream; per call on four:
//   2 * 10^6 codes, 4096 lists, 32 probes, R = 100, 16 x 4 bits: 1 query 46.7 / - / 42.1; 24.0 / - / 21.9; 256 83.8 / - / 80.4; 46.4 / - / 47.2;
//     340 86.9 / 83.4 / 85.8; 50.1 / 48.5 / 55.7; 512 93.1 / 90.8 / 92.5; 55.9 / 56.0 / 67.2
//   {6,5,5} x 4: 1 134 / - / 100; 67 / - / 50; 256 234 / - / 201; 150 / - / 148; 340 263 / 232 / 273; 179 / 161 / 192; 512 310 / 278 / 352; 234 / 221 / 279
//   8 x 8 bits, 1.3 * 10^7 codes, 43 probes, R = 200: 256 699 / - / 627; 511 / - / 478; 340 899 / 816 / 838; 658 / 618 / 631; 512 1112 / 1028 / 1046
//   32 x 4 bits, 5 * 10^6 codes, 26 probes: 256 265 / - / 201; 144 / - / 129; 288 266 / 218 / 248; 148 / 126 / 150; 512 290 / 239 / 307; 194 / 170 / 230
inline int calib_threads(int nq) { return nq <= 256 ? 1024 : (nq <= 512 ? 512 : 256); }

// Pilot codes that a search with long results counts at least, over all blocks of a query: the scan keeps about R / pilot of its
// codes for the selection, so fewer candidates stand against more codes to count.  1024 per result, but beyond 512 no more than a quarter of
// the list.  us a call of one query, gamma data, d = 128, 512 / 1024 per result: R = 1000, 10^7 codes 16 x 4 bits 50.9 / 46.5, 32 x 4
// 65.9 / 60.8, 40-bit 55.9 / 51.9, 8 x 8 69.5 / 64.5, {6,6,4} x 8 98.5 / 98.6; 10^6 codes 30.5 / 31.4, 35.0 / 37.4, 39.5 / 40.8, 47.5 / 49.5,
// 67.7 / 73.5; R = 2000, 10^7 65.9 / 62.8, 89.9 / 88.1, 78.0 / 76.3, 91.4 / 88.6, 144 / 151; 3 * 10^6 49.3 / 51.2, 60.9 / 65.0, 63.4 / 66.3,
// 72.8 / 76.4, 121 / 131; 5 * 10^6 between (a quarter: 53.4, 1024: 54.5; 69.3, 71.7; 68.9, 70.6; 76.8, 81.5; 133, 139).
// With more than four queries the blocks fill the chip and every code counted costs time: 512 (100 queries over 5 * 10^6 codes, R = 2000, 512 / 1024:
// 40-bit 734 / 774, {6,6,4} x 4 1117 / 1212, 8 x 8 1002 / 1098, 16 x 8 1829 / 2022).
inline int64_t pilot_for_results(int64_t n, int R, int nq) {
    const int64_t least = 512 * (int64_t)R, most = 1024 * (int64_t)R;
    return nq > 4 || n / 4 <= least ? least : (n / 4 < most ? n / 4 : most);
}

// When one pass over an inverted list for the (query, probe) pairs of its cell (k_ivf_scan_mx) is taken rather than a block per
// pair.  How long the lists are decides it, which the host does not know (their offsets are on the device): long lists gain from
// a quarter of a pair per cell on, short ones lose the four launches of the exact sort and blocks that wait for few
// codes up to about 6000 pairs.  The lines are a compromise, and PQ_OPT_IVF_SHARED_LISTS = 0 or 2 is for the caller who knows.  us a call,
// block per pair / shared, 16 x 4 bits, R = 100, codes per list first:
//   122, 16384 lists: 1.5 pairs per cell 155 / 166, 2 162 / 168, 4 226 / 204     200, 4096: 1.5 87 / 92, 3 102 / 101, 8 146 / 125
//   500, 512: 4 57 / 66, 16 76 / 78, 32 103 / 93     1000, 1024: 1.5 52 / 58, 4 65 / 64, 8 73 / 74     1200, 4096: 1.5 81 / 79, 4 109 / 95
//   1220, 16384: 0.5 102 / 109, 1.5 146 / 150, 2 171 / 161     2000, 256: 8 61 / 66, 32 91 / 88     2000, 512: 4 65 / 68, 32 126 / 100
//   4900, 4096: 0.25 148 / 115, 1.5 165 / 138     5000, 1024: 1 120 / 93, 2 121 / 96, 8 151 / 144     8000, 256: 1.5 100 / 91, 4 120 / 105
// Below 1024 pairs only lists of 5000 codes and more gain (by up to a tenth), shorter ones lose as much; and with fewer groups than about
// one per CU (a cell's pairs are taken sixteen at a time) even those lose: 5000, 100: 4 65 / 78, 12 81 / 91, 20 83 / 93; 2000, 64: 32 54 / 65.
inline bool ivf_shared_pays(int64_t pairs, int64_t cells) {
    return pairs >= 1024 && 2 * pairs >= 3 * cells && cells + pairs / 16 >= 320;
}

// Blocks of the look-up scan per query at most, where the caller has not set a number (PQ_OPT_SCAN_BLOCKS at its default).  2048 are eight per
// CU, all that fit: one query's scan ends soonest with them, but they leave no room for the next query's kernels, and a block stages its tables,
// adds up its records and counts itself in for few codes.  us a call, 2048 / 1024, one stream and per call on four:
//   2 to 16 queries (300 sizes of eight layouts, 1.2 to 30 million codes, R = 10 to 1000): 1.02 to 1.25 and 0.99 to 1.30 times faster; 16 x 4 bits, 10^7, two
//     queries 52.0 / 46.3 and 28.9 / 22.5; four (on four) 34.2 / 26.8; 12 x {6,6,4}, 5 million, eight 104 / 80 and 74 / 53
//   one query, irregular layouts, 10^7: 40-bit 39.3 / 39.3 and 13.4 / 12.5, {6,6,4} x 4 48.7 / 47.1 and 18.6 / 16.6, {6,5,5} x 4 47.0 / 45.7 and 18.3 / 15.9,
//     {6,6,4} x 8 74.1 / 73.4 and 31.9 / 30.3, 8 x 8 45.8 / 45.2 and 17.7 / 17.0, 16 x 8 73.0 / 73.9 and 34.5 / 32.8; longer lists, whose loops outweigh
//     the rest: 30 million of 40 bits, R = 1000 77.4 / 78.2 and 34.0 / 36.0, {6,6,4} x 4 95.6 / 92.1 and 48.2 / 49.3: up to 2^24 codes
//   one query, nibbles: 16 x 4 bits, 10^7 32.4 / 32.8 and 12.6 / 12.6, R = 300 38.1 / 37.9 and 18.0 / 19.1, 2 * 10^7 46.7 / 46.5 and 22.9 / 25.6; 32 x 4
//     2 * 10^7 R = 100 75.5 / 75.8 and 46.8 / 46.1, R = 1000 96.2 / 95.0 and 53.9 / 54.6: not
#define SCAN_BLOCKS_DEFAULT 2048
inline int scan_blocks_most(int nq, int64_t n, bool nibbles) {
    return nq > 1 || (!nibbles && n <= ((int64_t)1 << 24)) ? SCAN_BLOCKS_DEFAULT / 2 : SCAN_BLOCKS_DEFAULT;
}
