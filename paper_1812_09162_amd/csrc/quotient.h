#pragma once
// floor((p - p_min) / delta), saturated at 255, from an fp32 value x of the quotient (Section 3.4's quantizer with
// 8-bit tables).  The definition is in fp64, whose divisions run at a fraction of the fp32 rate; where no whole number lies
// within x's error both give the same result.  Plain C++ on the host, so that its share of a wave can be counted
// without a GPU.
#include <math.h>

// Twice the largest relative error of x where the difference, the reciprocal of delta and the product are each rounded
// once (3 * 2^-24), and where the reciprocal is the hardware's, within 2^-23, of a delta rounded to fp32 (5 * 2^-24).
#define QUOTIENT_SLACK 3.6e-7f
#define QUOTIENT_SLACK_RCP 6.0e-7f

// True where floor(x) is the result (x >= 255.5: where 255 is).  Below one half it is 0 whatever the error: every
// sub-quantizer's smallest entry has x == 0, so without that every wave would hold a lane that divides in fp64.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline bool quotient_sure(float x, float slack) {
#if defined(__HIP_DEVICE_COMPILE__)
    const float fract = __builtin_amdgcn_fractf(x);
#else
    const float fract = x - floorf(x);
#endif
    return (x < 0.5f) | (x >= 255.5f) | (fmaf(x, slack, fabsf(fract - 0.5f)) < 0.5f);
}
