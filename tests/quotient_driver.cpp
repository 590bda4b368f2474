// Counts, for tables of 16 sub-quantizers of 16 centroids, the waves of 64 entries in which a lane needs the fp64
// division, and the entries at which the fp32 result would differ where it is taken (there must be none).
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include "quotient.h"

static uint64_t seed = 88172645463325252ull;
static float uniform() {
    seed ^= seed << 13; seed ^= seed >> 7; seed ^= seed << 17;
    return (float)(seed >> 40) * 0x1p-24f;
}

int main() {
    long waves = 0, slow[2] = {0, 0}, wrong = 0, whole = 0;
    for (int rep = 0; rep < 4000; ++rep) {
        const float spread = exp2f(40.0f * uniform() - 20.0f);
        float p[256], pm[16];
        for (int j = 0; j < 16; ++j) {
            pm[j] = INFINITY;
            for (int e = 0; e < 16; ++e) {
                float acc = 0.0f;
                for (int t = 0; t < 6; ++t) { const float d = spread * (uniform() - uniform()); acc += d * d; }
                p[16 * j + e] = acc;
                pm[j] = fminf(pm[j], acc);
            }
        }
        double dmin = 0.0, delta;
        for (int j = 0; j < 16; ++j) dmin += pm[j];
        delta = (0.5 + 2.0 * uniform()) * dmin / 255.0;
        if (rep % 4 == 3) {  // quotients at and beside whole numbers
            delta = (double)(float)delta;
            for (int e = 0; e < 256; ++e)
                if (e % 16) p[e] = (float)((double)pm[e / 16] + (double)(e % 16) * 17.0 * delta);
            for (int e = 0; e < 256; e += 5) p[e] = fmaxf(nextafterf(p[e], e % 2 ? INFINITY : 0.0f), pm[e / 16]);
        }
        for (int form = 0; form < 2; ++form) {
            const float slack = form ? QUOTIENT_SLACK_RCP : QUOTIENT_SLACK;
            for (int w = 0; w < 4; ++w) {
                bool all = true;
                for (int e = 64 * w; e < 64 * w + 64; ++e) {
                    const double y = floor(((double)p[e] - (double)pm[e / 16]) / delta);
                    const uint32_t want = y >= 255.0 ? 255u : (uint32_t)y;
                    float inv = form ? 1.0f / (float)delta : (float)(1.0 / delta);
                    if (form) inv = nextafterf(inv, e % 2 ? INFINITY : 0.0f);  // (the hardware's is within one unit)
                    const float x = (p[e] - pm[e / 16]) * inv;
                    const bool sure = quotient_sure(x, slack);
                    all = all && sure;
                    wrong += sure && (uint32_t)fminf(x, 255.0f) != want;
                    whole += x >= 0.5f && x < 255.5f && x == floorf(x) && sure;
                }
                if (rep % 4 != 3) { waves += form == 0; slow[form] += !all; }
            }
        }
    }
    const float nan = NAN;
    const bool edges = quotient_sure(0.0f, QUOTIENT_SLACK) && quotient_sure(INFINITY, QUOTIENT_SLACK) && quotient_sure(1.5f, QUOTIENT_SLACK) &&
                       !quotient_sure(1.0f, QUOTIENT_SLACK) && !quotient_sure(255.0f, QUOTIENT_SLACK) && !quotient_sure(nan, QUOTIENT_SLACK);
    printf("%ld %ld %ld %ld %ld %d\n", waves, slow[0], slow[1], wrong, whole, (int)edges);
    return 0;
}
