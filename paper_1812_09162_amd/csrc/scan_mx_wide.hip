// Batched matrix-core scan: the irregular 64- and 128-bit codes.
#include "scan_mx.h"

#define MX_ARGS const pq_index *, const pq_qparams_t *, int, const uint8_t *, int64_t, int, int32_t *, uint16_t *, float *, \
                char *, const ScanPlan &, const MxPlan &, hipStream_t
template int mx_launch<SCAN_W64, uint8_t>(MX_ARGS);
template int mx_launch<SCAN_W64, uint16_t>(MX_ARGS);
template int mx_launch<SCAN_W128, uint8_t>(MX_ARGS);
template int mx_launch<SCAN_W128, uint16_t>(MX_ARGS);
