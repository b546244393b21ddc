// Row movement that the dedup operator shares with the cache (defined in hps_cache.hip).  Not part of the C ABI, and not exported.
#ifndef HPS_ROWS_H
#define HPS_ROWS_H

#include <hip/hip_runtime.h>

#include <cstdint>

// out[i] = rows[inverse[i]] for i < n, n > 0, rows of dim fp32, on a device of `cus` compute units.
__attribute__((visibility("hidden")))
hipError_t hps_launch_expand_rows(const float *rows, const uint32_t *inverse, uint32_t n, uint32_t dim, float *out,
                                  uint32_t cus, hipStream_t st);

#endif  // HPS_ROWS_H
