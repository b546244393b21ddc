// The deduplication of a miss list whose length only the device knows, inside the library (hps_lookup.hip).
#ifndef HPS_DEDUP_MISSED_H
#define HPS_DEDUP_MISSED_H

#include <hip/hip_runtime.h>

#include "hps_dedup.h"

// hps_dedup of the first min(*n_dev, n_max) keys of a session (1 <= n_max <= its max_n).  The length goes to *n_host and the distinct keys
// also to keys_host (pinned host memory, by its device address), so that the host reads all three after one wait.
// The stream must not be capturing: the call takes turns with the session's two tables, as hps_dedup does outside a capture.
__attribute__((visibility("hidden")))
hps_status_t hps_dedup_missed(hps_dedup_session *s, const int64_t *keys, size_t n_max, const uint32_t *n_dev, int64_t *unique_keys,
                              int64_t *keys_host, uint32_t *inverse, uint32_t *n_host, uint32_t *n_unique, hipStream_t st);

// The length that the call turned out to have, once known: the next call then clears no more slots than were used.
__attribute__((visibility("hidden"))) void hps_dedup_missed_were(hps_dedup_session *s, size_t n);

#endif  // HPS_DEDUP_MISSED_H
