// The log-add-exp reduce_by_index on the bucket-partitioned histogram path
// (defined with that path; used by the log-add-exp entry points).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pvjp.h"

namespace pvjp {

// The bytes that pvjp_hist takes at least: FP32 those of pvjp_hist_ws_bytes, FP64
// a few words a bin (beyond one block's LDS), with which it keeps the bin cache.
size_t hist_least_bytes(pvjp_op op, pvjp_dtype dtype, int64_t n, int64_t m);
// Whether the partitioned form serves (dtype, m): FP32 with bins beyond one
// block's LDS and at most 2^22 of them.
bool hist_lae_partition_ok(pvjp_dtype dtype, int64_t m);
size_t hist_lae_partition_bytes(int64_t n, int64_t m);
// hs[b] = log sum of e^x over bin b (-inf for an empty bin or -inf elements
// only); ws: at least hist_lae_partition_bytes(n, m), 256-byte aligned.
void hist_lae_partitioned(const int32_t* inds, const float* x, int64_t n, int32_t m, float* hs, char* ws,
                          hipStream_t st);

}  // namespace pvjp
