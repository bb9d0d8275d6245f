// cuts_impl.h -- the order statistics behind the exact quantile cuts, found
// on the device (cuts.hip).
#pragma once

#include "common.h"

namespace gbt {

// keys[seg[j] .. seg[j + 1]) are feature j's sketch keys in any order
// (order-preserving keys of finite floats; 0xffffffff = missing).  With N_j
// the keys of feature j that are not missing and B = max_bin, on return
// N[j] = N_j and, for N_j > 0,
//   vals[j * B + k - 1] = the key at rank ceil(k N_j / B) - 1, k = 1..B-1,
//   vals[j * B + B - 1] = the largest key.
// Every result is an exact order statistic.  The workspace is allocated
// from the context (GBT_E_BUDGET / GBT_E_OOM when it does not fit: nothing
// is held then, and the keys are as they were).  Synchronizes the stream.
gbt_status select_cut_keys(gbt_ctx *c, const uint32_t *keys, const std::vector<int64_t> &seg, int32_t max_bin,
                           std::vector<uint32_t> *vals, std::vector<int64_t> *N);

}  // namespace gbt
