// The candidate lists of a BMU search: per sample the kCand best (score, unit)
// pairs, ascending, the lower unit first among equal scores.  Used by the fp32
// products (som_eval.hip) and by those in halves (som_eval_half.hip).
#pragma once

#include "som_internal.h"

namespace som {

__device__ inline bool better(float sa, int ua, float sb, int ub) {
    return sa < sb || (sa == sb && (unsigned)ua < (unsigned)ub);
}

// Insert (s, u) into an ascending top-kCand list (u = -1 marks empty slots,
// whose score is +inf).
__device__ inline void insert_top(float (&ts)[kCand], int (&tu)[kCand], float s, int u) {
    if (!better(s, u, ts[kCand - 1], tu[kCand - 1])) return;
    ts[kCand - 1] = s;
    tu[kCand - 1] = u;
#pragma unroll
    for (int i = kCand - 1; i > 0; --i) {
        if (better(ts[i], tu[i], ts[i - 1], tu[i - 1])) {
            float t = ts[i]; ts[i] = ts[i - 1]; ts[i - 1] = t;
            int v = tu[i]; tu[i] = tu[i - 1]; tu[i - 1] = v;
        }
    }
}

}  // namespace som
