// The gather of a mini-batch from a device-resident training set, as work of
// one thread (of a launch of its own, or of another kernel's spare
// work-groups).
#pragma once

#include "bmlp_internal.h"

namespace bmlp {

// one thread per 64-bit word of the batch; the word-0 thread of a row also
// copies its label
inline long long gather_items(const GatherArgs &a) { return (long long)a.n * a.words; }

__device__ __forceinline__ void gather_item(const GatherArgs &a, uint32_t t) {
  if (t >= (uint32_t)a.n * (uint32_t)a.words) return;   // at most 2^14 rows of 2^9 words
  const uint32_t i = t / (uint32_t)a.words, w = t - i * (uint32_t)a.words;
  const int src = min(max(a.order[i], 0), a.n_all - 1);
  a.xb[t] = a.x_all[(size_t)src * a.words + w];
  if (w == 0) a.yb[i] = a.y_all[src];
}

}  // namespace bmlp
