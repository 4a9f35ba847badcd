// Index arithmetic of kernels whose lanes also read what they do not use, where every index has to be one that the caller's array
// has.  Plain C++, so that a host program can walk through it.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define DES_INDEX __host__ __device__ inline
#else
#define DES_INDEX inline
#endif

namespace des {

// Aggregation of the shards' partials P_sum[K][B][D] with eight lanes per sample: first of the four columns that lane `sub` of sample
// `b` requests of the first shard.  A lane without columns requests its sample's first ones, which are there and aligned as P_sum is.
DES_INDEX int64_t ahead_column(int64_t b, int D, int sub) { return b * D + (sub < D / 4 ? sub * 4 : 0); }

// Entry `ahead` places after entry `i`, or `last` if that comes before it.  A batch has fewer than 2^31 entries, so that indices are
// often held in 32 signed bits; an index ahead of the last ones need not fit them.
DES_INDEX uint32_t entry_ahead(uint32_t i, uint32_t ahead, uint32_t last) {
  const uint32_t at = i + ahead;
  return at < last ? at : last;
}

}  // namespace des
