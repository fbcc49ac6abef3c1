// Distance buckets of the near-far SSSP rounds, width delta > 0 (host and device).
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>

namespace grb {

// Bucket of a finite distance d >= 0, for the records only (saturates).
__host__ __device__ inline int bucket_of(float d, float delta) {
  const float q = d / delta;
  return q < 2147483648.0f ? (int)q : INT_MAX;
}

// Where the bucket of d ends: a limit above d, so that a round with this limit
// always takes d.  The product can round to d itself (delta 0.17527635, d
// 1.2269344) and stops growing once d / delta passes 2^24; the next float then.
__host__ __device__ inline float bucket_end(float d, float delta) {
  const float e = (floorf(d / delta) + 1.0f) * delta;
  return d < e ? e : __builtin_bit_cast(float, __builtin_bit_cast(unsigned, d) + 1u);
}

}  // namespace grb
