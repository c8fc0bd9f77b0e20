// Storage of the inverse of a diagonal block: 16-row panels of 4-index groups, so that what a wave of a block solve
// reads per 16 contraction indices is one contiguous kilobyte.  The inverse is symmetric.
#ifndef GPWS_AP_INVERSE_H
#define GPWS_AP_INVERSE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

constexpr int AP_TILE = 64;               // blocks are padded to a multiple of this many rows (identity)
constexpr int AP_FACTOR_BATCH = 64;       // blocks factorised side by side

__device__ __forceinline__ int64_t hinv_at(int r, int c, int BP) {
  return ((int64_t)(r >> 4) * (BP >> 2) + (c >> 2)) * 64 + (r & 15) * 4 + (c & 3);
}
__device__ __forceinline__ constexpr int hinv_step() { return 64; }   // floats between c and c + 4 at fixed r

}  // namespace

#endif
