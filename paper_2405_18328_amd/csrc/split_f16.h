// The split-fp16 operand format of the contraction side: constants and the scaling of a column, shared by the tile
// kernels and by every kernel that writes operands for them.
#ifndef GPWS_SPLIT_F16_H
#define GPWS_SPLIT_F16_H

#include <hip/hip_runtime.h>

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr unsigned HI_MASK = 0xFFFFE000u;       // keeps sign, exponent and the top 10 mantissa bits
constexpr int PHI_SHIFT = 15;                   // phi' = 2^15 phi <= 32768 stays inside fp16's range
constexpr int V_TOP = 14;                       // max |V'_c| in [2^13, 2^14)

// exponent e with max = f 2^e, f in [0.5, 1); 14 for an all-zero column (scale 1)
__device__ __forceinline__ int column_exponent(unsigned max_bits) {
  const float m = __uint_as_float(max_bits);
  if (!(m > 0.0f)) return V_TOP;
  int e;
  (void)frexpf(m, &e);
  return e < -60 ? -60 : e;
}

// four scaled values as fp16 halves, packed in pairs: hi is truncated to 11 significant bits, lo is what is left
__device__ __forceinline__ void split_quad(f32x4 v, unsigned (&hi)[2], unsigned (&lo)[2]) {
  float h[4], l[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    h[q] = __uint_as_float(__float_as_uint(v[q]) & HI_MASK);
    l[q] = v[q] - h[q];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    hi[k] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(h[2 * k], h[2 * k + 1]));
    lo[k] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(l[2 * k], l[2 * k + 1]));
  }
}

}  // namespace

#endif
