// The split-fp16 operand format of the contraction side: constants and the scaling of a column, shared by the tile
// kernels and by every kernel that writes operands for them.
#ifndef GPWS_SPLIT_F16_H
#define GPWS_SPLIT_F16_H

#include <hip/hip_runtime.h>

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr int PHI_SHIFT = 15;                   // phi' = 2^15 phi <= 32768 stays inside fp16's range
constexpr int V_TOP = 14;                       // max |V'_c| in [2^13, 2^14)

// Column passes of a product with t columns: up to four tiles of 16 columns each.  A lone column past whole tiles rides
// on the vector ALU of the first pass instead of a tile used for 1/16 of its width, where that saves a tile.
__host__ __device__ inline int pass_tiles(int rem) { return rem > 48 ? 4 : rem > 0 ? (rem + 15) / 16 : 0; }
__host__ __device__ inline int vec_columns(int t) { return t % 16 == 1 ? 1 : 0; }
// whether some tile of the last pass has columns that are not there
__host__ __device__ inline bool padded_tiles(int t) {
  const int rem = (t - vec_columns(t)) % 64;
  return rem != 0 && rem != 16 * pass_tiles(rem);
}

// exponent e with max = f 2^e, f in [0.5, 1); 14 for an all-zero column (scale 1)
__device__ __forceinline__ int column_exponent(unsigned max_bits) {
  const float m = __uint_as_float(max_bits);
  if (!(m > 0.0f)) return V_TOP;
  int e;
  (void)frexpf(m, &e);
  return e < -60 ? -60 : e;
}

// colmax[c] = max_i |V_ic| as a bit pattern (non-negative floats order like unsigned ints), block's share of the rows, for
// workgroups of 256 threads; smax: t words of LDS
__device__ __forceinline__ void column_maxima(const float* __restrict__ V, int64_t ldv, int64_t n, int t, int block, int blocks,
                                              unsigned* smax, unsigned* __restrict__ colmax) {
  // a thread keeps one column (per group of 256 columns) and walks rows: consecutive threads read
  // consecutive columns of a row, the running maximum stays in a register
  for (int c = threadIdx.x; c < t; c += 256) smax[c] = 0u;
  __syncthreads();
  const int64_t rows_per_block = (n + blocks - 1) / blocks;
  const int64_t r0 = (int64_t)block * rows_per_block;
  const int64_t r1 = min(n, r0 + rows_per_block);
  const int tw = t < 256 ? t : 256;        // columns handled side by side
  const int lanes = 256 / tw;              // rows handled side by side
  const int cl = threadIdx.x % tw, rl = threadIdx.x / tw;
  if (rl < lanes) {
    for (int c = cl; c < t; c += tw) {
      float m0 = 0.0f, m1 = 0.0f, m2 = 0.0f, m3 = 0.0f;
      int64_t i = r0 + rl;
      for (; i + 3 * lanes < r1; i += 4 * lanes) {
        m0 = fmaxf(m0, fabsf(V[i * ldv + c]));
        m1 = fmaxf(m1, fabsf(V[(i + lanes) * ldv + c]));
        m2 = fmaxf(m2, fabsf(V[(i + 2 * lanes) * ldv + c]));
        m3 = fmaxf(m3, fabsf(V[(i + 3 * lanes) * ldv + c]));
      }
      for (; i < r1; i += lanes) m0 = fmaxf(m0, fabsf(V[i * ldv + c]));
      m0 = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
      atomicMax(&smax[c], __float_as_uint(m0));
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < t; c += 256)
    if (smax[c]) atomicMax(&colmax[c], smax[c]);
}

// two values as fp16 halves of a word, rounded to nearest
__device__ __forceinline__ unsigned pack_f16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{a, b}), f16x2));
}

// x - (float)half H of pk, one v_fma_mix_f32 (source 0 read as the fp16 half, sources 1 and 2 as fp32)
template <int H>
__device__ __forceinline__ float minus_half(unsigned pk, float x) {
  float r;
  if (H == 0) asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pk), "v"(x));
  else asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pk), "v"(x));
  return r;
}

// Two values split into fp16 pieces, hi + lo, packed in pairs, two instructions per value.  Both pieces are rounded to nearest: with
// truncated ones every product comes out a little too small, by about 2^-22 of its size, and sums that cancel do not
// average that out.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& hi, unsigned& lo) {
  hi = pack_f16(a, b);
  lo = pack_f16(minus_half<0>(hi, a), minus_half<1>(hi, b));
}

// Two values >= 0 split with hi rounded towards zero, so that lo is not negative either; lo is rounded to nearest.  For the
// tile pass of a product, where this saves power, not instructions: with lo of either sign the matrix cores' operands change
// more from one product to the next, and at n = 500000, d = 90, t = 65 a product takes 227 ms instead of 216.
__device__ __forceinline__ void split_pair_positive(float a, float b, unsigned& hi, unsigned& lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(a, b));
  lo = pack_f16(minus_half<0>(hi, a), minus_half<1>(hi, b));
}

// four scaled values as fp16 halves, packed in pairs
__device__ __forceinline__ void split_quad(f32x4 v, unsigned (&hi)[2], unsigned (&lo)[2]) {
#pragma unroll
  for (int k = 0; k < 2; ++k) split_pair(v[2 * k], v[2 * k + 1], hi[k], lo[k]);
}

}  // namespace

#endif
