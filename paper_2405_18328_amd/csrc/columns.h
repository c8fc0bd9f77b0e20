// Solver vectors kept column by column: one workgroup of 1024 threads owns a right-hand side, so everything a
// column needs between two products (its dot products, its updates, its largest element and its packed
// operands) happens inside one workgroup, in one launch for all columns.  Shared by the solvers.
//
// Column arrays are [t][ld] fp32, ld = n rounded up to 32, rows from n on zero.  Thread k of the workgroup
// holds rows 4 k .. 4 k + 3 of every 4096, as one 16-byte load per array.
#ifndef GPWS_COLUMNS_H
#define GPWS_COLUMNS_H

#include "gpws_internal.h"
#include "split_f16.h"

namespace {

constexpr int CT = 1024;              // threads per column
constexpr int CROWS = 4 * CT;         // rows they cover at a time

// Block -> column.  Eight columns share every 128-byte line of the packed operands, so neighbouring columns are
// given to the same XCD (workgroup b runs on XCD b % 8), whose L2 then merges their pieces.  Blocks past t
// have no column.
inline int column_blocks(int t) { return (t + 7) / 8 * 8; }
__device__ __forceinline__ int block_column(int t) {
  const int per = (t + 7) / 8;
  const int c = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  return (int)(blockIdx.x >> 3) < per && c < t ? c : -1;
}

// where the packed operands of column c lie: unit (chunk*NT + nt)*2 + part of its pass, lanes c % 16 + 0, 16, 32, 48
struct PackSpot {
  u32x4* base;       // NULL: the vector-ALU column, read as it is
  int NT, nt, lane;
};
__device__ __forceinline__ PackSpot pack_spot(u32x4* VP, int t, int64_t nchunks, int c) {
  PackSpot s;
  const int c0 = vec_columns(t);
  s.base = nullptr;
  s.NT = 1; s.nt = 0; s.lane = 0;
  if (c < c0) return s;
  const int pass = (c - c0) / 64, cc = (c - c0) % 64;   // every pass but the last is 64 columns wide
  s.NT = pass_tiles(t - c0 - 64 * pass);
  s.nt = cc / 16;
  s.lane = cc & 15;
  s.base = VP + (int64_t)pass * nchunks * 8 * 64;
  return s;
}

// Rows 4 k .. 4 k + 3 of a column as operands: scaled, split into fp16 halves, and written in the order of the
// matrix instruction's accumulator layout.  The halves of quads k and k + 4 make up one 16-byte unit each,
// so lanes four apart exchange theirs and every lane writes one whole unit.  The lanes of a group of eight must
// call it together.
__device__ __forceinline__ void pack_quad(const PackSpot& s, int k, f32x4 v) {
  unsigned hi[2], lo[2];
  split_quad(v, hi, lo);
  const bool up = (k & 4) != 0;          // this lane writes the low part
  const unsigned x0 = (unsigned)__shfl_xor((int)(up ? hi[0] : lo[0]), 4);
  const unsigned x1 = (unsigned)__shfl_xor((int)(up ? hi[1] : lo[1]), 4);
  const u32x4 unit = up ? u32x4{x0, x1, lo[0], lo[1]} : u32x4{hi[0], hi[1], x0, x1};
  const int64_t g = (int64_t)(k >> 3) * s.NT + s.nt;   // chunk*NT + nt
  s.base[(g * 2 + (up ? 1 : 0)) * 64 + s.lane + 16 * (k & 3)] = unit;
}
__device__ __forceinline__ float pack_scale(float max_abs) {
  return ldexpf(1.0f, V_TOP - column_exponent(__float_as_uint(max_abs)));
}

// x . y of four rows; handed to an fp64 sum at once, since a longer fp32 chain loses small terms behind large ones
__device__ __forceinline__ double dot4(f32x4 x, f32x4 y) {
  return (double)fmaf(x[3], y[3], fmaf(x[2], y[2], fmaf(x[1], y[1], x[0] * y[0])));
}

// sum / max over the workgroup, in a fixed order, known to every thread afterwards
__device__ __forceinline__ double column_sum(double v, double* sh /* [16] */) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < CT / 64; ++w) s += sh[w];
  return s;
}
__device__ __forceinline__ float column_max(float v, float* sh /* [16] */) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float m = sh[0];
#pragma unroll
  for (int w = 1; w < CT / 64; ++w) m = fmaxf(m, sh[w]);
  return m;
}

// largest |.| of column c of A (mx: this thread's part of it) and the column's operands for the next product
__device__ __forceinline__ void pack_column(u32x4* VP, unsigned* colmax, int t, int64_t ld, int c, const float* A, float mx,
                                            float* shf) {
  const float m = column_max(mx, shf);
  if (threadIdx.x == 0) colmax[c] = __float_as_uint(m);
  const PackSpot spot = pack_spot(VP, t, ld / 32, c);
  if (!spot.base) return;
  const float scale = pack_scale(m);
  const int nk = (int)(ld / 4);
  for (int k0 = 0; k0 < nk; k0 += 4 * CT) {
    f32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const f32x4*>(A + 4 * min(k0 + CT * j + (int)threadIdx.x, nk - 1));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + CT * j + (int)threadIdx.x;
      if (k < nk) pack_quad(spot, k, v[j] * scale);
    }
  }
}

// maxima and operands of all columns of A
__global__ __launch_bounds__(CT) void pack_columns_kernel(const float* __restrict__ A, u32x4* __restrict__ VP,
                                                          unsigned* __restrict__ colmax, int t, int64_t ld) {
  __shared__ float shf[16];
  const int c = block_column(t);
  if (c < 0) return;
  const float* X = A + (int64_t)c * ld;
  float mx = 0.0f;
#pragma unroll 4
  for (int64_t k = threadIdx.x; k < ld / 4; k += CT) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(X + 4 * k);
#pragma unroll
    for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fabsf(x[q]));
  }
  pack_column(VP, colmax, t, ld, c, X, mx, shf);
}

// Sum over the images of a product at rows r .. r + 3 of a column, in order; rows from n on are 0.  Images are fetched
// eight at a time, all loads of a batch in flight together (surplus ones repeat the last image).
template <int BATCH = 8>
__device__ __forceinline__ f32x4 sum_images(const float* __restrict__ images, int JS, int64_t stride, int64_t at,
                                            int64_t r, int64_t n) {
  f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < JS; k += BATCH) {
    f32x4 v[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = *reinterpret_cast<const f32x4*>(images + (int64_t)min(k + u, JS - 1) * stride + at);
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (k + u < JS) s += v[u];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (r + q >= n) s[q] = 0.0f;
  return s;
}

// What a solver's device side tells the host loop, in one 8-byte store to pinned memory (nothing to order, so
// no fence): steps finished in the low half, flags in the high half.
constexpr unsigned COL_DONE = 1u;
struct ColFlags {
  int all_done;
  int bad;
  int iters;
  int pad;
  unsigned long long ticket;   // columns through with the running step, how many of them go on, how many failed
  unsigned long long pad2;
};

// One thread per column, at its end: the column that arrives last raises the flags and posts the step.  The
// ticket counts arrivals (bits 0-15), columns that go on (16-31) and failures of kind 1 (32-47) and 2
// (48-63; reported in preference): one atomic says all, so nothing else has to be visible to the last one.
// The caller has a barrier between it and every read of all_done and of the column's own state by the workgroup's other
// waves: the last arrival raises all_done at once, and a wave that read it late would leave the running step.
__device__ __forceinline__ void column_arrive(ColFlags* f, unsigned long long* post, int t, bool goes_on, int bad, bool counts) {
  const unsigned long long mine = 1ull | ((unsigned long long)goes_on << 16) | (bad == 1 ? 1ull << 32 : bad == 2 ? 1ull << 48 : 0ull);
  const unsigned long long all = atomicAdd(&f->ticket, mine) + mine;
  if ((int)(all & 0xFFFFu) != t) return;
  const int any_bad = (all >> 48) ? 2 : (all >> 32) ? 1 : 0;
  const bool done = any_bad || ((all >> 16) & 0xFFFFu) == 0;
  const int iters = f->iters + (counts ? 1 : 0);
  f->ticket = 0;
  f->iters = iters;
  f->bad = any_bad;
  f->all_done = done ? 1 : 0;
  const unsigned long long word = (unsigned long long)(unsigned)(iters + 1) |
                                  ((unsigned long long)(done ? COL_DONE : 0u) << 32);
  __hip_atomic_store(post, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// row-major n x t (leading dimension lds) -> columns; two matrices per launch (blockIdx.z), a NULL source gives zeros
__global__ __launch_bounds__(256) void to_columns_kernel(const float* __restrict__ S0, int64_t ld0, float* __restrict__ D0,
                                                         const float* __restrict__ S1, int64_t ld1, float* __restrict__ D1,
                                                         int64_t n, int64_t ld, int t) {
  __shared__ float tile[32][129];
  const float* S = blockIdx.z ? S1 : S0;
  float* D = blockIdx.z ? D1 : D0;
  const int64_t lds = blockIdx.z ? ld1 : ld0;
  const int64_t r0 = (int64_t)blockIdx.x * 128;
  const int c0 = blockIdx.y * 32;
  const int c = c0 + (int)(threadIdx.x & 31);
  if (S)
    for (int r = threadIdx.x >> 5; r < 128; r += 8)
      tile[threadIdx.x & 31][r] = (c < t && r0 + r < n) ? S[(r0 + r) * lds + c] : 0.0f;
  __syncthreads();
  const int r = threadIdx.x & 127;
  if (r0 + r < ld)
    for (int k = threadIdx.x >> 7; k < 32; k += 2)
      if (c0 + k < t) D[(int64_t)(c0 + k) * ld + r0 + r] = S ? tile[k][r] : 0.0f;
}

// columns -> row-major n x t; columns with a zero right-hand side give 0
__global__ __launch_bounds__(256) void from_columns_kernel(const float* __restrict__ S, int64_t ld, int64_t n, int t,
                                                           const int* __restrict__ zero_rhs, float* __restrict__ D,
                                                           int64_t ldd) {
  __shared__ float tile[32][129];
  const int64_t r0 = (int64_t)blockIdx.x * 128;
  const int c0 = blockIdx.y * 32;
  const int r = threadIdx.x & 127;
  for (int k = threadIdx.x >> 7; k < 32; k += 2)
    if (c0 + k < t && r0 + r < ld) tile[k][r] = zero_rhs[c0 + k] ? 0.0f : S[(int64_t)(c0 + k) * ld + r0 + r];
  __syncthreads();
  const int c = c0 + (int)(threadIdx.x & 31);
  if (c < t)
    for (int q = threadIdx.x >> 5; q < 128; q += 8)
      if (r0 + q < n) D[(r0 + q) * ldd + c] = tile[threadIdx.x & 31][q];
}

inline dim3 transpose_grid(int64_t ld, int t, int matrices) {
  return dim3((unsigned)((ld + 127) / 128), (unsigned)((t + 31) / 32), (unsigned)matrices);
}

// zeroes 16-byte units (a kernel: workspaces are cleared inside solves that a caller may capture)
__global__ __launch_bounds__(256) void clear_units_kernel(u32x4* __restrict__ p, int64_t units) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < units; e += (int64_t)gridDim.x * 256) p[e] = u32x4{0, 0, 0, 0};
}

// Waits until the posted word reports `want` steps, or that the solve is over.  The stream is looked at now and then
// so that a failed launch or a missing post ends the wait instead of hanging it.
inline int wait_post(gp_ctx* ctx, const char* who, const volatile unsigned long long* post, unsigned want, unsigned long long* seen) {
  for (unsigned spins = 1;; ++spins) {
    const unsigned long long w = *post;
    if ((unsigned)w >= want || (w >> 32) & COL_DONE) {
      *seen = w;
      return GP_OK;
    }
    if ((spins & 4095u) == 0) {
      const hipError_t q = hipStreamQuery(ctx->stream);
      if (q == hipSuccess) {          // nothing left to run: the post must be there by now
        const unsigned long long v = *post;
        if ((unsigned)v >= want || (v >> 32) & COL_DONE) {
          *seen = v;
          return GP_OK;
        }
        return gp_fail(ctx, GP_ERR_HIP, "%s: the solver kernels did not report their state", who);
      }
      if (q != hipErrorNotReady) return gp_fail(ctx, GP_ERR_HIP, "%s: %s", who, hipGetErrorString(q));
    }
  }
}

}  // namespace

#endif
