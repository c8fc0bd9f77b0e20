// O(n d) preparation done at gp_create / gp_set_theta: column means of X and
// the packed, pre-scaled operand arrays the tile kernels read (layout in
// gpws_internal.h).  Distances are translation invariant, so centring only
// shrinks |xs|^2 and with it the rounding of the dot-form r^2.
#include <chrono>
#include <cstring>

#include "dist_f16.h"
#include "gpws_internal.h"
#include "split_f16.h"

namespace {

// one workgroup per input dimension; fp64 accumulation
__global__ void column_mean_kernel(const float* __restrict__ X, int64_t n, int d, double* __restrict__ mean) {
  const int k = blockIdx.x;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) s += (double)X[i * d + k];
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) mean[k] = red[0] / (double)n;
}

// one workgroup per input dimension: max_i |x_ik - mean_k| (max is order-independent, so exact and reproducible), and behind those of
// all dimensions the mean of its squares
__global__ void column_spread_kernel(const float* __restrict__ X, int64_t n, int d, const double* __restrict__ mean,
                                     double* __restrict__ out) {
  const int k = blockIdx.x;
  const double mu = mean[k];
  double m = 0.0, s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
    const double v = fabs((double)X[i * d + k] - mu);
    m = (v > m || v != v) ? v : m;      // a NaN input propagates
    s += v * v;
  }
  __shared__ double red[256], sum[256];
  red[threadIdx.x] = m;
  sum[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      const double o = red[threadIdx.x + w];
      if (o > red[threadIdx.x] || o != o) red[threadIdx.x] = o;
      sum[threadIdx.x] += sum[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[k] = red[0];
    out[d + k] = sum[0] / (double)n;
  }
}

// x = hi + mid + lo, each rounded to nearest: with truncated pieces every product would come out a little too small, and with it
// every distance, of one sign
__device__ __forceinline__ void split3(float x, float& hi, float& mid, float& lo) {
  hi = (float)(_Float16)x;
  const float r1 = x - hi;
  mid = (float)(_Float16)r1;
  lo = r1 - mid;
}

// Operands of 32 points: scaled and centred rows, their squared norms, and both packings of the distance contraction.  One
// workgroup per chunk keeps the scaled rows in LDS, so that inputs are read and operands written in whole lines; a thread per row
// (256 to a workgroup) was a chain of strided loads on few compute units, and a second launch read its rows back: n = 16384,
// d = 26 15.2 + 4.5 -> 8.7 us, 1500 rows 11.6 + 3.0 -> 6.9 us.  For the tile pass, whole groups of 32 dimensions go from the rows to
// memory; what the slots behind them hold is listed in LDS first, a piece at a time (all dimensions that way: n = 1000000, d = 90 681 us
// for a gp_set_theta, not 536).
// XA: NULL where only the row side is wanted.  max_norm: the largest squared norm under the tag `seq` in the
// upper half of the word, which makes whatever an earlier tag left there count as less; NULL where nobody asks.
struct PackArgs {
  const float* X;         // [n][d]
  const double* mean;     // [d]
  const double* theta;    // [d] 1 / ell
  float* XA;              // fp32 operands, both sides, or NULL
  float* XB;
  float* Xs;              // [n][d] scaled rows, or NULL
  int XP;                 // operands of the tile pass on so many pieces, both sides (DA: NULL where only the row side is wanted); 0: none
  u32x4* DA;
  u32x4* DB;
  float* CI;              // gamma |xs|^2, or NULL
  u32x4* A[3];            // pieces of the operands of the gradient pass, or NULL
  u32x4* B[3];
  unsigned long long* max_norm;
  unsigned seq;
  int64_t n, chunk0;
  // Work beside the packing, by workgroups from pack_blocks on (0: none): the column maxima of V [nv][t] (colmax), or a copy of its
  // one column with zeros up to vy_rows (VY).
  unsigned pack_blocks;
  const float* V;
  int64_t ldv, nv, vy_rows;
  int t;
  unsigned* colmax;
  float* VY;
  const unsigned short* slots;    // per side (B, A): [group][32] places in a point's list of pieces
  int d, KS, KH, is_se, Q, groups;     // Q: groups of 32 dimensions with a group per piece
  float gamma;
};
__global__ __launch_bounds__(256) void pack_points_kernel(PackArgs p) {
  extern __shared__ float xs[];        // [32][ds] rows, then 32 norms, then their maximum
  if (p.pack_blocks && blockIdx.x >= p.pack_blocks) {
    const int block = (int)(blockIdx.x - p.pack_blocks), blocks = (int)(gridDim.x - p.pack_blocks);
    if (p.colmax) column_maxima(p.V, p.ldv, p.nv, p.t, block, blocks, reinterpret_cast<unsigned*>(xs), p.colmax);
    else
      for (int64_t i = (int64_t)block * 256 + threadIdx.x; i < p.vy_rows; i += (int64_t)blocks * 256) p.VY[i] = i < p.nv ? p.V[i * p.ldv] : 0.0f;
    return;
  }
  const int d = p.d, ds = d | 1;
  float* norm = xs + 32 * ds;
  unsigned* top = reinterpret_cast<unsigned*>(norm + 32);
  _Float16* pieces = reinterpret_cast<_Float16*>(top + 1);    // [32][list]: see gp_dist_slots
  const int XP = p.XP, whole = 32 * p.Q, rest = max(d - whole, 0);      // dimensions in whole groups, and the others
  const int tail = 2 * XP * rest, list = (tail + GP_DIST_LIST_EXTRA) | 1;
  __shared__ u32x4 slots[2 * 4 * DIST_MOST_GROUPS_X3];     // eight places each
  const int tid = threadIdx.x;
  static_assert(8 * DIST_MOST_GROUPS_X3 <= 256, "a thread fetches one of them");
  u32x4 slot{};      // on its way while the rows are read
  if (tid < 8 * p.groups) slot = reinterpret_cast<const u32x4*>(p.slots)[tid];
  // element e = tid + 256 j of the rows is component k of row r; one division, not one for each
  const int rows256 = 256 / d, rest256 = 256 - rows256 * d, r_first = tid / d, k_first = tid - r_first * d;
  auto next = [&](int& r, int& k) {
    r += rows256;
    k += rest256;
    if (k >= d) {
      k -= d;
      ++r;
    }
  };
  const int64_t chunk = p.chunk0 + blockIdx.x, row0 = chunk * 32;
  const int live = (int)(p.n - row0 < 0 ? 0 : p.n - row0 < 32 ? p.n - row0 : 32);
  if (tid == 0) *top = 0u;
  for (int e = tid, r = r_first, k = k_first; e < 32 * d; e += 256, next(r, k)) {
    float v = 0.0f;
    if (r < live) {
      v = (float)(((double)p.X[row0 * d + e] - p.mean[k]) * p.theta[k]);
      if (p.Xs) p.Xs[row0 * d + e] = v;
    }
    xs[r * ds + k] = v;
    if (XP && k >= whole) {
      float hi, mid, lo;
      _Float16* at = pieces + r * list + k - whole;
      split3(v, hi, mid, lo);
      at[0] = (_Float16)hi;
      at[rest] = (_Float16)mid;
      if (XP == 3) at[2 * rest] = (_Float16)lo;
      at += XP * rest;
      split3(-2.0f * p.gamma * v, hi, mid, lo);
      at[0] = (_Float16)hi;
      at[rest] = (_Float16)mid;
      if (XP == 3) at[2 * rest] = (_Float16)lo;
    }
  }
  if (tid < 8 * p.groups) slots[tid] = slot;
  __syncthreads();
  {   // eight neighbouring threads per row
    const int r = tid >> 3;
    double nrm = 0.0;
    for (int k = tid & 7; k < d; k += 8) nrm += (double)xs[r * ds + k] * (double)xs[r * ds + k];
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) nrm += __shfl_xor(nrm, off);
    if ((tid & 7) == 0) {
      const float nf = (float)nrm;
      norm[r] = nf;
      // with the bits that fp32 would round away: on three pieces the norms cancel against each other
      const double g = r < live ? (double)p.gamma * nrm : p.gamma < 0.0f ? -(double)GP_PAD_NORM_H : (double)GP_PAD_NORM_H;   // padding: the kernel value is exactly 0
      if (XP) {
        const float hi = (float)(_Float16)(float)g, mid = (float)(_Float16)(float)(g - hi);
        _Float16* at = pieces + r * list + tail;
        at[0] = (_Float16)hi;
        at[1] = (_Float16)mid;
        at[2] = (_Float16)(float)(g - hi - mid);
        at[3] = (_Float16)1.0f;
        at[4] = (_Float16)(float)PHI_SHIFT;
        at[5] = (_Float16)0.0f;
      }
      if (p.CI) p.CI[row0 + r] = r < live ? (float)g : 0.0f;
      if (p.max_norm && r < live) atomicMax(top, __float_as_uint(nf));     // non-negative floats order like unsigned ints
    }
  }
  __syncthreads();
  if (p.max_norm && tid == 0) atomicMax(p.max_norm, (unsigned long long)p.seq << 32 | *top);
  for (int e = tid; p.XB && e < p.KS * 64; e += 256) {
    const int k = 2 * (e >> 6) + ((e >> 5) & 1), r = e & 31;
    const bool ok = r < live;
    float va = 0.0f, vb = 0.0f;
    if (k < d) { va = xs[r * ds + k]; vb = -2.0f * p.gamma * va; }
    else if (!ok) va = k == d ? GP_PAD_NORM : 0.0f;     // padding rows: r^2 is huge, the kernel value exactly 0
    else if (k == d) { va = norm[r]; vb = p.gamma; }
    else if (k == d + 1) { va = 1.0f; vb = p.gamma * norm[r]; }
    if (p.XA) p.XA[chunk * p.KS * 64 + e] = va;
    p.XB[chunk * p.KS * 64 + e] = vb;
  }
  if (XP) {
    const int G = p.groups;
    for (int v = tid; v < 2 * p.Q * 64; v += 256) {      // whole groups: eight consecutive components to a unit, all pieces at once
      const int lane = v & 63, jt = (v >> 6) >= p.Q, f = (v >> 6) - (jt ? p.Q : 0), c0 = 32 * f + 8 * (lane >> 4);
      const float* x = xs + (16 * jt + (lane & 15)) * ds;
      const int64_t at = chunk * 2 * G * 64 + (jt * G + XP * f) * 64 + lane;
      auto pieces_of = [&](float times, u32x4* to) {
        u32x4 out[3];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          float pc[3][2];
#pragma unroll
          for (int z = 0; z < 2; ++z) {
            const int c = c0 + 2 * e2 + z;
            split3(c < d ? times * x[c] : 0.0f, pc[0][z], pc[1][z], pc[2][z]);
          }
#pragma unroll
          for (int k = 0; k < 3; ++k) out[k][e2] = pack_f16(pc[k][0], pc[k][1]);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
          if (k < XP) to[at + k * 64] = out[k];
      };
      if (p.DA) pieces_of(1.0f, p.DA);
      pieces_of(-2.0f * p.gamma, p.DB);
    }
    const int g0 = XP * p.Q, units = 2 * (G - g0) * 64;
    for (int v = tid; v < (p.DA ? 2 : 1) * units; v += 256) {
      const int side = v >= units, u = side ? v - units : v;
      const int lane = u & 63, jt = (u >> 6) >= G - g0, g = (u >> 6) + (jt ? 2 * g0 - G : g0);
      const u32x4 where = slots[(side * G + g) * 4 + (lane >> 4)];
      const _Float16* from = pieces + (16 * jt + (lane & 15)) * list;
      u32x4 out;
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const unsigned a = __builtin_bit_cast(unsigned short, from[where[e2] & 0xFFFFu]), b = __builtin_bit_cast(unsigned short, from[where[e2] >> 16]);
        out[e2] = a | b << 16;
      }
      (side ? p.DA : p.DB)[chunk * 2 * G * 64 + (jt * G + g) * 64 + lane] = out;
    }
  }
  if (!p.B[0] && !p.B[1] && !p.B[2]) return;
  for (int u = tid; u < p.KH * 64; u += 256) {
    const int r = u & 31, k0 = 16 * (u >> 6) + 8 * ((u >> 5) & 1);
    const bool ok = r < live;
    u32x4 a[3], b[3];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      float pa[3][2], pb[3][2];
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        const int k = k0 + 2 * e2 + z;
        float va = 0.0f, vb = 0.0f;
        if (k < d) { va = xs[r * ds + k]; vb = -2.0f * p.gamma * va; }
        else if (!ok) va = k == d ? GP_PAD_NORM_H : 0.0f;
        else if (k == d) { va = norm[r]; vb = p.gamma; }
        else if (k == d + 1) { va = 1.0f; vb = p.gamma * norm[r]; }
        else if (k == d + 2 && p.is_se) { va = 1.0f; vb = 15.0f; }   // phi is carried as 2^15 phi
        split3(va, pa[0][z], pa[1][z], pa[2][z]);
        split3(vb, pb[0][z], pb[1][z], pb[2][z]);
      }
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) {
        a[pc][e2] = pack_f16(pa[pc][0], pa[pc][1]);
        b[pc][e2] = pack_f16(pb[pc][0], pb[pc][1]);
      }
    }
    const int64_t at = chunk * p.KH * 64 + u;
#pragma unroll
    for (int pc = 0; pc < 3; ++pc)
      if (p.B[pc]) {
        p.A[pc][at] = a[pc];
        p.B[pc][at] = b[pc];
      }
  }
}

// hands the tagged maximum to the host: one 8-byte store to pinned memory
__global__ void post_norm_kernel(const unsigned long long* max_norm, unsigned long long* post) {
  __hip_atomic_store(post, *max_norm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

int gp_launch_column_means(gp_ctx* ctx) {
  hipLaunchKernelGGL(column_mean_kernel, dim3(ctx->d), dim3(256), 0, ctx->stream, ctx->dX, ctx->n, ctx->d,
                     ctx->dMean);
  GP_HIP(ctx, hipGetLastError());
  // per-dimension spread, kept on the host: sum_k (xabs_k / ell_k)^2 bounds every scaled squared norm, which
  // lets gp_set_theta choose the product path without reading anything back in the common case; the mean of the scaled squared norms
  // bounds their maximum from below, which tells it what to pack in most others
  double* dspread = ctx->dRed;
  hipLaunchKernelGGL(column_spread_kernel, dim3(ctx->d), dim3(256), 0, ctx->stream, ctx->dX, ctx->n, ctx->d,
                     (const double*)ctx->dMean, dspread);
  GP_HIP(ctx, hipGetLastError());
  double* h = (double*)ctx->hPinned;
  GP_HIP(ctx, hipMemcpyAsync(h, dspread, sizeof(double) * 2 * ctx->d, hipMemcpyDeviceToHost, ctx->stream));
  GP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (int k = 0; k < ctx->d; ++k) {
    ctx->xabs[k] = h[k];
    ctx->xvar[k] = h[ctx->d + k];
  }
  return GP_OK;
}

namespace {

// beside: workgroups for the work beside it, in the first launch
int launch_pack_points(gp_ctx* ctx, PackArgs& p, int64_t n_pad, int beside = 0) {
  size_t lds = sizeof(float) * (32 * (size_t)(p.d | 1) + 33) + (p.XP ? 32 * sizeof(_Float16) * ((2 * p.XP * (p.d > 32 * p.Q ? p.d - 32 * p.Q : 0) + GP_DIST_LIST_EXTRA) | 1) : 0);
  if (beside && p.colmax && lds < sizeof(unsigned) * p.t) lds = sizeof(unsigned) * p.t;
  // all chunks in one launch would be more than the 2^32 threads it may have from 2^29 points on.  (Workgroups that walk over several
  // chunks instead cost the usual sizes time: n = 500000, d = 3 41 -> 52 us for a gp_set_theta.)
  constexpr int64_t MOST = 1 << 20;
  for (p.chunk0 = 0; p.chunk0 < n_pad / 32; p.chunk0 += MOST) {
    const int64_t left = n_pad / 32 - p.chunk0;
    const unsigned pack = (unsigned)(left < MOST ? left : MOST), more = p.chunk0 == 0 ? (unsigned)beside : 0u;
    p.pack_blocks = more ? pack : 0u;
    hipLaunchKernelGGL(pack_points_kernel, dim3(pack + more), dim3(256), lds, ctx->stream, p);
    GP_HIP(ctx, hipGetLastError());
  }
  return GP_OK;
}

inline int shape_groups(const gp_ctx* ctx, int XP) { return dist_groups(XP, dist_shape_of(XP, ctx->d, ctx->kernel == GP_SE_ARD)); }
inline int path_pieces(int path) { return path == GP_PATH_F16X2 ? 2 : path == GP_PATH_F16X3 ? 3 : 0; }

PackArgs pack_args(const gp_ctx* ctx, int path) {
  PackArgs p{};
  p.mean = ctx->dMean;
  p.theta = ctx->dTheta;
  p.d = ctx->d;
  p.KS = ctx->KS;
  p.KH = ctx->KH;
  p.is_se = ctx->kernel == GP_SE_ARD ? 1 : 0;
  p.XP = path_pieces(path);
  if (p.XP) {
    p.Q = dist_shape(p.XP, dist_shape_of(p.XP, ctx->d, p.is_se)).Q;
    p.groups = shape_groups(ctx, p.XP);
  }
  p.slots = (const unsigned short*)ctx->dDistSlots + (p.XP == 3 ? 2 * 32 * shape_groups(ctx, 2) : 0);
  p.gamma = ctx->kernel == GP_SE_ARD ? (float)(-0.5 * 1.4426950408889634) : 3.0f;
  return p;
}

// a tag of its own for the next maximum
int next_norm_tag(gp_ctx* ctx, PackArgs& p) {
  if (++ctx->norm_seq == 0) {      // the tags start again: so does the word
    GP_HIP(ctx, hipMemsetAsync(ctx->dMaxNorm, 0, sizeof(unsigned long long), ctx->stream));
    ctx->norm_seq = 1;
  }
  p.max_norm = ctx->dMaxNorm;
  p.seq = ctx->norm_seq;
  return GP_OK;
}

int post_norm(gp_ctx* ctx) {
  unsigned long long* post = (unsigned long long*)((char*)ctx->dPinned + GP_PIN_NORM);
  hipLaunchKernelGGL(post_norm_kernel, dim3(1), dim3(1), 0, ctx->stream, (const unsigned long long*)ctx->dMaxNorm, post);
  GP_HIP(ctx, hipGetLastError());
  return GP_OK;
}

}  // namespace

// The post is what is waited for; the stream is asked only every millisecond, whether anything is left on it that could post.  A query
// takes the host about 16 us, and one every 4096 reads of the post was what a short prediction spent its time on: n = 1000, m = 100, d = 9, t = 1
// 37.3 -> 18.8 us a call, and 30.5 -> 34.3 when the launch went that had been in front of the wait.
int gp_wait_norm(gp_ctx* ctx, const char* who, float* norm) {
  const volatile unsigned long long* post = (const volatile unsigned long long*)((char*)ctx->hPinned + GP_PIN_NORM);
  constexpr auto ASK = std::chrono::milliseconds(1);
  auto ask = std::chrono::steady_clock::now() + ASK;
  for (unsigned spins = 1;; ++spins) {
    const unsigned long long w = *post;
    if ((unsigned)(w >> 32) == ctx->norm_seq) {
      const unsigned bits = (unsigned)w;
      memcpy(norm, &bits, sizeof(float));
      return GP_OK;
    }
    if ((spins & 255u) != 0) continue;
    const auto now = std::chrono::steady_clock::now();
    if (now < ask) continue;
    ask = now + ASK;
    // a failed launch or a missing post ends the wait
    const hipError_t q = hipStreamQuery(ctx->stream);
    if (q == hipSuccess) {
      if ((unsigned)(*post >> 32) != ctx->norm_seq) return gp_fail(ctx, GP_ERR_HIP, "%s: the norms were not reported", who);
    } else if (q != hipErrorNotReady) {
      return gp_fail(ctx, GP_ERR_HIP, "%s: %s", who, hipGetErrorString(q));
    }
  }
}

namespace {

// Device memory of what a path reads and gp_create does not allocate: most contexts never ask for it
int allocate_path(gp_ctx* ctx, int path) {
  size_t bytes[4] = {};
  void** where[4] = {};
  void** block = nullptr;
  if (path == GP_PATH_FP32 && !ctx->dXA) {
    block = (void**)&ctx->dXA;
    where[0] = (void**)&ctx->dXA;
    where[1] = (void**)&ctx->dXB;
    bytes[0] = bytes[1] = ((size_t)(ctx->n_pad / GP_CHUNK) * ctx->KS * 64 + GP_PACK_SLACK) * sizeof(float);
  } else if (path == GP_PATH_F16X3 && !ctx->dDA[1]) {
    block = &ctx->dDA[1];
    where[0] = &ctx->dDA[1];
    where[1] = &ctx->dDB[1];
    where[2] = &ctx->dXAh[2];
    where[3] = &ctx->dXBh[2];
    bytes[0] = bytes[1] = gp_dist_bytes(ctx, 3, ctx->n_pad);
    bytes[2] = bytes[3] = gp_grad_piece_bytes(ctx);
  } else {
    return GP_OK;
  }
  size_t total = 0;
  for (size_t& b : bytes) total += b = (b + 255) / 256 * 256;
  const hipError_t e = hipMalloc(block, total);
  if (e != hipSuccess) {
    (void)hipGetLastError();      // else the next launch would be taken for failed
    *block = nullptr;
    return gp_fail(ctx, GP_ERR_HIP, "%zu bytes for the operands of path %d: %s", total, path, hipGetErrorString(e));
  }
  char* at = (char*)*block;
  for (int k = 0; k < 4 && where[k]; at += bytes[k++]) *where[k] = at;
  return GP_OK;
}

// what `path` reads and is not packed for the current theta yet
int pack_path(gp_ctx* ctx, int path, bool want_norm) {
  int rc = allocate_path(ctx, path);
  if (rc < 0) return rc;
  PackArgs p = pack_args(ctx, path);
  p.X = ctx->dX;
  p.n = ctx->n;
  if (!ctx->packed) p.Xs = ctx->dXs;
  if (p.XP) {
    p.DA = (u32x4*)ctx->dDA[p.XP - 2];
    p.DB = (u32x4*)ctx->dDB[p.XP - 2];
    p.CI = ctx->dCI;
    for (int pc = ctx->grad_pieces; pc < p.XP; ++pc) {
      p.A[pc] = (u32x4*)ctx->dXAh[pc];
      p.B[pc] = (u32x4*)ctx->dXBh[pc];
    }
  } else {
    p.XA = ctx->dXA;
    p.XB = ctx->dXB;
  }
  if (want_norm && (rc = next_norm_tag(ctx, p)) < 0) return rc;
  if ((rc = launch_pack_points(ctx, p, ctx->n_pad)) < 0) return rc;
  ctx->packed |= 1u << path;
  if (ctx->grad_pieces < p.XP) ctx->grad_pieces = p.XP;
  return want_norm ? post_norm(ctx) : GP_OK;
}

}  // namespace

// A path's operands are packed when a theta or a prediction asks for that path.  With those on two pieces, fp32's and the gradient's third
// pieces made at every theta, and those on three pieces by a launch of their own, gp_set_theta took (two pieces / three) n = 16384, d = 26
// 23.3 / 49.6 us, now 21.7 / 37.2; n = 1000000, d = 90 1036 / 1721, now 536 / 741.
int gp_launch_pack(gp_ctx* ctx, int path, bool want_norm) {
  ctx->packed = 0;
  ctx->grad_pieces = 0;
  return pack_path(ctx, path, want_norm);
}

int gp_need_path(gp_ctx* ctx, int path) { return ctx->packed >> path & 1u ? GP_OK : pack_path(ctx, path, false); }

namespace {
inline size_t up256(size_t v) { return (v + 255) / 256 * 256; }

struct RowBufs {
  size_t off_xb, off_ci, off_db[2], total;
  int64_t m_pad;
};
RowBufs row_bufs(const gp_ctx* ctx, int64_t m) {
  RowBufs L;
  L.m_pad = (m + GP_ROW_ALIGN - 1) / GP_ROW_ALIGN * GP_ROW_ALIGN;
  size_t o = 0;
  L.off_xb = o; o += up256(((size_t)(L.m_pad / 32) * ctx->KS * 64 + GP_PACK_SLACK) * sizeof(float));
  L.off_ci = o; o += up256((size_t)L.m_pad * sizeof(float));
  for (int x = 0; x < 2; ++x) { L.off_db[x] = o; o += up256(gp_dist_bytes(ctx, x + 2, L.m_pad)); }
  L.total = o;
  return L;
}
}  // namespace

// Where every slot behind the whole groups finds its piece in a point's list, for both layouts and sides: pieces of x's other components
// (hi, mid and on three pieces lo), those of -2 gamma x, those of gamma |x|^2, then 1, 15 and 0.
int gp_dist_slots(const gp_ctx* ctx, unsigned short* slots) {
  const bool shift = ctx->kernel == GP_SE_ARD;
  int n = 0;
  for (int XP = 2; XP <= 3; ++XP) {
    const int id = dist_shape_of(XP, ctx->d, shift), G = dist_groups(XP, id);
    const DistShape s = dist_shape(XP, id);
    for (int side = 0; side < 2; ++side)
      for (int g = 0; g < G; ++g)
        for (int k = 0; k < 32; ++k) {
          const DistSlot t = dist_slot(XP, s.Q, s.R, ctx->d, shift, side != 0, g, k);
          const int rest = ctx->d > 32 * s.Q ? ctx->d - 32 * s.Q : 0, tail = 2 * XP * rest;
          int at = tail + 5;
          if (g < XP * s.Q) at = 0;      // not from the list
          else if (t.what == DIST_X) at = (side ? 0 : XP * rest) + t.piece * rest + t.comp - 32 * s.Q;
          else if (t.what == DIST_NORM) at = tail + t.piece;
          else if (t.what == DIST_ONE) at = tail + 3;
          else if (t.what == DIST_SHIFT) at = tail + 4;
          if (slots) slots[n] = (unsigned short)at;
          ++n;
        }
  }
  return n;
}

size_t gp_dist_bytes(const gp_ctx* ctx, int XP, int64_t rows) {
  return (size_t)(rows / 16) * shape_groups(ctx, XP) * 64 * 16;
}
size_t gp_grad_piece_bytes(const gp_ctx* ctx) { return (size_t)(ctx->n_pad / GP_CHUNK) * ctx->KH * 64 * 16; }

size_t gp_pack_rows_bytes(const gp_ctx* ctx, int64_t m) { return row_bufs(ctx, m).total; }

int gp_pack_rows(gp_ctx* ctx, const float* dXstar, int64_t m, void* buf, KmvRows* rows, const float* dV, int64_t ldv, int t, void* kmv_scratch) {
  const RowBufs L = row_bufs(ctx, m);
  char* w = (char*)buf;
  // farther rows do not bring the path back from where the context's own points have it: with its layout first
  PackArgs p = pack_args(ctx, ctx->path);
  p.X = dXstar;
  p.n = m;
  p.XB = (float*)(w + L.off_xb);
  p.CI = (float*)(w + L.off_ci);
  for (int x = 0; x < 2; ++x) rows->DB[x] = w + L.off_db[x];
  if (p.XP) p.DB = (u32x4*)rows->DB[p.XP - 2];
  int rc, beside = 0;
  // What V needs first has nothing to do with the rows: it goes along with their packing instead of into a launch behind it
  rows->v_prepared = ctx->path != GP_PATH_FP32 && !gp_short_pack(ctx, t);
  if (rows->v_prepared) {
    p.V = dV;
    p.ldv = ldv;
    p.nv = ctx->n;
    p.t = t;
    if (t > 1) {
      if ((rc = gp_clear_maxima(ctx, t)) < 0) return rc;
      p.colmax = ctx->dColmax;
      beside = gp_colmax_blocks(ctx, t);
    } else {
      p.VY = (float*)((char*)kmv_scratch + gp_vec_column_offset(ctx, t));
      p.vy_rows = (ctx->n + 31) / 32 * 32;
      beside = (int)((p.vy_rows + 1023) / 1024 < ctx->num_cu ? (p.vy_rows + 1023) / 1024 : ctx->num_cu);
    }
  }
  if ((rc = next_norm_tag(ctx, p)) < 0) return rc;
  if ((rc = launch_pack_points(ctx, p, L.m_pad, beside)) < 0) return rc;
  if ((rc = post_norm(ctx)) < 0) return rc;
  rows->m = m;
  rows->X = dXstar;
  rows->XB = p.XB;
  rows->CI = p.CI;
  rows->gather = nullptr;
  rows->reads_X = false;
  rows->path = ctx->path == GP_PATH_FP32 ? GP_PATH_FP32 : GP_PATH_PENDING;
  return GP_OK;
}

// Rows that need three pieces where the context's points need two: both sides once more.  The rows are read again, under a tag of their
// own: gp_predict waits for it before the caller may have them back.
int gp_rows_x3(gp_ctx* ctx, KmvRows* rows) {
  int rc = gp_need_path(ctx, GP_PATH_F16X3);
  if (rc < 0 || ctx->XP == 3 || rows->gather) return rc;
  PackArgs p = pack_args(ctx, GP_PATH_F16X3);
  p.X = rows->X;
  p.n = rows->m;
  p.DB = (u32x4*)rows->DB[1];
  if ((rc = next_norm_tag(ctx, p)) < 0) return rc;
  if ((rc = launch_pack_points(ctx, p, (rows->m + GP_ROW_ALIGN - 1) / GP_ROW_ALIGN * GP_ROW_ALIGN)) < 0) return rc;
  rows->reads_X = true;
  return post_norm(ctx);
}

// the product path must cover the scaled norms of both point sets
int gp_rows_path(gp_ctx* ctx, KmvRows* rows) {
  float mx;
  const int rc = gp_wait_norm(ctx, "gp_predict", &mx);
  if (rc < 0) return rc;
  if (ctx->max_norm > mx) mx = ctx->max_norm;
  rows->path = mx <= GP_NORM_X2_MAX ? GP_PATH_F16X2 : (mx <= GP_NORM_X3_MAX ? GP_PATH_F16X3 : GP_PATH_FP32);
  if (ctx->path_forced >= 0 && !(ctx->path_forced != GP_PATH_FP32 && mx > GP_NORM_X3_MAX)) rows->path = ctx->path_forced;
  return GP_OK;
}
