// Stochastic gradient descent with one workgroup per column, for n <= SGD_COLUMNS_FEW_N (SGD_COLUMNS_MAX_N with one or
// more than 64 columns) on the split-fp16 product paths: the same step, stopping rule and freezing as the streaming kernels of sgd_kernels.hip, in two
// or three launches per step instead of seven.  The product's rows are gathered by the tile kernel itself from the
// context's packed operands; the gradient on the mini-batch rows, momentum, iterate, the stopping test and the packing of
// the iterate for the next product are per column (columns.h).  With few columns the gradient is spread over the chip in a launch of its own
// (with_gradient).
// Measured on MI355X, n = 16384 d = 26 t = 65, batch 1000: a solve with the streaming kernels 78 us per step, with three launches 43, with the
// gradient in the step's launch 38 (a whole marginal-likelihood step 6.60 -> 5.90 ms).  Bound by memory latency and by the
// partial images of the product.
#include "columns.h"

namespace {

struct SgdCols {
  ColFlags* flags;
  unsigned long long* post;
  double* rr;         // [t] squared norm of the residual estimate
  double* bn2;        // [t]
  float* tol;         // [t]
  float* relres;      // [t]
  int* frozen;        // [t]
  int* zero_rhs;      // [t]
  unsigned* colmax;   // [t]
  float *B, *U, *M, *R;   // [t][ld]
  float* G;           // [t][gld] step * gradient per mini-batch slot
  double* deltas;     // [t][slices] change of the squared norm of the residual estimate
  int* bad_index;     // raised by a mini-batch index outside [0, n)
  u32x4* VP;
  const float* images;
  int JS;
  int64_t stride;     // between images
  int64_t n, ld, gld; // gld: rows per column of the product with the mini-batch rows
  int t, batch;
  float sigma2, step, rho;
};

// R holds B, U holds x0 (or 0): M <- 0; warm: R -= H x0; initial state of the column
__global__ __launch_bounds__(CT) void sgdc_start_kernel(SgdCols s, int warm) {
  __shared__ double shd[16];
  const int c = block_column(s.t);
  if (c < 0) return;
  const int64_t col = (int64_t)c * s.ld;
  double bb = 0.0, rr = 0.0;
  for (int64_t k = threadIdx.x; k < s.ld / 4; k += CT) {
    f32x4 r = *reinterpret_cast<const f32x4*>(s.B + col + 4 * k);
    bb += dot4(r, r);
    if (warm) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(s.U + col + 4 * k);
      const f32x4 hx = sum_images(s.images, s.JS, s.stride, col + 4 * k, 4 * k, s.n);
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] -= fmaf(s.sigma2, x[q], hx[q]);
    }
    *reinterpret_cast<f32x4*>(s.R + col + 4 * k) = r;
    *reinterpret_cast<f32x4*>(s.M + col + 4 * k) = f32x4{0.f, 0.f, 0.f, 0.f};
    rr += dot4(r, r);
  }
  const double bn2 = column_sum(bb, shd);
  const double r2 = column_sum(rr, shd);
  if (threadIdx.x == 0) {
    const int zero = bn2 == 0.0;
    const double rel = zero ? 0.0 : sqrt(r2 / bn2);
    const int bad = !zero && (!(rel == rel) || rel > 3.0e38) ? 1 : 0;
    const int fr = zero || (float)rel < s.tol[c];
    s.bn2[c] = bn2;
    s.rr[c] = r2;
    s.relres[c] = (float)rel;
    s.zero_rhs[c] = zero;
    s.frozen[c] = fr;
    if (!warm) s.colmax[c] = 0u;
    column_arrive(s.flags, s.post, s.t, !fr, bad, false);
  }
}

// The mini-batch rows I behind their product: G = (H U)[I] - B[I], R[I] <- -G, step * G kept per slot, and the change of
// the residual estimate's squared norm per slice of slots.  Bound by the latency of the images (64 of them for 1000 rows,
// 16.6 MB at t = 65): a workgroup takes 64 slots, 16 groups of threads share the images between them, 16 bytes a load.  With one
// slot and all images to a thread there were too few workgroups to hide it: 9.8 -> 8.6 us a step at n = 16384, t = 65.  Grid: slices x t.
constexpr int GS = 64;      // slots per workgroup
constexpr int GG = 16;      // groups of images; group g sums images g, g + GG, ..
__global__ __launch_bounds__(GS / 4 * GG) void sgdc_grad_kernel(SgdCols s, const int* __restrict__ I) {
  __shared__ f32x4 part[GG][GS / 4];
  const int c = blockIdx.y, tid = threadIdx.x;
  const int64_t col = (int64_t)c * s.ld, gcol0 = (int64_t)c * s.gld;
  const int slot = blockIdx.x * GS + tid;
  const bool mine = tid < GS && slot < s.batch;
  int64_t i = 0;
  float ui = 0.0f, bi = 0.0f, old = 0.0f;
  bool outside = false;
  if (mine) {
    i = I[slot];
    outside = i < 0 || i >= s.n;
    if (outside) i = 0;
    ui = s.U[col + i];
    bi = s.B[col + i];
    old = s.R[col + i];
  }
  const int stopped = s.frozen[c], over = s.flags->all_done;
  const int quad = tid % (GS / 4), g = tid / (GS / 4);
  const float* at = s.images + gcol0 + min((int)blockIdx.x * GS + 4 * quad, (int)s.gld - 4);
  f32x4 h = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k = g; k < s.JS; k += 4 * GG) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const f32x4*>(at + (int64_t)min(k + GG * u, s.JS - 1) * s.stride);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (k + GG * u < s.JS) h += v[u];
  }
  part[g][quad] = h;
  if (over) return;
  __syncthreads();
  if (tid >= GS) return;      // one wave of slots
  if (outside) *s.bad_index = 1;
  double acc = 0.0;
  if (mine && !stopped) {
    float hx = 0.0f;
#pragma unroll
    for (int k = 0; k < GG; ++k) hx += part[k][tid / 4][tid % 4];
    hx = fmaf(s.sigma2, ui, hx);
    const float gr = hx - bi;
    s.R[col + i] = -gr;
    s.G[gcol0 + slot] = s.step * gr;
    acc = (double)gr * (double)gr - (double)old * (double)old;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (tid == 0) s.deltas[(int64_t)c * gridDim.x + blockIdx.x] = acc;
}

// A step of one column behind its product.  FUSED: the gradient on the mini-batch rows first, as in sgdc_grad_kernel but by the
// workgroup that owns the column, so that it needs neither a launch nor a way through memory: four groups of threads share the
// images, 1024 slots at a time.  Then stopping test, momentum, iterate, the operands of the next product.
// Q > 0: ld <= 4096 Q; momentum and iterate are in registers from the start, the gradient is scattered over the
// column in LDS.  Q = 0: momentum and iterate are streamed, the mini-batch rows corrected afterwards and the iterate
// read again to be packed (the column maximum is then an upper bound, all its scaling needs).
template <int Q, bool FUSED>
__global__ __launch_bounds__(CT) void sgdc_step_kernel(SgdCols s, const int* __restrict__ I, int slices) {
  __shared__ float shf[16];
  __shared__ double shd[16];
  __shared__ f32x4 part[FUSED ? 4 : 1][FUSED ? CT / 4 : 1];
  extern __shared__ float gcol[];     // [ld], Q > 0 only
  const int c = block_column(s.t);
  if (c < 0) return;
  const int tid = threadIdx.x;
  const int64_t col = (int64_t)c * s.ld, gcol0 = (int64_t)c * s.gld;
  const int nk = (int)(s.ld / 4);
  f32x4 u[Q ? Q : 1], m[Q ? Q : 1];
  int64_t i0 = 0;
  float g0 = 0.0f;
  if constexpr (Q > 0) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int k = tid + CT * j;
      u[j] = m[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (k < nk) {
        u[j] = *reinterpret_cast<const f32x4*>(s.U + col + 4 * k);
        m[j] = *reinterpret_cast<const f32x4*>(s.M + col + 4 * k);
      }
    }
    if constexpr (!FUSED) {
      i0 = I[min(tid, s.batch - 1)];
      g0 = s.G[gcol0 + min(tid, s.batch - 1)];
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int k = tid + CT * j;
      if (k < nk) *reinterpret_cast<f32x4*>(gcol + 4 * k) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  bool go = !s.frozen[c];
  const double rr0 = s.rr[c], bn2 = s.bn2[c];
  const float tol = s.tol[c];
  int bad = !FUSED && *s.bad_index ? 2 : 0;
  double delta = 0.0;
  if constexpr (!FUSED)      // every wave adds up all slices
    for (int k = tid & 63; k < slices; k += 64) delta += s.deltas[(int64_t)c * slices + k];
  if (s.flags->all_done) return;
  if constexpr (!FUSED) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) delta += __shfl_xor(delta, off);
  }
  if constexpr (FUSED) {
    if (go) {
      const int quad = tid % (CT / 4), grp = tid / (CT / 4);
      int outside = 0;
      for (int slot0 = 0; slot0 < s.batch; slot0 += CT) {
        const int slot = slot0 + tid;
        bool mine = slot < s.batch;
        int64_t i = 0;
        if (mine) {
          i = I[slot];
          if (i < 0 || i >= s.n) outside = 1, mine = false, i = 0;
        }
        const float ui = s.U[col + i], bi = s.B[col + i], old = s.R[col + i];
        const float* at = s.images + gcol0 + min(slot0 + 4 * quad, (int)s.gld - 4);
        f32x4 h = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int k = grp; k < s.JS; k += 32) {
          f32x4 v[8];
#pragma unroll
          for (int x = 0; x < 8; ++x) v[x] = *reinterpret_cast<const f32x4*>(at + (int64_t)min(k + 4 * x, s.JS - 1) * s.stride);
#pragma unroll
          for (int x = 0; x < 8; ++x)
            if (k + 4 * x < s.JS) h += v[x];
        }
        if (slot0 > 0) __syncthreads();      // the sums of the slots before are read
        part[grp][quad] = h;
        __syncthreads();
        if (mine) {
          float hx = 0.0f;
#pragma unroll
          for (int k = 0; k < 4; ++k) hx += part[k][tid / 4][tid % 4];
          const float gr = fmaf(s.sigma2, ui, hx) - bi;
          s.R[col + i] = -gr;
          if constexpr (Q > 0) gcol[i] = s.step * gr;
          else s.G[gcol0 + slot] = s.step * gr;
          delta += (double)gr * (double)gr - (double)old * (double)old;
        }
      }
      delta = column_sum(delta, shd);      // with barriers behind the scatter and behind every wave's reads above
      bad = __syncthreads_or(outside) ? 2 : 0;
    }
  } else if constexpr (Q > 0) {
    if (go) {
      __syncthreads();
      if (tid < s.batch && i0 >= 0 && i0 < s.n) gcol[i0] = g0;
      for (int slot = tid + CT; slot < s.batch; slot += CT) {
        const int64_t i = I[slot];
        if (i >= 0 && i < s.n) gcol[i] = s.G[gcol0 + slot];
      }
      __syncthreads();
    }
  }
  if (go) {
    // Thread 0 publishes below what every thread reads above (the column's stop, and through the last arrival all_done):
    // not before all waves have read it.  The register forms have a barrier around the scatter into LDS.
    if constexpr (Q == 0 && !FUSED) __syncthreads();
    double rr = rr0 + delta;
    if (rr < 0.0) rr = 0.0;
    const double rel = sqrt(rr / bn2);
    if (!bad && (!(rel == rel) || rel > 3.0e38)) bad = 1;
    if (tid == 0) {
      const int fr = (float)rel < tol ? 1 : 0;
      s.rr[c] = rr;
      s.relres[c] = (float)rel;
      s.frozen[c] = fr;
      column_arrive(s.flags, s.post, s.t, !fr, bad, true);   // nothing below is waited for by the others
    }
    float mx = 0.0f;
    if constexpr (Q > 0) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const int k = tid + CT * j;
        if (k < nk) {
          const f32x4 g = *reinterpret_cast<const f32x4*>(gcol + 4 * k);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float mm = s.rho * m[j][q];
            m[j][q] = mm - g[q];
            u[j][q] = (u[j][q] + mm) - g[q];
            mx = fmaxf(mx, fabsf(u[j][q]));
          }
          *reinterpret_cast<f32x4*>(s.M + col + 4 * k) = m[j];
          *reinterpret_cast<f32x4*>(s.U + col + 4 * k) = u[j];
        }
      }
      const float top = column_max(mx, shf);
      if (tid == 0) s.colmax[c] = __float_as_uint(top);
      const PackSpot spot = pack_spot(s.VP, s.t, s.ld / 32, c);
      if (spot.base) {
        const float scale = pack_scale(top);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          const int k = tid + CT * j;
          if (k < nk) pack_quad(spot, k, u[j] * scale);
        }
      }
    } else {
      for (int k0 = 0; k0 < nk; k0 += 4 * CT) {
        f32x4 uu[4], mm[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = min(k0 + CT * j + tid, nk - 1);
          uu[j] = *reinterpret_cast<const f32x4*>(s.U + col + 4 * k);
          mm[j] = *reinterpret_cast<const f32x4*>(s.M + col + 4 * k);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = k0 + CT * j + tid;
          if (k < nk) {
            mm[j] *= s.rho;
            uu[j] += mm[j];
#pragma unroll
            for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fabsf(uu[j][q]));
            *reinterpret_cast<f32x4*>(s.M + col + 4 * k) = mm[j];
            *reinterpret_cast<f32x4*>(s.U + col + 4 * k) = uu[j];
          }
        }
      }
      __syncthreads();     // the streamed rows are in memory before the mini-batch rows are corrected
      for (int slot = tid; slot < s.batch; slot += CT) {
        int64_t i = I[slot];
        if (i < 0 || i >= s.n) i = 0;
        const float g = s.G[gcol0 + slot];
        s.M[col + i] -= g;
        const float v = s.U[col + i] - g;
        s.U[col + i] = v;
        mx = fmaxf(mx, fabsf(v));
      }
      __syncthreads();
      pack_column(s.VP, s.colmax, s.t, s.ld, c, s.U + col, mx, shf);
    }
  } else if (tid == 0) {
    column_arrive(s.flags, s.post, s.t, false, bad, true);
  }
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Layout {
  int64_t ld, gld, units;
  size_t off_B, off_U, off_M, off_R, off_G, off_deltas, off_state, off_VP, off_images, total;
};

Layout layout(const gp_ctx* ctx, int t, int batch) {
  Layout L;
  L.ld = (ctx->n + 31) / 32 * 32;
  L.gld = ((int64_t)batch + 31) / 32 * 32;
  L.units = gp_packed_units(t, L.ld / 32);
  const size_t arr = align_up((size_t)L.ld * t * sizeof(float), 256);
  const size_t garr = align_up((size_t)L.gld * t * sizeof(float), 256);
  size_t o = 0;
  L.off_B = o; o += arr;
  L.off_U = o; o += arr;
  L.off_M = o; o += arr;
  L.off_R = o; o += arr;
  L.off_G = o; o += garr;
  L.off_deltas = o; o += align_up((size_t)t * ((batch + GS - 1) / GS) * sizeof(double), 256);
  L.off_state = o; o += align_up(sizeof(ColFlags) + 16 + (size_t)t * (2 * sizeof(double) + 2 * sizeof(float) + 3 * sizeof(int)), 256);
  L.off_VP = o; o += align_up((size_t)L.units * 16, 256);
  const size_t square = arr * (size_t)gp_packed_images(ctx, t, ctx->n);
  const size_t rows = garr * (size_t)gp_packed_images(ctx, t, batch);
  L.off_images = o; o += square > rows ? square : rows;
  L.total = o;
  return L;
}

typedef void (*step_fn)(SgdCols, const int*, int);

// Whether the step's workgroups take the gradient along.  One of them reads all images of its column, batch x ranges, on one compute unit;
// a launch of its own spreads them over the chip, which costs 3 to 4 us with few columns and 9 with 65.  Below 49 columns the launch is the
// faster way, and so it is for mini-batches of a few images' lines and of more rows than four rounds of a workgroup.  A step, d = 26,
// launch -> taken along: n = 16384, batch 1000 t = 9 27.7 -> 28.5 us, 17 30.4 -> 31.1, 33 35.3 -> 34.5, 49 39.0 -> 36.7, 65 41.3 -> 37.9,
// 97 57.4 -> 52.9; n = 8192 t = 1 19.7 -> 22.6, 33 27.6 -> 27.6, 65 34.9 -> 31.4; t = 65, n = 8192 batch 100 24.2 -> 24.6, 500 27.7 -> 25.2,
// 2048 41.8 -> 39.2, 4000 53.2 -> 53.9; n = 30000 57.2 -> 55.1 (1000), 80.7 -> 80.7 (2048), 124.3 -> 128.2 (4000).
bool with_gradient(int t, int batch) { return t > 48 && batch >= 200 && batch <= 2048; }

}  // namespace

bool gp_sgd_by_columns(const gp_ctx* ctx, int t) {
  return ctx->n <= (t == 1 || t > 64 ? SGD_COLUMNS_MAX_N : SGD_COLUMNS_FEW_N);
}
size_t gp_sgd_columns_workspace_bytes(const gp_ctx* ctx, int t, int batch) { return layout(ctx, t, batch).total; }

int gp_sgd_columns_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
                       const float* h_tol, const int* dBatches, int batch, int max_iters, double lr, double momentum,
                       void* dWork, int* h_iters, int* h_kmv_count, float* h_relres) {
  const Layout L = layout(ctx, t, batch);
  hipStream_t st = ctx->stream;
  char* w = (char*)dWork;
  SgdCols s;
  s.B = (float*)(w + L.off_B);
  s.U = (float*)(w + L.off_U);
  s.M = (float*)(w + L.off_M);
  s.R = (float*)(w + L.off_R);
  s.G = (float*)(w + L.off_G);
  s.deltas = (double*)(w + L.off_deltas);
  {
    char* q = w + L.off_state;
    s.flags = (ColFlags*)q; q += sizeof(ColFlags);
    s.bad_index = (int*)q; q += 16;
    s.rr = (double*)q; q += sizeof(double) * t;
    s.bn2 = (double*)q; q += sizeof(double) * t;
    s.tol = (float*)q; q += sizeof(float) * t;
    s.relres = (float*)q; q += sizeof(float) * t;
    s.frozen = (int*)q; q += sizeof(int) * t;
    s.zero_rhs = (int*)q; q += sizeof(int) * t;
    s.colmax = (unsigned*)q;
  }
  s.VP = (u32x4*)(w + L.off_VP);
  s.images = (const float*)(w + L.off_images);
  s.n = ctx->n;
  s.ld = L.ld;
  s.gld = L.gld;
  s.t = t;
  s.batch = batch;
  s.sigma2 = (float)(ctx->sigma * ctx->sigma);
  s.step = (float)(lr / (double)batch);
  s.rho = (float)momentum;
  s.JS = 1;
  s.stride = L.ld * (int64_t)t;

  // Pinned staging: tolerances in, flags and residuals out.  Written by the host only here; every solver
  // synchronises the stream before it returns, so the copy a previous call queued from it has run.
  if (sizeof(ColFlags) + sizeof(float) * t * 2 > GP_PIN_THETA)
    return gp_fail(ctx, GP_ERR_ARG, "gp_sgd_solve: t too large for the pinned staging block");
  ColFlags* hflags = (ColFlags*)((char*)ctx->hPinned + GP_PIN_SOLVER);
  float* htol = (float*)(hflags + 1);
  float* hrel = htol + t;
  for (int c = 0; c < t; ++c) htol[c] = h_tol[c];
  volatile unsigned long long* hpost = (volatile unsigned long long*)((char*)ctx->hPinned + GP_PIN_POST);
  s.post = (unsigned long long*)((char*)ctx->dPinned + GP_PIN_POST);
  *hpost = 0;

  // an error return leaves nothing of this solve running: queued kernels would post into the next solve
  auto drained = [&](int rc) -> int {
    (void)hipStreamSynchronize(st);
    return rc;
  };
  auto failed = [&](hipError_t e) -> bool {
    if (e != hipSuccess) (void)drained(gp_fail(ctx, GP_ERR_HIP, "gp_sgd_solve: %s", hipGetErrorString(e)));
    return e != hipSuccess;
  };

  const dim3 grid(column_blocks(t)), block(CT);
  KmvPacked pk;
  pk.VP = s.VP;
  pk.VY = s.U;
  pk.colmax = s.colmax;
  pk.images = (float*)(w + L.off_images);
  pk.ld = L.ld;
  pk.done = nullptr;
  if (failed(hipMemcpyAsync(s.tol, htol, sizeof(float) * t, hipMemcpyHostToDevice, st))) return GP_ERR_HIP;
  hipLaunchKernelGGL(clear_units_kernel, dim3(1), dim3(256), 0, st, (u32x4*)s.flags, (int64_t)(sizeof(ColFlags) / 16 + 1));
  if (!dX0 || padded_tiles(t)) {   // U = 0, or columns that pad the last tile: operands nobody writes before the product reads them
    int blocks = (int)((L.units + 255) / 256);
    if (blocks > 4 * ctx->num_cu) blocks = 4 * ctx->num_cu;
    if (blocks > 0) hipLaunchKernelGGL(clear_units_kernel, dim3(blocks), dim3(256), 0, st, s.VP, L.units);
  }
  hipLaunchKernelGGL(to_columns_kernel, transpose_grid(L.ld, t, 2), dim3(256), 0, st, dB, ldb, s.B, dX0, ldv, s.U, ctx->n, L.ld, t);
  if (failed(hipGetLastError())) return GP_ERR_HIP;
  int kmv_count = 0;
  if (dX0) {
    hipLaunchKernelGGL(pack_columns_kernel, grid, block, 0, st, (const float*)s.U, s.VP, s.colmax, t, L.ld);
    const int rc = gp_kmv_packed(ctx, t, pk, nullptr, 0, nullptr, &s.JS);
    if (rc < 0) return drained(rc);
    ++kmv_count;
  }
  hipLaunchKernelGGL(sgdc_start_kernel, grid, block, 0, st, s, dX0 ? 1 : 0);
  if (failed(hipGetLastError())) return GP_ERR_HIP;

  pk.ld = L.gld;
  pk.done = &s.flags->all_done;
  s.stride = L.gld * (int64_t)t;
  const bool fused = with_gradient(t, batch);
  const int q = L.ld <= CROWS ? 1 : L.ld <= 2 * CROWS ? 2 : L.ld <= 4 * CROWS ? 4 : 0;
  const step_fn step = fused ? (q == 1 ? sgdc_step_kernel<1, true> : q == 2 ? sgdc_step_kernel<2, true> : q == 4 ? sgdc_step_kernel<4, true> : sgdc_step_kernel<0, true>)
                             : (q == 1 ? sgdc_step_kernel<1, false> : q == 2 ? sgdc_step_kernel<2, false> : q == 4 ? sgdc_step_kernel<4, false> : sgdc_step_kernel<0, false>);
  const size_t lds = L.ld <= 4 * CROWS ? (size_t)L.ld * sizeof(float) : 0;
  if (lds > 48 * 1024 && failed(hipFuncSetAttribute((const void*)step, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)))
    return GP_ERR_HIP;
  const int slices = (batch + GS - 1) / GS;
  // Steps queued ahead of the flags the host has seen; kernels queued past the end return at once.
  const int ahead = ctx->prof_mask ? 0 : 4;
  unsigned long long seen = 0;
  bool done = false;
  auto wait_steps = [&](int steps) -> int {
    const int rc = wait_post(ctx, "gp_sgd_solve", hpost, (unsigned)steps + 1, &seen);
    done = ((seen >> 32) & COL_DONE) != 0;
    return rc;
  };
  if (!ahead) {
    const int rc = wait_steps(0);
    if (rc < 0) return drained(rc);
  }
  for (int finished = 0, queued = 0; !done && finished < max_iters; ++finished) {
    for (; queued < max_iters && queued <= finished + ahead; ++queued) {
      const int* I = dBatches + (int64_t)queued * batch;
      const int rc = gp_kmv_packed(ctx, t, pk, I, batch, nullptr, &s.JS);
      if (rc < 0) return drained(rc);
      if (!fused) hipLaunchKernelGGL(sgdc_grad_kernel, dim3(slices, t), dim3(GS / 4 * GG), 0, st, s, I);
      hipLaunchKernelGGL(step, grid, block, lds, st, s, I, slices);
      if (failed(hipGetLastError())) return GP_ERR_HIP;
    }
    const int rc = wait_steps(finished + 1);
    if (rc < 0) return drained(rc);
  }

  hipLaunchKernelGGL(from_columns_kernel, transpose_grid(L.ld, t, 1), dim3(256), 0, st, (const float*)s.U, L.ld, ctx->n, t,
                     (const int*)s.zero_rhs, dV, ldv);
  if (failed(hipGetLastError())) return GP_ERR_HIP;
  if (failed(hipMemcpyAsync(hrel, s.relres, sizeof(float) * t, hipMemcpyDeviceToHost, st))) return GP_ERR_HIP;
  if (failed(hipMemcpyAsync(hflags, s.flags, sizeof(ColFlags), hipMemcpyDeviceToHost, st))) return GP_ERR_HIP;
  if (failed(hipStreamSynchronize(st))) return GP_ERR_HIP;
  if (h_iters) *h_iters = hflags->iters;
  if (h_kmv_count) *h_kmv_count = kmv_count;
  if (h_relres)
    for (int c = 0; c < t; ++c) h_relres[c] = hrel[c];
  if (hflags->bad == 2) return gp_fail(ctx, GP_ERR_ARG, "gp_sgd_solve: a mini-batch index is outside [0, n)");
  if (hflags->bad) return gp_fail(ctx, GP_ERR_BREAKDOWN, "gp_sgd_solve: non-finite residual estimate at step %d (learning rate too large?)", hflags->iters);
  return hflags->all_done ? GP_OK : GP_NOT_CONVERGED;
}
