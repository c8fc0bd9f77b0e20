// Batched conjugate gradients for problems whose column fits one workgroup's stride (n <= CG_COLUMNS_MAX_N) on the
// split-fp16 product path: the same recurrence, stopping rule and freezing as the streaming kernels of
// cg_kernels.hip, in two launches per iteration instead of seven.
//
// The streaming kernels spend 5 to 10 us each on vectors that fit the caches, one launch after the other: product,
// dot product, alpha, x and r, beta, p, packing.  All but the product are per column, so here a workgroup
// owns a column (columns.h) and does them in one go; the product leaves its images column by column.
// Iterations are queued ahead of the host's view of the flags: kernels queued past the end return at once.
// Bound by memory latency: 65 workgroups pull 450 KB each at n = 16384 (about 15 us).  One marginal-likelihood step on
// MI355X, before -> after: n = 2048 d = 8 t = 17 (88 iterations) 4.38 -> 1.56 ms; n = 16384 d = 26 t = 65 (7 iterations)
// 1.82 -> 1.65 ms; n = 43945 d = 20 t = 17 (21 iterations; with cgc_sum_kernel) 18.2 -> 17.0 ms.
// CG_COLUMNS_MAX_N is where the two forms meet at the least favourable shape: per iteration, streaming -> columns, n = 65536,
// d = 11 t = 65 2092 -> 2105 us, d = 5 t = 33 1598 -> 1591; ahead by 5 - 40 % at other d and t there, and more below.
#include "columns.h"

namespace {

struct CgCols {
  ColFlags* flags;
  unsigned long long* post;
  double* rho;        // [t]
  double* bn2;        // [t]
  float* tol;         // [t]
  float* relres;      // [t]
  int* frozen;        // [t]
  int* zero_rhs;      // [t]
  unsigned* colmax;   // [t]
  float *X, *R, *P, *HP;   // [t][ld]
  double* dots;       // [t][slices] (long columns only)
  u32x4* VP;
  const float* images;
  int JS;
  int64_t stride;     // between images
  int64_t n, ld;
  int t;
  float sigma2;
};

// R holds B: ||b||^2; warm: R -= H x0; P <- R, its operands; initial state of the column
__global__ __launch_bounds__(CT) void cgc_start_kernel(CgCols s, int warm) {
  __shared__ double shd[16];
  __shared__ float shf[16];
  const int c = block_column(s.t);
  if (c < 0) return;
  const int64_t col = (int64_t)c * s.ld;
  double bb = 0.0, rr = 0.0;
  float mx = 0.0f;
  for (int64_t k = threadIdx.x; k < s.ld / 4; k += CT) {
    f32x4 r = *reinterpret_cast<const f32x4*>(s.R + col + 4 * k);
    bb += dot4(r, r);
    if (warm) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(s.X + col + 4 * k);
      const f32x4 hx = sum_images(s.images, s.JS, s.stride, col + 4 * k, 4 * k, s.n);
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] -= fmaf(s.sigma2, x[q], hx[q]);
      *reinterpret_cast<f32x4*>(s.R + col + 4 * k) = r;
    }
    *reinterpret_cast<f32x4*>(s.P + col + 4 * k) = r;
    rr += dot4(r, r);
#pragma unroll
    for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fabsf(r[q]));
  }
  const double bn2 = column_sum(bb, shd);
  const double rho = column_sum(rr, shd);
  pack_column(s.VP, s.colmax, s.t, s.ld, c, s.P + col, mx, shf);
  if (threadIdx.x == 0) {
    const int zero = !(bn2 > 0.0);
    const double rel = zero ? 0.0 : sqrt(rho / bn2);
    const int fr = zero || rel < (double)s.tol[c];
    s.bn2[c] = bn2;
    s.rho[c] = rho;
    s.relres[c] = (float)rel;
    s.zero_rhs[c] = zero;
    s.frozen[c] = fr;
    column_arrive(s.flags, s.post, s.t, !fr, 0, false);
  }
}

// Columns longer than the registers of a workgroup hold: H p = sum of the images + sigma^2 p into a column of its
// own, and the dot products p.Hp of every slice of CROWS rows.  One workgroup alone would pull all images of a
// column through one compute unit.  Grid: slices x t.
__global__ __launch_bounds__(256) void cgc_sum_kernel(CgCols s) {
  __shared__ double sh[4];
  const int c = blockIdx.y;
  const int64_t col = (int64_t)c * s.ld;
  const int nk = (int)(s.ld / 4);
  double v = 0.0;
  f32x4 p[4], h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = blockIdx.x * CT + threadIdx.x + 256 * j;
    if (k < nk) {
      p[j] = *reinterpret_cast<const f32x4*>(s.P + col + 4 * k);
      h[j] = sum_images<4>(s.images, s.JS, s.stride, col + 4 * k, 4 * k, s.n);
    }
  }
  if (s.flags->all_done || s.frozen[c]) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = blockIdx.x * CT + threadIdx.x + 256 * j;
    if (k < nk) {
#pragma unroll
      for (int q = 0; q < 4; ++q) h[j][q] = fmaf(s.sigma2, p[j][q], h[j][q]);
      v += dot4(p[j], h[j]);
      *reinterpret_cast<f32x4*>(s.HP + col + 4 * k) = h[j];
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) s.dots[(int64_t)c * gridDim.x + blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// One iteration of one column behind its product: alpha, x and r, beta, p, the operands of the next product.
// Q > 0: ld <= 4096 Q, the column's r, p and H p stay in registers between the three passes, and everything
// is requested before the first value is looked at.  Q = 0: behind cgc_sum_kernel, vectors are read again (from L2).
template <int Q>
__global__ __launch_bounds__(CT) void cgc_iter_kernel(CgCols s) {
  __shared__ double shd[16];
  __shared__ float shf[16];
  const int c = block_column(s.t);
  if (c < 0) return;
  const int64_t col = (int64_t)c * s.ld;
  const int nk = (int)(s.ld / 4);
  const int tid = threadIdx.x;
  f32x4 hp[Q ? Q : 1], p[Q ? Q : 1], r[Q ? Q : 1], x[Q ? Q : 1];
  if constexpr (Q > 0) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int k = tid + CT * j;
      p[j] = hp[j] = r[j] = x[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (k < nk) {
        p[j] = *reinterpret_cast<const f32x4*>(s.P + col + 4 * k);
        r[j] = *reinterpret_cast<const f32x4*>(s.R + col + 4 * k);
        x[j] = *reinterpret_cast<const f32x4*>(s.X + col + 4 * k);
        hp[j] = sum_images<Q == 4 ? 4 : 8>(s.images, s.JS, s.stride, col + 4 * k, 4 * k, s.n);
      }
    }
  }
  const double rho = s.rho[c], bn2 = s.bn2[c];
  const double tol = (double)s.tol[c];
  bool go = !s.frozen[c], bad = false;
  if (s.flags->all_done) return;
  if (go) {
    double acc = 0.0;
    double gamma;
    if constexpr (Q > 0) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) hp[j][q] = fmaf(s.sigma2, p[j][q], hp[j][q]);
        acc += dot4(p[j], hp[j]);
      }
      gamma = column_sum(acc, shd);
    } else {
      gamma = 0.0;
      const int slices = (nk + CT - 1) / CT;
      for (int k = 0; k < slices; ++k) gamma += s.dots[(int64_t)c * slices + k];
    }
    float al = 0.0f;
    if (!(gamma > 0.0) || !isfinite(gamma)) bad = true;
    else al = (float)(rho / gamma);
    acc = 0.0;
    if constexpr (Q > 0) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const int k = tid + CT * j;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          x[j][q] = fmaf(al, p[j][q], x[j][q]);
          r[j][q] = fmaf(-al, hp[j][q], r[j][q]);
        }
        acc += dot4(r[j], r[j]);
        if (k < nk) {
          *reinterpret_cast<f32x4*>(s.X + col + 4 * k) = x[j];
          *reinterpret_cast<f32x4*>(s.R + col + 4 * k) = r[j];
        }
      }
    } else {
#pragma unroll 2
      for (int k = tid; k < nk; k += CT) {
        const f32x4 pk = *reinterpret_cast<const f32x4*>(s.P + col + 4 * k);
        const f32x4 h = *reinterpret_cast<const f32x4*>(s.HP + col + 4 * k);
        f32x4 rk = *reinterpret_cast<const f32x4*>(s.R + col + 4 * k);
        f32x4 xk = *reinterpret_cast<const f32x4*>(s.X + col + 4 * k);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          xk[q] = fmaf(al, pk[q], xk[q]);
          rk[q] = fmaf(-al, h[q], rk[q]);
        }
        acc += dot4(rk, rk);
        *reinterpret_cast<f32x4*>(s.X + col + 4 * k) = xk;
        *reinterpret_cast<f32x4*>(s.R + col + 4 * k) = rk;
      }
    }
    const double rho_new = column_sum(acc, shd);
    const double rel = sqrt(rho_new / bn2);
    if (!isfinite(rho_new)) bad = true;
    const float be = (float)(rho_new / rho);
    go = !(rel < tol);
    if (tid == 0) {
      s.rho[c] = rho_new;
      s.relres[c] = (float)rel;
      s.frozen[c] = go ? 0 : 1;
      column_arrive(s.flags, s.post, s.t, go, bad ? 1 : 0, true);   // nothing below is waited for by the others
    }
    if (go) {   // a column that has stopped needs no direction any more
      float mx = 0.0f;
      if constexpr (Q > 0) {
#pragma unroll
        for (int j = 0; j < Q; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            p[j][q] = fmaf(be, p[j][q], r[j][q]);
            mx = fmaxf(mx, fabsf(p[j][q]));
          }
        const float m = column_max(mx, shf);
        if (tid == 0) s.colmax[c] = __float_as_uint(m);
        const PackSpot spot = pack_spot(s.VP, s.t, s.ld / 32, c);
        const float scale = pack_scale(m);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          const int k = tid + CT * j;
          if (k < nk) {
            *reinterpret_cast<f32x4*>(s.P + col + 4 * k) = p[j];
            if (spot.base) pack_quad(spot, k, p[j] * scale);
          }
        }
      } else {
#pragma unroll 4
        for (int k = tid; k < nk; k += CT) {
          f32x4 pk = *reinterpret_cast<const f32x4*>(s.P + col + 4 * k);
          const f32x4 rk = *reinterpret_cast<const f32x4*>(s.R + col + 4 * k);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            pk[q] = fmaf(be, pk[q], rk[q]);
            mx = fmaxf(mx, fabsf(pk[q]));
          }
          *reinterpret_cast<f32x4*>(s.P + col + 4 * k) = pk;
        }
        pack_column(s.VP, s.colmax, s.t, s.ld, c, s.P + col, mx, shf);
      }
    }
  } else if (tid == 0) {
    column_arrive(s.flags, s.post, s.t, false, 0, true);
  }
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Layout {
  int64_t ld, units;
  size_t off_X, off_R, off_P, off_HP, off_dots, off_state, off_VP, off_images, total;
};

Layout layout(const gp_ctx* ctx, int t) {
  Layout L;
  L.ld = (ctx->n + 31) / 32 * 32;
  L.units = gp_packed_units(t, L.ld / 32);
  const size_t arr = align_up((size_t)L.ld * t * sizeof(float), 256);
  size_t o = 0;
  L.off_X = o; o += arr;
  L.off_R = o; o += arr;
  L.off_P = o; o += arr;
  L.off_HP = o; o += arr;
  L.off_dots = o; o += align_up((size_t)t * ((L.ld + CROWS - 1) / CROWS) * sizeof(double), 256);
  L.off_state = o; o += align_up(sizeof(ColFlags) + (size_t)t * (2 * sizeof(double) + 2 * sizeof(float) + 3 * sizeof(int)), 256);
  L.off_VP = o; o += align_up((size_t)L.units * 16, 256);
  L.off_images = o; o += arr * (size_t)gp_packed_images(ctx, t, ctx->n);
  L.total = o;
  return L;
}

}  // namespace

bool gp_cg_by_columns(const gp_ctx* ctx) { return ctx->n <= CG_COLUMNS_MAX_N; }
size_t gp_cg_columns_workspace_bytes(const gp_ctx* ctx, int t) { return layout(ctx, t).total; }

int gp_cg_columns_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
                      const float* h_tol, int max_iters, void* dWork, int* h_iters, int* h_kmv_count, float* h_relres) {
  const Layout L = layout(ctx, t);
  hipStream_t st = ctx->stream;
  char* w = (char*)dWork;
  CgCols s;
  s.X = (float*)(w + L.off_X);
  s.R = (float*)(w + L.off_R);
  s.P = (float*)(w + L.off_P);
  s.HP = (float*)(w + L.off_HP);
  s.dots = (double*)(w + L.off_dots);
  {
    char* q = w + L.off_state;
    s.flags = (ColFlags*)q; q += sizeof(ColFlags);
    s.rho = (double*)q; q += sizeof(double) * t;
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
  s.t = t;
  s.stride = L.ld * (int64_t)t;
  s.sigma2 = (float)(ctx->sigma * ctx->sigma);
  s.JS = 1;

  // Pinned staging: tolerances in, flags and residuals out.  Written by the host only here; every solver
  // synchronises the stream before it returns, so the copy a previous call queued from it has run.
  if (sizeof(ColFlags) + sizeof(float) * t * 2 > GP_PIN_THETA)
    return gp_fail(ctx, GP_ERR_ARG, "gp_cg_solve: t too large for the pinned staging block");
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
    if (e != hipSuccess) (void)drained(gp_fail(ctx, GP_ERR_HIP, "gp_cg_solve: %s", hipGetErrorString(e)));
    return e != hipSuccess;
  };

  const dim3 grid(column_blocks(t)), block(CT);
  KmvPacked pk;
  pk.VP = s.VP;
  pk.colmax = s.colmax;
  pk.images = (float*)(w + L.off_images);
  pk.ld = L.ld;
  if (failed(hipMemcpyAsync(s.tol, htol, sizeof(float) * t, hipMemcpyHostToDevice, st))) return GP_ERR_HIP;
  hipLaunchKernelGGL(clear_units_kernel, dim3(1), dim3(256), 0, st, (u32x4*)s.flags, (int64_t)(sizeof(ColFlags) / 16));
  if (padded_tiles(t)) {   // the columns that pad the last tile are never written
    int blocks = (int)((L.units + 255) / 256);
    if (blocks > 4 * ctx->num_cu) blocks = 4 * ctx->num_cu;
    hipLaunchKernelGGL(clear_units_kernel, dim3(blocks), dim3(256), 0, st, s.VP, L.units);
  }
  hipLaunchKernelGGL(to_columns_kernel, transpose_grid(L.ld, t, 2), dim3(256), 0, st, dB, ldb, s.R, dX0, ldv, s.X, ctx->n, L.ld, t);
  if (failed(hipGetLastError())) return GP_ERR_HIP;
  int kmv_count = 0;
  if (dX0) {
    hipLaunchKernelGGL(pack_columns_kernel, grid, block, 0, st, (const float*)s.X, s.VP, s.colmax, t, L.ld);
    pk.VY = s.X;
    pk.done = nullptr;
    const int rc = gp_kmv_packed(ctx, t, pk, nullptr, 0, nullptr, &s.JS);
    if (rc < 0) return drained(rc);
    ++kmv_count;
  }
  hipLaunchKernelGGL(cgc_start_kernel, grid, block, 0, st, s, dX0 ? 1 : 0);
  if (failed(hipGetLastError())) return GP_ERR_HIP;

  pk.VY = s.P;
  pk.done = &s.flags->all_done;
  const bool long_columns = L.ld > 4 * CROWS;
  auto* iter = L.ld <= CROWS ? cgc_iter_kernel<1> : L.ld <= 2 * CROWS ? cgc_iter_kernel<2> : L.ld <= 4 * CROWS ? cgc_iter_kernel<4>
                                                                                            : cgc_iter_kernel<0>;
  // Iterations queued ahead of the flags the host has seen.  While launches are being timed nothing is queued that
  // might not run.  An iteration of a short column (about 17 us at n = 2048) is over before the host has seen the one before and queued
  // the next: three of them ahead n = 2048, t = 17, 88 iterations 1450 -> 1320 us; at n = 16384 the launches past the end cost 0.5 %.
  const int ahead = ctx->prof_mask ? 0 : L.ld <= CROWS ? 3 : 1;
  unsigned long long seen = 0;
  bool done = false;
  auto wait_steps = [&](int steps) -> int {
    const int rc = wait_post(ctx, "gp_cg_solve", hpost, (unsigned)steps + 1, &seen);
    done = ((seen >> 32) & COL_DONE) != 0;
    return rc;
  };
  if (!ahead) {
    const int rc = wait_steps(0);
    if (rc < 0) return drained(rc);
  }
  for (int finished = 0, queued = 0; !done && finished < max_iters; ++finished) {
    for (; queued < max_iters && queued <= finished + ahead; ++queued) {
      const int rc = gp_kmv_packed(ctx, t, pk, nullptr, 0, nullptr, &s.JS);
      if (rc < 0) return drained(rc);
      if (long_columns) {
        const bool pr = gp_prof_begin(ctx, GP_PROF_CG_DOT);
        hipLaunchKernelGGL(cgc_sum_kernel, dim3((unsigned)((L.ld + CROWS - 1) / CROWS), t), dim3(256), 0, st, s);
        gp_prof_end(ctx, pr);
      }
      const bool pr = gp_prof_begin(ctx, GP_PROF_CG_XR);
      hipLaunchKernelGGL(iter, grid, block, 0, st, s);
      gp_prof_end(ctx, pr);
      if (failed(hipGetLastError())) return GP_ERR_HIP;
    }
    const int rc = wait_steps(finished + 1);
    if (rc < 0) return drained(rc);
  }

  hipLaunchKernelGGL(from_columns_kernel, transpose_grid(L.ld, t, 1), dim3(256), 0, st, (const float*)s.X, L.ld, ctx->n, t,
                     (const int*)s.zero_rhs, dV, ldv);
  if (failed(hipGetLastError())) return GP_ERR_HIP;
  if (failed(hipMemcpyAsync(hrel, s.relres, sizeof(float) * t, hipMemcpyDeviceToHost, st))) return GP_ERR_HIP;
  if (failed(hipMemcpyAsync(hflags, s.flags, sizeof(ColFlags), hipMemcpyDeviceToHost, st))) return GP_ERR_HIP;
  if (failed(hipStreamSynchronize(st))) return GP_ERR_HIP;
  if (h_iters) *h_iters = hflags->iters;
  if (h_kmv_count) *h_kmv_count = kmv_count + hflags->iters;
  if (h_relres)
    for (int c = 0; c < t; ++c) h_relres[c] = hrel[c];
  if (hflags->bad) return gp_fail(ctx, GP_ERR_BREAKDOWN, "gp_cg_solve: p^T H p <= 0 or non-finite value at iteration %d", hflags->iters);
  return hflags->all_done ? GP_OK : GP_NOT_CONVERGED;
}
