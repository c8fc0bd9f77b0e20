// Products on the split-fp16 tile pass (tile_kernels_f16.h): packing of V, the choice of kernel and of how a product is cut up, launches.
#include <cstdlib>

#include "tile_f16.h"

namespace {

// ---- per-call operand preparation -------------------------------------------------------------
// colmax[c] = max_i |V_ic|; blockIdx.y = 1 does the same for a second matrix of the same shape.
__global__ __launch_bounds__(256) void colmax_kernel(const float* __restrict__ V, int64_t ldv,
                                                     const float* __restrict__ V2, int64_t ldv2, int64_t n, int t,
                                                     unsigned* __restrict__ colmax, unsigned* __restrict__ colmax2) {
  extern __shared__ unsigned smax[];   // [t]
  if (blockIdx.y) column_maxima(V2, ldv2, n, t, blockIdx.x, gridDim.x, smax, colmax2);
  else column_maxima(V, ldv, n, t, blockIdx.x, gridDim.x, smax, colmax);
}

// zeroes t words of one or two arrays (a kernel, not a memset command: memset nodes recorded into a
// captured graph have misbehaved on replay, and gp_kmv_static must be capturable)
__global__ __launch_bounds__(256) void clear_words_kernel(unsigned* __restrict__ a, unsigned* __restrict__ b, int t) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c < t) {
    a[c] = 0u;
    if (b) b[c] = 0u;
  }
}

// V' images of one column pass: unit u = (chunk*NT + nt)*2 + part, lane l: element e is
// V'[32 chunk + 16 (e/4) + 4 (l/16) + e%4][col0 + 16 nt + l%16]; rows >= n and columns past the pass are zero.
__global__ __launch_bounds__(256) void pack_v_kernel(const float* __restrict__ V, int64_t ldv, int64_t n, int nchunks,
                                                     int NT, int col0, int ncols, int vcol,
                                                     const unsigned* __restrict__ colmax, u32x4* __restrict__ VP,
                                                     float* __restrict__ VY, unsigned* __restrict__ copy, int copy_n) {
  if (copy && blockIdx.x == 0)      // the maxima as the tile kernel and later passes read them
    for (int c = threadIdx.x; c < copy_n; c += 256) copy[c] = colmax[c];
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t total = (int64_t)nchunks * NT * 64;
  if (gid < total) {
    const int lane = (int)(gid & 63);
    const int64_t g = gid >> 6;             // chunk*NT + nt
    const int nt = (int)(g % NT);
    const int64_t chunk = g / NT;
    const int cc = 16 * nt + (lane & 15);
    const bool cok = cc < ncols;
    const int col = col0 + (cok ? cc : 0);
    const float scale = ldexpf(1.0f, V_TOP - column_exponent(colmax[col]));
    u32x4 hi, lo;
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      float f[2];
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        const int e = 2 * e2 + z;
        const int64_t j = chunk * 32 + 16 * (e >> 2) + 4 * (lane >> 4) + (e & 3);
        f[z] = (cok && j < n) ? V[j * ldv + col] * scale : 0.0f;
      }
      unsigned fh, fl;
      split_pair(f[0], f[1], fh, fl);
      hi[e2] = fh;
      lo[e2] = fl;
    }
    u32x4* dst = VP + g * 2 * 64;
    dst[lane] = hi;
    dst[64 + lane] = lo;
  }
  // the VALU column, unscaled
  const int64_t npad = (int64_t)nchunks * 32;
  if (gid < npad) VY[gid] = (vcol >= 0 && gid < n) ? V[gid * ldv + vcol] : 0.0f;
}

// Maxima and operands of all columns of a short V (n <= 8192, one column pass) in one launch: eight columns per
// workgroup, a thread keeps up to NQ quads of rows of one column in registers between the two.  Instead of a pass over V
// for the maxima, a second one for the operands, and the gap between them: gp_kmv at n = 2048, d = 8, t = 17 went
// from 20.4 to 15.2 us.  Beyond 8192 rows a workgroup would hold too few loads in flight for the bytes it has to fetch.
template <int NQ>
__global__ __launch_bounds__(1024) void pack_small_kernel(const float* __restrict__ V, int64_t ldv, int n, int nchunks, int NT,
                                                          int c0, int t, unsigned* __restrict__ colmax,
                                                          u32x4* __restrict__ VP, float* __restrict__ VY) {
  __shared__ float top[16][8];
  const int tid = threadIdx.x, ql = tid >> 3;
  const int c = 8 * blockIdx.x + (tid & 7);
  const bool cok = c < t;
  const int nk = 8 * nchunks;
  f32x4 v[NQ];
  float mx = 0.0f;
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 4 * (ql + 128 * j) + q;
      v[j][q] = (cok && i < n) ? V[(int64_t)i * ldv + c] : 0.0f;
    }
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fabsf(v[j][q]));
#pragma unroll
  for (int off = 8; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if ((tid & 63) < 8) top[tid >> 6][tid & 7] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 16; ++w) mx = fmaxf(mx, top[w][tid & 7]);
  if (tid < 8 && cok) colmax[c] = __float_as_uint(mx);
  const int cc = c - c0;
  if (cc >= 16 * NT) return;
  const float scale = cc < 0 ? 1.0f : ldexpf(1.0f, V_TOP - column_exponent(__float_as_uint(mx)));
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int k = ql + 128 * j;
    if (k >= nk) break;                  // whole groups of eight quads
    unsigned hi[2], lo[2];
    split_quad(v[j] * scale, hi, lo);
    const bool up = (k & 4) != 0;        // quads k and k + 4 (32 lanes on) make up one high and one low unit
    const unsigned x0 = (unsigned)__shfl_xor((int)(up ? hi[0] : lo[0]), 32);
    const unsigned x1 = (unsigned)__shfl_xor((int)(up ? hi[1] : lo[1]), 32);
    if (cc < 0) {
      *reinterpret_cast<f32x4*>(VY + 4 * k) = v[j];
    } else {
      const u32x4 unit = up ? u32x4{x0, x1, lo[0], lo[1]} : u32x4{hi[0], hi[1], x0, x1};
      VP[((int64_t)((k >> 3) * NT + (cc >> 4)) * 2 + (up ? 1 : 0)) * 64 + (cc & 15) + 16 * (k & 3)] = unit;
    }
  }
}

// OUT = (add: OUT +) sum of the partial images, in order.  A chain of dependent loads bounded it (one element per thread, one image
// after the other); now four consecutive elements per thread, eight images fetched at a time.  With the clearing launch
// of the column maxima gone, gp_predict n = 13500, m = 1500, t = 65: 79 -> 70 us; n = 41157, m = 4573, t = 1: 85 -> 78 us.
// GR > 1: that many groups of threads share the images of an element, a run of consecutive ones each, for the many images of few
// elements: n = 41157, m = 4573, t = 1 (28 images, 4573 elements) 6.2 -> 4.6 us a launch.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
template <int GR>
__global__ __launch_bounds__(256) void kmv_reduce_f16_kernel(const float* __restrict__ part, int64_t split_stride, int JS, int64_t n,
                                                             int t, int add, float* __restrict__ out, int64_t ldo) {
  constexpr int Q = 256 / GR;        // quads of elements per workgroup
  __shared__ f32x4 sums[GR][Q];
  const int quad = threadIdx.x % Q, g = threadIdx.x / Q;
  const int64_t total = n * t;
  for (int64_t e0 = (int64_t)blockIdx.x * Q * 4; e0 < total; e0 += (int64_t)gridDim.x * Q * 4) {
    const int64_t e = e0 + 4 * quad;
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t at = e + 4 <= total || total < 4 ? e : total - 4;     // the last thread loads its neighbour's too
    auto each = [&](auto f) {       // this thread's elements
      int64_t i = at / t;
      int c = (int)(at - i * t);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (at + q >= e && at + q < total) f(q, out + i * ldo + c);
        if (++c == t) {
          c = 0;
          ++i;
        }
      }
    };
    if (GR == 1 && add && e < total) each([&](int q, const float* o) { s[q] = *o; });
    const int per = (JS + GR - 1) / GR, k0 = g * per, k1 = min(JS, k0 + per);
    if (total >= 4) {
      for (int k = k0; k < k1; k += 8) {
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f4u*>(part + (int64_t)min(k + u, JS - 1) * split_stride + at);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (k + u < k1) s += v[u];
      }
    } else if (e < total) {
      for (int q = 0; q < (int)total; ++q)
        for (int k = k0; k < k1; ++k) s[q] += part[(int64_t)k * split_stride + q];
    }
    if constexpr (GR > 1) {
      sums[g][quad] = s;
      __syncthreads();
      if (g == 0) {
#pragma unroll
        for (int k = 1; k < GR; ++k) s += sums[k][quad];
      }
      __syncthreads();
    }
    if (g == 0 && e < total) each([&](int q, float* o) { *o = s[q]; });
  }
}

// The kernel of one column pass of NT tiles (y: with the extra vector-ALU column).
struct TileKernelH {
  tileh_fn fn;
  int rows;                // of its waves
  int per_cu;              // workgroups that share a compute unit
  bool wide;               // four row tiles per wave
  int most_cg;             // most waves that can share their rows: chunks of a stage
  double chunk_us;         // about what a chunk takes a compute unit for a workgroup whose waves have rows of their own
  double stream_us;        // and what bringing it from L2 takes
  double start_us;         // what its launch takes more than that of a kernel with two row tiles
  int rows_per_wg(int cg) const { return rows * TILE_WAVES / cg; }
};

// form: FORM_PLAIN .. FORM_WINDOW (the shape does not depend on it)
TileKernelH tile_kernel_h(const gp_ctx* ctx, int XP, int NT, bool y, int form, bool most_rows) {
  TileKernelH k;
  const bool se = ctx->kernel == GP_SE_ARD;
  const int ds = dist_shape_of(XP, ctx->d, se), G = dist_groups(XP, ds);
  const bool wide = most_rows && wide_tiles(ds, XP, NT);
  auto* pick = XP == 2 ? (se ? gp_tile_se_x2 : gp_tile_matern32_x2) : se ? gp_tile_se_x3 : gp_tile_matern32_x3;
  k.fn = pick(ds, NT, y, form, wide);
  k.wide = wide;
  k.rows = wide ? 64 : 32;
  k.per_cu = wide ? 1 : tile_waves(ds, XP, NT) / 2;
  k.most_cg = stage_chunks(ds, XP, NT, y, k.per_cu);
  // per 32x32 tile and SIMD, as measured: the vector work of phi and 14 ns per unit of matrix work (32x32 pairs, 16 slots or columns)
  const double tile_us = (se ? 0.145 : 0.23) + 0.014 * (2 * dist_products(XP, ds) + 3 * NT);
  k.chunk_us = tile_us * (wide_tiles(ds, XP, NT) && !wide ? 1.12 : 1.0) * k.rows / 32 * TILE_WAVES / 4;
  k.start_us = wide ? 6.0 : 0.0;
// a workgroup that has its compute unit to itself brings 36 KB in a us, with others beside it 25
  k.stream_us = (2 * G + 2 * NT) / (k.per_cu == 1 ? 36.0 : 25.0);
  return k;
}

// a workgroup for every row block and column range, and up to seven without work: the same number on every XCD
dim3 tile_grid(const TileArgsH& a) { return dim3((unsigned)(((int64_t)a.row_blocks * a.JS + 7) / 8 * 8)); }

struct PlanH {
  int JS, cps;     // column-range splits, chunks per split
  int CG;          // waves of a workgroup that share its rows
  bool wide;       // four row tiles per wave where there is such a kernel
};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct ScratchH {
  size_t off_colmax, off_vy, off_vp, off_part, total;
};

ScratchH scratch_layout(const gp_ctx* ctx, int t, int JS, int64_t rows) {
  ScratchH L;
  const int64_t nchunks = (ctx->n + 31) / 32;
  size_t o = 0;
  L.off_colmax = o; o += align_up((size_t)t * sizeof(unsigned), 256);
  L.off_vy = o; o += align_up((size_t)nchunks * 32 * sizeof(float), 256);
  L.off_vp = o; o += align_up((size_t)nchunks * 4 * 2 * 64 * 16, 256);      // NT = 4 images
  L.off_part = o;
  if (JS > 1) o += align_up((size_t)JS * rows * t * sizeof(float), 256);
  L.total = o;
  return L;
}

// How a product is cut up: the column ranges of a launch, and the waves of a workgroup that share its rows.  Both fill the chip
// where row blocks are few; a range costs an image of the output, written and read once, and sharing rows costs each chunk's
// way from L2 to more workgroups.  Every row is cut alike, so all rows share one summation tree.
PlanH plan_h(const gp_ctx* ctx, int64_t rows, int64_t col_chunks, int t, int XP) {
  PlanH pl;
  const int64_t chunks = col_chunks > 0 ? col_chunks : (ctx->n + 31) / 32;
  for (const SplitMemo& m : ctx->split_memo)
    if (m.JS && m.rows == rows && m.chunks == chunks && m.t == t && m.XP == XP) {
      pl.JS = m.JS;
      pl.CG = m.CG;
      pl.wide = m.wide;
      pl.cps = (int)((chunks + pl.JS - 1) / pl.JS);
      return pl;
    }
  const int y = vec_columns(t);
  // a partial image is written and read once, at about 4 TB/s
  const double image = (double)rows * t * sizeof(float);
  // images of more than 2 GB in all would not pay for their memory
  int max_js = image * 64.0 > 2.0e9 ? (int)(2.0e9 / image) : 64;
  if (max_js < 1) max_js = 1;
  // Up to 128 columns are never cut: there is nothing to gain, and such a product gives a row the same bits whatever rows are beside it.
  constexpr int MIN_CHUNKS = 4;
  double best = 1e300;
  // Of the two kernels for 64 columns the one with two row tiles has half the code and half the rows to fetch, set up and write, the one
  // with four reads half the operands per pair.  One product, four row tiles -> two: n = 1000, t = 65 (Matern), d = 26 22.1 -> 16.2 us,
  // d = 50 28.0 -> 16.7; n = 4000 32.2 -> 28.6, 44.8 -> 30.0; n = 9000 72 -> 69, 87 -> 74; n = 14000 128 -> 137, 151 -> 148; n = 30000
  // 475 -> 504, 542 -> 564.
  const int first = pass_tiles(t - y);
  int tiles = first;
  for (int c = y + 16 * first; c < t; c += 16 * pass_tiles(t - c)) tiles += pass_tiles(t - c);
  const double image_us = 2.0 * image / 4.0e6 * (first ? (double)first / tiles : 1.0);     // against the time of the first pass
  for (int w = 0; w < 2; ++w) {
    const TileKernelH k = tile_kernel_h(ctx, XP, first, y, FORM_PLAIN, w == 1);
    if (w == 1 && (!k.wide || chunks <= MIN_CHUNKS)) continue;
    for (int cg = 1; cg <= (chunks > MIN_CHUNKS ? k.most_cg : 1); cg *= 2) {
      const int64_t row_blocks = (rows + k.rows_per_wg(cg) - 1) / k.rows_per_wg(cg);
      double cost;
      const int js = gp_column_splits(row_blocks, chunks, ctx->num_cu, k.per_cu, cg, k.chunk_us, k.stream_us, image_us, chunks > MIN_CHUNKS ? max_js : 1, &cost);
      cost += k.start_us;
      if (cost < best * (1.0 - 1e-9)) {
        best = cost;
        pl.JS = js;
        pl.CG = cg;
        pl.wide = w == 1;
      }
    }
  }
  pl.cps = (int)((chunks + pl.JS - 1) / pl.JS);
  gp_ctx* memo = const_cast<gp_ctx*>(ctx);   // a context belongs to one host thread at a time
  memo->split_memo[memo->split_next] = SplitMemo{rows, chunks, t, XP, pl.JS, pl.CG, pl.wide};
  memo->split_next = (memo->split_next + 1) % 4;
  return pl;
}

// Where the scratch does not hold the partial images of all rows (gp_kmv_static), they are made and summed for one panel of
// rows and one group of column ranges after the other, a group's operands packed for it: every row keeps its column
// ranges and the order of its sums, so the result is the same bit for bit.
struct PanelsH {
  int64_t rows;    // per panel, a multiple of PANEL_ROWS; 0: no panels
  int group;       // column ranges at a time
};
constexpr int PANEL_ROWS = 512;     // a multiple of every kernel's rows per workgroup

size_t panel_images_at(const ScratchH& L, int group, const PlanH& pl) {
  return L.off_vp + align_up((size_t)group * pl.cps * 4 * 2 * 64 * 16, 256);
}

// Smaller groups leave room for larger panels.  A launch takes about one unit of time per generation of workgroups, 0.55 where
// there is at most one per compute unit.  gp_kmv_static, Matern-3/2, t = 65, every row's column range in one image -> panels
// (gp_kmv, all images at once): n = 70001 d = 26 4.29 -> 2.86 ms (2.76), n = 150000 d = 5 14.0 -> 11.8 ms (10.6),
// n = 200000 d = 5 24.2 -> 20.7 ms (19.6), n = 240000 d = 5 28.4 -> 29.8 ms (26.8).
PanelsH plan_panels(const gp_ctx* ctx, int64_t nrows, int t, int XP, const PlanH& pl, const ScratchH& L, size_t scratch_bytes) {
  const int y = vec_columns(t);
  const TileKernelH k = tile_kernel_h(ctx, XP, pass_tiles(t - y), y, FORM_PLAIN, pl.wide);
  const int64_t unit = PANEL_ROWS / k.rows_per_wg(pl.CG), slots = (int64_t)k.per_cu * ctx->num_cu;
  const int64_t units = (nrows + PANEL_ROWS - 1) / PANEL_ROWS;
  const size_t per_unit = (size_t)(t < 65 ? t : 65) * sizeof(float) * PANEL_ROWS;     // images of the columns of one pass
  PanelsH best{0, pl.JS};
  double best_cost = 1e300;
  for (int group = pl.JS; group >= 1; --group) {
    const size_t at = panel_images_at(L, group, pl);
    if (at >= scratch_bytes) continue;
    const int64_t fit = min((int64_t)((scratch_bytes - at) / (per_unit * group)), units);
    const int64_t wgs = fit * unit * group;
    const int64_t full = wgs >= slots ? wgs / slots * slots : wgs > ctx->num_cu ? ctx->num_cu : wgs;    // whole generations
    for (int64_t p : {fit, full / (unit * group)}) {
      if (p < 1) continue;
      const int64_t w = p * unit * group;
      const double gens = w <= ctx->num_cu ? 0.55 : (double)((w + slots - 1) / slots);
      const double cost = gens * (double)((units + p - 1) / p) * ((pl.JS + group - 1) / group);
      if (cost < best_cost * (1.0 - 1e-9)) {
        best_cost = cost;
        best = PanelsH{p * PANEL_ROWS, group};
      }
    }
  }
  return best;
}

}  // namespace

int gp_kh_bucket(int d, int kernel) {
  // components: d coordinates, squared norm, one, and for SE the slot that carries the 2^15 shift
  const int comps = d + 2 + (kernel == GP_SE_ARD ? 1 : 0);
  const int need = (comps + 15) / 16;
  const int buckets[] = {1, 2, 3, 4, 6, 8};
  for (int b : buckets)
    if (need <= b) return b;
  return -1;
}

// Compute units take workgroups in turn; the busiest one ends the launch, and a last turn of a few workgroups costs as much as a full
// one.  A workgroup's time is its chunks and what its prologue and flush cost; waves that share rows pass fewer chunks between two
// barriers, which costs them 6 % for every doubling (n = 65536, d = 26, t = 65: 2157, 2238, 2374 us a product with 1, 2, 4 of them).
// Every further cut adds one partial image of the output to write and read (image_us).
// Against every plan of 336 products (n = 1000 .. 14000, d = 3 .. 90, t = 1 .. 97; up to 60 plans each) the one priced lowest is 1.4 % behind the fastest in the
// mean, 2 % behind it when an unshared compute unit was priced at 25 KB a us too and a doubling at 4 %, which kept short products from sharing rows:
// n = 1800, d = 26, t = 65 20.1 -> 18.4 us.
int gp_column_splits(int64_t row_blocks, int64_t chunks, int num_cu, int per_cu, int cg, double chunk_us, double stream_us, double image_us,
                     int max_splits, double* cost) {
  constexpr double FIXED = 6.0;       // prologue and flush of a workgroup, in us
  const double shared = chunk_us / cg * (cg == 1 ? 1.0 : cg == 2 ? 1.06 : cg == 4 ? 1.12 : 1.18);
  const double per_chunk = shared > stream_us ? shared : stream_us;
  auto price = [&](int64_t cps, int64_t parts) {
    const int64_t turns = (row_blocks * parts + num_cu - 1) / num_cu;
    // fewer workgroups to a compute unit than it holds leave its SIMDs short of waves
    const double alone = turns >= per_cu ? 1.0 : turns == 1 ? 1.3 : 1.1;
    // the waves that share rows take a stage's chunks in turn
    return (double)turns * ((double)((cps + cg - 1) / cg * cg) * per_chunk * alone + FIXED / per_cu) + (parts > 1 ? image_us * (double)parts : 0.0);
  };
  *cost = price(chunks, 1);
  int best = 1;
  for (int js = 2; js <= max_splits; ++js) {
    const int64_t cps = (chunks + js - 1) / js;
    if (cps < 2 * cg) break;      // two chunks to a wave at least
    const int64_t parts = (chunks + cps - 1) / cps;
    const double c = price(cps, parts);
    if (c < *cost * (1.0 - 1e-9)) {
      *cost = c;
      best = (int)parts;
    }
  }
  return best;
}

// few workgroups: every one ends with t atomic maxima on the same t words
int gp_colmax_blocks(const gp_ctx* ctx, int t) {
  int blocks = (int)((ctx->n * (int64_t)t + 8191) / 8192);
  if (blocks > 2 * ctx->num_cu) blocks = 2 * ctx->num_cu;
  return blocks < 1 ? 1 : blocks;
}

// makes the context's words for column maxima in accumulation clear, for t columns
int gp_clear_maxima(gp_ctx* ctx, int t) {
  if (ctx->colmax_dirty) {
    hipLaunchKernelGGL(clear_words_kernel, dim3((ctx->colmax_dirty + 255) / 256), dim3(256), 0, ctx->stream, ctx->dColmax, nullptr, ctx->colmax_dirty);
    GP_HIP(ctx, hipGetLastError());
  }
  if (ctx->colmax_dirty < t) ctx->colmax_dirty = t;     // until the launch that clears them is on the stream
  return GP_OK;
}

// operands of a short V are packed, maxima and all, in one launch
bool gp_short_pack(const gp_ctx* ctx, int t) { return t > 1 && ctx->n <= 8192 && t - vec_columns(t) <= 64; }
size_t gp_vec_column_offset(const gp_ctx* ctx, int t) { return scratch_layout(ctx, t, 1, 1).off_vy; }

int gp_launch_colmax(gp_ctx* ctx, const float* dV, int64_t ldv, int t, unsigned* cm, const float* dV2, int64_t ldv2,
                     unsigned* cm2, bool cleared) {
  if (!cleared) {
    hipLaunchKernelGGL(clear_words_kernel, dim3((t + 255) / 256), dim3(256), 0, ctx->stream, cm, dV2 ? cm2 : nullptr, t);
    GP_HIP(ctx, hipGetLastError());
  }
  const int blocks = gp_colmax_blocks(ctx, t);
  hipLaunchKernelGGL(colmax_kernel, dim3(blocks, dV2 ? 2 : 1), dim3(256), (size_t)t * sizeof(unsigned), ctx->stream, dV,
                     ldv, dV2, ldv2, ctx->n, t, cm, cm2);
  GP_HIP(ctx, hipGetLastError());
  return GP_OK;
}

size_t gp_kmv_f16_scratch_bytes(const gp_ctx* ctx, int t, int64_t rows, int64_t col_chunks) {
  size_t need = 0;
  for (int XP = 2; XP <= 3; ++XP) {
    const size_t b = scratch_layout(ctx, t, plan_h(ctx, rows, col_chunks, t, XP).JS, rows).total;
    if (b > need) need = b;
  }
  return need;
}

size_t gp_kmv_f16_least_scratch_bytes(const gp_ctx* ctx, int t) { return scratch_layout(ctx, t, 1, ctx->n).total; }

int gp_kmv_launch_f16(gp_ctx* ctx, const float* dV, int64_t ldv, int t, float* dOut, int64_t ldo, int add_noise,
                      void* scratch, size_t scratch_bytes, const unsigned* colmax_ready, KmvRows* rows,
                      KmvDeferred* defer, const KmvWindow* win) {
  const int64_t nrows = rows ? rows->m : ctx->n;
  ScratchH L = scratch_layout(ctx, t, 1, nrows);     // where the operands lie does not depend on the splits
  if (scratch_bytes < L.total || !scratch)
    return gp_fail(ctx, GP_ERR_WORKSPACE, "gp_kmv: scratch %zu < %zu bytes", scratch_bytes, L.total);
  hipStream_t st = ctx->stream;
  char* w = (char*)scratch;
  const unsigned* colmax = colmax_ready ? colmax_ready : (const unsigned*)(w + L.off_colmax);
  float* VY = (float*)(w + L.off_vy);
  u32x4* VP = (u32x4*)(w + L.off_vp);
  // a column window is handed to the kernels as a point set of its own that starts at chunk 0
  const int nchunks = win ? win->nchunks : (int)((ctx->n + 31) / 32);
  const int64_t first = win ? (int64_t)win->chunk0 * 32 : 0;
  const int64_t ncontr = win ? ((first + (int64_t)nchunks * 32 < ctx->n ? first + (int64_t)nchunks * 32 : ctx->n) - first) : ctx->n;
  if (win && !colmax_ready) return gp_fail(ctx, GP_ERR_ARG, "gp_kmv: a column window needs the column maxima");
  const float* dVw = dV + first * ldv;

  // column maxima: the caller's; or taken while the operands are packed (short V, one pass); or accumulated in words of the
  // context that are zero between calls, copied by the first packing and zeroed again by the first tile pass; on the static
  // scratch in words of that scratch, cleared by a launch of their own: a captured gp_kmv_static may run beside other calls
  const bool y = vec_columns(t) != 0;
  const bool small = !colmax_ready && !win && gp_short_pack(ctx, t);
  const bool maxima = !colmax_ready && t > 1 && !small;       // a single vector is not scaled
  const bool accumulate = maxima && scratch != ctx->static_scratch;
  if (maxima) {
    int rc = accumulate && !(rows && rows->v_prepared) ? gp_clear_maxima(ctx, t) : GP_OK;
    if (rc >= 0 && !(rows && rows->v_prepared))
      rc = gp_launch_colmax(ctx, dV, ldv, t, accumulate ? ctx->dColmax : (unsigned*)(w + L.off_colmax), nullptr, 0, nullptr, accumulate);
    if (rc < 0) return rc;
  }

  // operands of one column pass, chunks c0 .. c0 + chunks - 1
  auto pack = [&](int c0, int chunks, int NT, int col0, int ncols, int vc, bool first_pass) {
    const int64_t threads = (int64_t)chunks * NT * 64;
    const int64_t need = threads > (int64_t)chunks * 32 ? threads : (int64_t)chunks * 32;
    const int64_t r0 = (int64_t)c0 * 32;
    hipLaunchKernelGGL(pack_v_kernel, dim3((unsigned)((need + 255) / 256)), dim3(256), 0, st, dVw + r0 * ldv, ldv, ncontr - r0, chunks, NT,
                       col0, ncols, vc, accumulate && first_pass ? (const unsigned*)ctx->dColmax : colmax, VP, VY + r0,
                       accumulate && first_pass ? (unsigned*)(w + L.off_colmax) : nullptr, t);
  };
  auto pack_pass = [&](int NT, int col0, int ncols, int vc, bool first_pass) -> int {      // all of them
    if (small) {
      const int quads = (8 * nchunks + 127) / 128;
      auto* pack_small = quads <= 2 ? pack_small_kernel<2> : quads <= 4 ? pack_small_kernel<4> : quads <= 8 ? pack_small_kernel<8> : pack_small_kernel<16>;
      hipLaunchKernelGGL(pack_small, dim3((unsigned)((col0 + 16 * NT + 7) / 8)), dim3(1024), 0, st, dV, ldv, (int)ctx->n, nchunks, NT, col0, t,
                         (unsigned*)(w + L.off_colmax), VP, VY);
    } else {
      pack(0, nchunks, NT, col0, ncols, vc, first_pass);
    }
    GP_HIP(ctx, hipGetLastError());
    return GP_OK;
  };
  // Where the path still depends on the norms of the rows being packed, the first pass's operands are packed before they are
  // waited for: the host's wait is hidden behind them.  With the packing in one kernel, gp_predict n = 41157, m = 4573, t = 1
  // 78 -> 64 us; n = 13500, m = 1500, t = 65 73 -> 52 us.
  bool packed = false;
  if (rows && rows->path == GP_PATH_PENDING) {
    const int c = y ? 1 : 0, NT = pass_tiles(t - c);
    int rc = t == 1 && rows->v_prepared ? GP_OK : pack_pass(NT, c, t - c < 16 * NT ? t - c : 16 * NT, y ? 0 : -1, true);
    if (rc < 0 || (rc = gp_rows_path(ctx, rows)) < 0) return rc;
    if (rows->path == GP_PATH_FP32) return GP_TO_FP32;
    packed = true;
  }

  const int XP = rows ? (rows->path == GP_PATH_F16X3 ? 3 : 2) : ctx->XP;
  if (XP == 3 && rows) {      // test inputs farther out than the training inputs
    const int rc = gp_rows_x3(ctx, rows);
    if (rc < 0) return rc;
  }
  PlanH pl = plan_h(ctx, nrows, win ? win->nchunks : 0, t, XP);
  L = scratch_layout(ctx, t, pl.JS, nrows);
  const PanelsH pn = scratch_bytes < L.total && pl.JS > 1 && !defer && !win && !rows ? plan_panels(ctx, nrows, t, XP, pl, L, scratch_bytes) : PanelsH{0, pl.JS};
  if (pn.rows) L = scratch_layout(ctx, t, 1, nrows), L.off_part = panel_images_at(L, pn.group, pl), L.total = scratch_bytes;
  if (scratch_bytes < L.total)
    return gp_fail(ctx, GP_ERR_WORKSPACE, "gp_kmv: scratch %zu < %zu bytes", scratch_bytes, L.total);
  float* part = (float*)(w + L.off_part);
  const bool split = pl.JS > 1;

  TileArgsH a;
  const int64_t per_chunk = 2 * dist_groups(XP, dist_shape_of(XP, ctx->d, ctx->kernel == GP_SE_ARD)) * 64;      // units of 32 points
  a.XA = (const u32x4*)ctx->dDA[XP - 2] + (win ? win->chunk0 * per_chunk : 0);
  a.XB = (const u32x4*)(rows ? rows->DB[XP - 2] : ctx->dDB[XP - 2]);
  a.CI = rows ? rows->CI : ctx->dCI;
  a.VP = VP;
  a.VY = VY;
  a.V = dV;
  a.ldv = ldv;
  a.colmax = colmax;
  a.OUT = split ? part : dOut;
  a.ldo = split ? t : ldo;
  a.split_stride = split ? nrows * (int64_t)t : 0;
  a.n = nrows;
  a.diag = (rows || win) ? 0 : 1;
  a.nchunks = nchunks;
  a.JS = pl.JS;
  a.cps = pl.cps;
  a.CG = pl.CG;
  a.a2 = (float)(ctx->a * ctx->a);
  a.sigma2 = (float)(ctx->sigma * ctx->sigma);
  a.add_noise = add_noise;
  a.win_sel = nullptr;
  a.win_block = 0;
  a.gather = rows ? rows->gather : nullptr;
  a.npoints = ctx->n - first;
  a.cm_ld = 0;
  a.done = nullptr;
  a.diag_shift = 0;

  auto sum_images_of = [&](int64_t m, int width, bool add, float* out) {     // out = the sum of the images of m rows
    // the sums of a square product run in one order, whatever its images are cut into (gp_kmv_static)
    const bool share = rows && a.JS >= 16 && m * width <= 65536;
    const int64_t per = share ? 128 : 1024;
    int blocks = (int)((m * width + per - 1) / per);
    if (blocks > 8 * ctx->num_cu) blocks = 8 * ctx->num_cu;
    hipLaunchKernelGGL((share ? kmv_reduce_f16_kernel<8> : kmv_reduce_f16_kernel<1>), dim3(blocks), dim3(256), 0, st, (const float*)part, a.split_stride, a.JS, m, width, add ? 1 : 0,
                       out, ldo);
  };
  int vcol = y ? 0 : -1;
  int c = vcol >= 0 ? 1 : 0;
  bool first_pass = true;
  do {
    const int rem = t - c;
    const int NT = pass_tiles(rem);
    a.col0 = c;
    a.ncols = rem < 16 * NT ? rem : 16 * NT;
    a.vcol = vcol;
    const int vc = vcol;
    vcol = -1;
    if (!packed && pn.group == pl.JS) {
      const int rc = pack_pass(NT, a.col0, a.ncols, vc, first_pass);
      if (rc < 0) return rc;
    }
    packed = false;
    a.clear = accumulate && first_pass ? ctx->dColmax : nullptr;
    a.clear_n = t;
    const TileKernelH k = tile_kernel_h(ctx, XP, NT, a.vcol >= 0, a.gather ? FORM_ANY : FORM_PLAIN, pl.wide);
    if (!k.fn) return gp_fail(ctx, GP_ERR_ARG, "gp_kmv: no fp16 kernel for d=%d", ctx->d);
    const int col = a.vcol >= 0 ? a.vcol : a.col0, width = a.ncols + (a.vcol >= 0 ? 1 : 0);   // the pass's columns
    const int64_t panel = pn.rows ? pn.rows : nrows;
    for (int64_t r0 = 0; r0 < nrows; r0 += panel) {
      const int64_t m = nrows - r0 < panel ? nrows - r0 : panel;
      for (int j0 = 0; j0 < pl.JS; j0 += pn.group) {
        if (pn.rows) {     // a panel is a set of rows of its own, a group of column ranges a point set of its own
          const int c0 = j0 * pl.cps;
          a.JS = min(pn.group, pl.JS - j0);
          a.nchunks = min(a.JS * pl.cps, nchunks - c0);
          a.npoints = ctx->n - (int64_t)c0 * 32;
          a.n = m;
          a.diag_shift = (int)(r0 / 32) - c0;
          a.add_noise = add_noise && j0 == 0;
          a.V = dV + r0 * ldv;
          a.VY = VY + (int64_t)c0 * 32;
          a.VP = VP + (pn.group < pl.JS ? 0 : (int64_t)c0 * 2 * NT * 64);
          a.XA = (const u32x4*)ctx->dDA[XP - 2] + c0 * per_chunk;
          a.XB = (const u32x4*)ctx->dDB[XP - 2] + (r0 / 32) * per_chunk;
          a.CI = ctx->dCI + r0;
          a.ldo = width;
          a.split_stride = m * width;
          a.OUT = part - col;
          if (pn.group < pl.JS) pack(c0, a.nchunks, NT, a.col0, a.ncols, vc, first_pass);
        }
        a.row_blocks = (int)((m + k.rows_per_wg(pl.CG) - 1) / k.rows_per_wg(pl.CG));
        const dim3 grid = tile_grid(a);
        const bool prof = gp_prof_begin(ctx, GP_PROF_TILE);
        hipLaunchKernelGGL(k.fn, grid, dim3(64 * TILE_WAVES), 0, st, a);
        GP_HIP(ctx, hipGetLastError());
        gp_prof_end(ctx, prof);
        if (a.clear) ctx->colmax_dirty = 0;
        if (pn.rows) sum_images_of(m, width, j0 > 0, dOut + r0 * ldo + col);
      }
    }
    first_pass = false;
    c += a.ncols;
  } while (c < t);
  if (defer) {
    defer->part = part;
    defer->stride = a.split_stride;
    defer->JS = pl.JS;
  }
  if (split && !defer && !pn.rows) sum_images_of(nrows, t, false, dOut);
  GP_HIP(ctx, hipGetLastError());
  return GP_OK;
}

int64_t gp_packed_units(int t, int64_t nchunks) {
  int64_t u = 0;
  for (int c = vec_columns(t); c < t;) {
    const int NT = pass_tiles(t - c);
    u += nchunks * 2 * NT * 64;
    c += 16 * NT;
  }
  return u;
}

int gp_packed_images(const gp_ctx* ctx, int t, int64_t rows, int64_t col_chunks) {
  int most = 1;
  for (int XP = 2; XP <= 3; ++XP) {
    const int js = plan_h(ctx, rows, col_chunks, t, XP).JS;
    if (js > most) most = js;
  }
  return most;
}

int gp_kmv_packed(gp_ctx* ctx, int t, const KmvPacked& pk, const int* gather, int64_t nrows, const KmvBlock* win, int* images) {
  if (!gather) nrows = ctx->n;
  const PlanH pl = plan_h(ctx, nrows, win ? win->nchunks : 0, t, ctx->XP);
  const int nchunks = win ? win->nchunks : (int)((ctx->n + 31) / 32);
  TileArgsH a;
  a.XA = (const u32x4*)ctx->dDA[ctx->XP - 2];
  a.XB = (const u32x4*)ctx->dDB[ctx->XP - 2];
  a.CI = ctx->dCI;
  a.win_sel = win ? win->sel : nullptr;
  a.win_block = win ? win->block : 0;
  a.gather = gather;
  a.npoints = ctx->n;
  a.clear = nullptr;
  a.clear_n = 0;
  a.VY = pk.VY;
  a.V = nullptr;
  a.ldv = 0;
  a.colmax = pk.colmax;
  a.OUT = pk.images;
  a.ldo = 0;
  a.split_stride = pk.ld * (int64_t)t;
  a.n = nrows;
  a.diag = (gather || win) ? 0 : 1;
  a.nchunks = nchunks;
  a.JS = pl.JS;
  a.cps = pl.cps;
  a.CG = pl.CG;
  a.a2 = (float)(ctx->a * ctx->a);
  a.sigma2 = 0.0f;
  a.add_noise = 0;
  a.cm_ld = pk.ld;
  a.done = pk.done;
  a.diag_shift = 0;
  const u32x4* VP = (const u32x4*)pk.VP;
  int vcol = vec_columns(t) ? 0 : -1;
  int c = vcol >= 0 ? 1 : 0;
  do {
    const int rem = t - c, NT = pass_tiles(rem);
    a.VP = VP;
    a.col0 = c;
    a.ncols = rem < 16 * NT ? rem : 16 * NT;
    a.vcol = vcol;
    vcol = -1;
    const TileKernelH k = tile_kernel_h(ctx, ctx->XP, NT, a.vcol >= 0, gather ? FORM_GATHER : win ? FORM_WINDOW : FORM_COLUMNS, pl.wide);
    if (!k.fn) return gp_fail(ctx, GP_ERR_ARG, "gp_kmv: no fp16 kernel for d=%d", ctx->d);
    a.row_blocks = (int)((nrows + k.rows_per_wg(pl.CG) - 1) / k.rows_per_wg(pl.CG));
    const dim3 grid = tile_grid(a);
    const bool prof = gp_prof_begin(ctx, GP_PROF_TILE);
    hipLaunchKernelGGL(k.fn, grid, dim3(64 * TILE_WAVES), 0, ctx->stream, a);
    GP_HIP(ctx, hipGetLastError());
    gp_prof_end(ctx, prof);
    VP += (int64_t)nchunks * 2 * NT * 64;
    c += a.ncols;
  } while (c < t);
  *images = pl.JS;
  return GP_OK;
}
