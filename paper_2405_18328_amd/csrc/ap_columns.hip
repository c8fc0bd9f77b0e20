// Alternating projections with one workgroup per column, for n <= AP_COLUMNS_MAX_N and at most AP_COLUMNS_MAX_BLOCKS
// blocks on the split-fp16 product paths: the same step, block choice and stopping rule as ap_kernels.hip (whose
// factorisation it uses), in four launches per step instead of five and without the host between steps.
//
//   apc_solve   d = H[I,I]^-1 R[I,:] on the fp32 matrix cores, spread over the chip
//   apc_pack    V[I] += d, the columns' largest |d| and the operands of the product with d
//   tile pass   H[:,I] d over the chosen block's column window, images column by column
//   apc_update  R -= H[:,I] d, squared residual norms per block; the workgroup that arrives last
//               applies the stopping rule and picks the next block
// The chosen block is read on the device by all of them, so the host queues steps ahead; kernels queued past the
// end return at once.
// Measured on MI355X, n = 16384 d = 26 t = 65, block 2000: 79 -> 65 us per block update (product 27, solve 12, pack 6, update
// 14 us), the whole marginal-likelihood step 6.45 -> 6.09 ms (the factorisation is most of it).  Ahead of the general kernels at
// every size measured up to its limits, n = 2048 .. 65536, 3 .. 256 blocks, t = 1 .. 256, by 3 % or more.
#include "columns.h"
#include "ap_inverse.h"

namespace {

struct ApCols {
  ColFlags* flags;            // pad: the block chosen for the running step
  unsigned long long* post;   // [POSTS], step k in entry k % POSTS: steps finished (low half), done bit, block << 1
  double* bn2;        // [t]
  double* bnorm;      // [t][nb] squared residual norms per block
  double* bpart;      // [t][parts] squared norms of the right-hand sides per part (start only)
  float* tol;         // [t]
  float* relres;      // [t]
  int* frozen;        // [t]
  int* zero_rhs;      // [t]
  unsigned* colmax;   // [t]
  const int* fac_breakdown;
  const float* Hinv;  // [nb] inverses
  float *V, *R;       // [t][ld]
  float* D;           // [SOLVE_KS][t][BP] the solve's ranges; their sum, the update on the chosen block's rows, in the first
  float* VY;          // the vector-ALU column of the product with D
  u32x4* VP;
  const float* images;
  int JS;
  int64_t stride;     // between images
  int64_t n, ld;
  int t, block, nb, BP, win_chunks;
  float sigma2;
};

constexpr int POSTS = 16;
constexpr int AP_FEW_BLOCKS = 40;    // up to here one wave per block ends a step, beyond it a thread per block (see there)

// d = H[I,I]^-1 R[I,:] for the block the last step chose.  One workgroup per 32 rows, 16 NTL columns and one of SOLVE_KS
// ranges of the contraction index, whose sums apc_pack adds (v_mfma_f32_16x16x4_f32: A operand lane l holds A[l % 16][l / 16],
// B operand B[l / 16][l % 16], result register v of lane l is D[4 (l / 16) + v][l % 16]).  Every operand load is 16 bytes per
// lane: four consecutive contraction indices 4 (l / 16) .. + 3 of a row of the inverse (see ap_inverse.h) and of a column
// of R; instruction j of four contracts over the indices {4 h + j}.  The range is cut over the eight waves, whose tiles
// are added in a fixed order through LDS.
// Bound by memory latency and, below it, by the fp32 matrix rate (4.3 us for a block of 2000 and 80 columns): the inverse
// (16 MB) is read once for all columns up to 80, and a wave has its whole range in flight at once.  One workgroup per
// 16 rows and 32 columns, with the range uncut, took 19 us (the inverse read three times); now 12 us.
constexpr int SOLVE_WAVES = 8;
constexpr int SOLVE_KS = 4;
constexpr int SOLVE_G = 4;     // groups of 16 contraction indices per batch of loads
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // four floats at a 4-byte aligned address

template <int NTL>
__global__ __launch_bounds__(64 * SOLVE_WAVES) void apc_solve_kernel(ApCols s) {
  __shared__ f32x4 red[SOLVE_WAVES][2 * NTL][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lo = lane & 15, hi = lane >> 4;
  const int row0 = 32 * (blockIdx.x / SOLVE_KS), ks = blockIdx.x % SOLVE_KS;
  const int cbase = 16 * NTL * blockIdx.y;
  const int done = s.flags->all_done, k = s.flags->pad;
  if (done) return;
  const int64_t j0 = (int64_t)k * s.block;
  const int bs = (int)min((int64_t)s.block, s.n - j0);
  if (row0 >= bs) return;
  const int kw = ((bs + SOLVE_WAVES * SOLVE_KS - 1) / (SOLVE_WAVES * SOLVE_KS) + 15) & ~15;   // indices per wave, a multiple of 16
  const int mb = (ks * SOLVE_WAVES + wave) * kw;
  const int me = min(mb + kw, bs);
  const float* ap = s.Hinv + (int64_t)k * s.BP * s.BP + hinv_at(row0 + lo, 4 * hi, s.BP);
  const int64_t next_panel = row0 + 16 < s.BP ? (int64_t)16 * s.BP : 0;
  const float* bp[NTL];
#pragma unroll
  for (int i = 0; i < NTL; ++i) bp[i] = s.R + (int64_t)min(cbase + 16 * i + lo, s.t - 1) * s.ld + j0 + 4 * hi;
  const int ntile = min(NTL, (s.t - cbase + 15) / 16);    // tiles with a column
  f32x4 acc[2][NTL];
#pragma unroll
  for (int z = 0; z < 2; ++z)
#pragma unroll
    for (int i = 0; i < NTL; ++i) acc[z][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int m0 = mb; m0 < me; m0 += 16 * SOLVE_G) {
    f32x4 av[SOLVE_G][2];
    f4u bv[SOLVE_G][NTL];
#pragma unroll
    for (int g = 0; g < SOLVE_G; ++g) {
      const int m = min(m0 + 16 * g, (me - 1) & ~15);
#pragma unroll
      for (int z = 0; z < 2; ++z) av[g][z] = *reinterpret_cast<const f32x4*>(ap + z * next_panel + hinv_step() * (m >> 2));
#pragma unroll
      for (int i = 0; i < NTL; ++i) bv[g][i] = *reinterpret_cast<const f4u*>(bp[i] + m);
    }
#pragma unroll
    for (int g = 0; g < SOLVE_G; ++g) {
      const int m = m0 + 16 * g;
      if (m < me) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool ok = m + 4 * hi + j < me;    // past the block: not the block's rows (or the array's), whatever they hold
#pragma unroll
          for (int i = 0; i < NTL; ++i) {
            if (i < ntile) {
              const float b = ok ? bv[g][i][j] : 0.0f;
#pragma unroll
              for (int z = 0; z < 2; ++z) acc[z][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? av[g][z][j] : 0.0f, b, acc[z][i], 0, 0, 0);
            }
          }
        }
      }
    }
  }
#pragma unroll
  for (int z = 0; z < 2; ++z)
#pragma unroll
    for (int i = 0; i < NTL; ++i) red[wave][z * NTL + i][lane] = acc[z][i];
  __syncthreads();
  for (int q = wave; q < 2 * NTL; q += SOLVE_WAVES) {
    const int z = q / NTL, i = q % NTL;
    const int c = cbase + 16 * i + lo, row = row0 + 16 * z + 4 * hi;
    f32x4 sum = red[0][q][lane];
#pragma unroll
    for (int w = 1; w < SOLVE_WAVES; ++w) sum += red[w][q][lane];
    if (c < s.t && row < s.BP) *reinterpret_cast<f32x4*>(s.D + ((int64_t)ks * s.t + c) * s.BP + row) = sum;   // rows past bs: padding of D
  }
}

// d = the sum of the solve's ranges, V[I] += d; its largest element and its operands for one column, shifted to the chunk the block starts in, zero off the block.
__global__ __launch_bounds__(CT) void apc_pack_kernel(ApCols s) {
  __shared__ float shf[16];
  const int c = block_column(s.t);
  if (c < 0) return;
  const int done = s.flags->all_done, k = s.flags->pad, stopped = s.frozen[c];
  if (done || stopped) return;
  const int64_t j0 = (int64_t)k * s.block;
  const int bs = (int)min((int64_t)s.block, s.n - j0);
  const int shift = (int)(j0 & 31);
  const int q4 = 4 * (int)threadIdx.x - shift;       // the block's row of this thread's first window row
  f32x4 d = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (q4 + q >= 0 && q4 + q < bs) {
      float* at = s.D + (int64_t)c * s.BP + q4 + q;
      float v = 0.0f;
#pragma unroll
      for (int ks = 0; ks < SOLVE_KS; ++ks) v += at[(int64_t)ks * s.t * s.BP];
      d[q] = v;
      *at = v;               // for the update of this step
      s.V[(int64_t)c * s.ld + j0 + q4 + q] += v;
    }
  const float m = column_max(fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fmaxf(fabsf(d[2]), fabsf(d[3]))), shf);
  if (threadIdx.x == 0) s.colmax[c] = __float_as_uint(m);
  const PackSpot spot = pack_spot(s.VP, s.t, s.win_chunks, c);
  if ((int)threadIdx.x < 8 * s.win_chunks) {
    if (spot.base) pack_quad(spot, threadIdx.x, d * pack_scale(m));
    else *reinterpret_cast<f32x4*>(s.VY + 4 * threadIdx.x) = d;
  }
}

// Squared norms of sq over the blocks that meet rows [r0, r1), sq[0] being row `base`, added to bn[k - k0]: one wave per
// block, fixed order.
__device__ __forceinline__ void block_norms(const float* sq, int64_t base, int64_t r0, int64_t r1, const ApCols& s, int k0, double* bn) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int64_t k = r0 / s.block + wave; k * s.block < r1; k += CT / 64) {
    const int64_t b0 = max(k * s.block, r0), b1 = min((k + 1) * s.block, r1);
    const float* p = sq - base;
    double v = 0.0, v1 = 0.0, v2 = 0.0, v3 = 0.0;
    int64_t r = b0 + lane;
    for (; r + 192 < b1; r += 256) {
      v += (double)p[r];
      v1 += (double)p[r + 64];
      v2 += (double)p[r + 128];
      v3 += (double)p[r + 192];
    }
    for (; r < b1; r += 64) v += (double)p[r];
    v = (v + v1) + (v2 + v3);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) bn[k - k0] += v;
  }
}

__device__ __forceinline__ void put(double* at, double v) { __hip_atomic_store(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double get(const double* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// START: R holds B and V holds x0 (or 0); R -= H x0 when warm; initial state.  Otherwise one step behind its product.
// Workgroup (c, p) works on part p of the blocks of column c, in stretches of 4096 Q rows whose loads are all in flight
// together; the squares of a stretch go to LDS, where a wave adds up each block's.  The workgroup that takes the last
// ticket then applies the stopping rule to every column and picks the block with the largest residual over the columns still
// being updated, lowest index on a tie.  What it reads of the others (block norms) is written and read with
// agent-scope accesses, which go past the XCDs' own L2, and every writer waits for its stores before it takes
// its ticket: no release fence, which would write the whole L2 back.
template <int Q, bool START>
__global__ __launch_bounds__(CT) void apc_update_kernel(ApCols s, int warm) {
  __shared__ float sq[CROWS * Q];
  __shared__ double bn[AP_COLUMNS_MAX_BLOCKS];
  __shared__ double shd[16];
  __shared__ int live[GP_MAX_T];
  __shared__ int best_at[CT / 64];
  __shared__ int last, any_live, any_bad;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int c = blockIdx.y, parts = gridDim.x;
  const int64_t col = (int64_t)c * s.ld;
  const int k0 = (int)((int64_t)s.nb * blockIdx.x / parts), k1 = (int)((int64_t)s.nb * (blockIdx.x + 1) / parts);
  const int64_t r0 = (int64_t)k0 * s.block, r1 = min((int64_t)k1 * s.block, s.n);
  const int q_end = (int)((r1 + 3) / 4);
  f32x4 r[Q], h[Q];
  auto fetch = [&](int base) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int k = min(base + CT * j + tid, q_end - 1);
      r[j] = *reinterpret_cast<const f32x4*>(s.R + col + 4 * k);
      if (!START || warm) h[j] = sum_images<4>(s.images, s.JS, s.stride, col + 4 * k, 4 * k, s.n);
    }
  };
  // what the workgroup that ends the step needs of the column it will judge, requested by all (it is not known yet which)
  const int q0 = min(tid, s.t - 1);
  const int stopped0 = START ? 0 : s.frozen[q0];
  double bn2 = START ? 0.0 : s.bn2[q0];
  const float tol = s.tol[q0];
  const int broken = *s.fac_breakdown;
  fetch((int)(r0 / 4));      // ahead of what says whether and where there is something to do
  int64_t j0 = 0;
  int bs = 0;
  bool go = true;
  if (!START) {
    const int done = s.flags->all_done, k = s.flags->pad, stopped = s.frozen[c];
    if (done) return;
    j0 = (int64_t)k * s.block;
    bs = (int)min((int64_t)s.block, s.n - j0);
    go = !stopped;
  }
  if (go) {
    for (int k = tid; k < k1 - k0; k += CT) bn[k] = 0.0;
    double bb = 0.0;
    for (int base = (int)(r0 / 4); base < q_end; base += CT * Q) {
      if (base > (int)(r0 / 4)) fetch(base);
      __syncthreads();     // bn is cleared, and the squares of the stretch before have been read
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const int k = base + CT * j + tid;
        if (k < q_end) {
          if (START) {
            f32x4 own = r[j];
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (4 * k + q < r0 || 4 * k + q >= r1) own[q] = 0.0f;
            bb += dot4(own, own);
            if (warm) {
              const f32x4 x = *reinterpret_cast<const f32x4*>(s.V + col + 4 * k);
#pragma unroll
              for (int q = 0; q < 4; ++q) r[j][q] -= fmaf(s.sigma2, x[q], h[j][q]);
            }
          } else {
            const int64_t own = 4 * (int64_t)k - j0;       // row of the block of this quad's first row
            if (own > -4 && own < bs) {
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (own + q >= 0 && own + q < bs) h[j][q] = fmaf(s.sigma2, s.D[(int64_t)c * s.BP + own + q], h[j][q]);
            }
            r[j] -= h[j];
          }
          *reinterpret_cast<f32x4*>(sq + 4 * (k - base)) = r[j] * r[j];
          if (!START || warm) {
            if (4 * k >= r0 && 4 * k + 4 <= r1) {
              *reinterpret_cast<f32x4*>(s.R + col + 4 * k) = r[j];
            } else {                                       // shared with the neighbouring part: own rows only
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (4 * k + q >= r0 && 4 * k + q < r1) s.R[col + 4 * k + q] = r[j][q];
            }
          }
        }
      }
      __syncthreads();
      block_norms(sq, 4 * (int64_t)base, max(4 * (int64_t)base, r0), min(4 * (int64_t)(base + CT * Q), r1), s, k0, bn);
    }
    if (START) {
      const double b2 = column_sum(bb, shd);
      if (tid == 0) put(&s.bpart[(int64_t)c * parts + blockIdx.x], b2);
    }
    __syncthreads();
    for (int k = tid; k < k1 - k0; k += CT) put(&s.bnorm[(int64_t)c * s.nb + k0 + k], bn[k]);
  }
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
  __syncthreads();
  if (tid == 0) {
    last = atomicAdd(&s.flags->ticket, 1ull) + 1 == (unsigned long long)gridDim.x * gridDim.y;
    any_live = 0;
    any_bad = broken ? 1 : 0;
  }
  __syncthreads();
  if (!last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  // Judges a column by the sum of its block norms; by the thread of the column's number.
  auto judge = [&](double v) {
    bool goes_on = false;
    if (!stopped0) {
      const int zero = bn2 == 0.0;
      const double rel = zero ? 0.0 : sqrt(v / bn2);
      goes_on = !(zero || (float)rel < tol);
      if (START) {
        s.bn2[tid] = bn2;
        s.zero_rhs[tid] = zero;
      }
      s.relres[tid] = (float)rel;
      s.frozen[tid] = goes_on ? 0 : 1;
      if (goes_on) any_live = 1;
      if (!zero && (!(rel == rel) || rel > 3.0e38)) any_bad = 1;
    }
    live[tid] = goes_on ? 1 : 0;
  };
  // The block norms are staged in LDS, as many columns at a time as fit: all loads of a thread in flight together, those of the
  // next columns ahead of the work on these.
  double* norms = reinterpret_cast<double*>(sq);
  constexpr int NORMS = CROWS * Q / 2, PER = NORMS / CT;
  const int cols = min(min(s.t, AP_COLUMNS_MAX_BLOCKS), NORMS / s.nb);    // their sums go to bn
  double next[PER];
  auto request = [&](int c0) {
    const int count = min(cols, s.t - c0) * s.nb;
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (tid + CT * u < count) next[u] = get(&s.bnorm[(int64_t)c0 * s.nb + tid + CT * u]);
  };
  auto stage = [&](int c0) {
    const int count = min(cols, s.t - c0) * s.nb;
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (tid + CT * u < count) norms[tid + CT * u] = next[u];
    __syncthreads();
  };
  request(0);
  if (START && tid < s.t)
    for (int k = 0; k < parts; ++k) bn2 += get(&s.bpart[(int64_t)tid * parts + k]);
  stage(0);
  double best = -1.0;
  int at = 0x7fffffff;
  if (cols == s.t && s.nb <= AP_FEW_BLOCKS) {
    // few blocks: a thread per column, then a wave per block
    if (tid < s.t) {
      double v = 0.0;
      for (int k = 0; k < s.nb; ++k) v += norms[tid * s.nb + k];
      judge(v);
    }
    __syncthreads();
    for (int k = wave; k < s.nb; k += CT / 64) {
      double v = 0.0;
      for (int q = lane; q < s.t; q += 64)
        if (live[q]) v += norms[q * s.nb + k];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
      if (v > best) {
        best = v;
        at = k;
      }
    }
  } else {
    // 16 lanes add up a column; a thread per block, in `groups` groups of columns, adds up the block over the columns that go on.
    // Per block update: n = 65536 block 256 t = 65 (three stages; the thread of a column read its norms one after the other)
    // 87 -> 70 us; n = 16384 t = 17, a wave per block -> a thread per block: 128 blocks 41.7 -> 36.2 us, 41 blocks 36.5 -> 36.2,
    // 17 blocks (n = 8192) 36.1 -> 36.9.
    const int log_nb = s.nb <= 64 ? 6 : s.nb <= 128 ? 7 : 8;
    const int mine = tid & ((1 << log_nb) - 1), group = tid >> log_nb, groups = CT >> log_nb;
    double score = 0.0;
    for (int c0 = 0; c0 < s.t; c0 += cols) {
      const int nc = min(cols, s.t - c0);
      if (c0 + cols < s.t) request(c0 + cols);
      for (int q = tid >> 4; q < nc; q += CT / 16) {
        double v = 0.0;
        for (int k = tid & 15; k < s.nb; k += 16) v += norms[q * s.nb + k];
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if ((tid & 15) == 0) bn[q] = v;
      }
      __syncthreads();
      if (tid >= c0 && tid < c0 + nc) judge(bn[tid - c0]);
      __syncthreads();
      if (mine < s.nb)
        for (int q = group; q < nc; q += groups)
          if (live[c0 + q]) score += norms[q * s.nb + mine];
      __syncthreads();     // the next columns take the place of these
      if (c0 + cols < s.t) stage(c0 + cols);
    }
    norms[tid] = score;
    __syncthreads();
    if (tid < s.nb) {
      double v = 0.0;
      for (int g = 0; g < groups; ++g) v += norms[(g << log_nb) + tid];
      if (v > best) {
        best = v;
        at = tid;
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {     // the largest, the lowest block on a tie
      const double v = __shfl_xor(best, off);
      const int k = __shfl_xor(at, off);
      if (v > best || (v == best && k < at)) {
        best = v;
        at = k;
      }
    }
  }
  if (lane == 0) {
    shd[wave] = best;
    best_at[wave] = at;
  }
  __syncthreads();
  if (tid) return;
  for (int w = 1; w < CT / 64; ++w)
    if (shd[w] > best || (shd[w] == best && best_at[w] < at)) {
      best = shd[w];
      at = best_at[w];
    }
  ColFlags* f = s.flags;
  const bool over = any_bad || !any_live;
  const int iters = f->iters + (START ? 0 : 1);
  const int sel = at < s.nb ? at : 0;
  f->ticket = 0;
  f->iters = iters;
  f->bad = any_bad;
  f->pad = sel;
  f->all_done = over ? 1 : 0;
  const unsigned long long word = (unsigned long long)(unsigned)(iters + 1) |
                                  ((unsigned long long)((over ? COL_DONE : 0u) | ((unsigned)sel << 1)) << 32);
  __hip_atomic_store(s.post + iters % POSTS, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Layout {
  int nb, BP, batch, win_chunks, parts;
  int64_t ld, units;
  size_t off_hinv, off_A, off_W, off_T, off_DI, off_V, off_R, off_D, off_VY, off_bnorm, off_bpart, off_state, off_VP, off_images, total;
};

Layout layout(const gp_ctx* ctx, int t, int block) {
  Layout L;
  L.nb = (int)((ctx->n + block - 1) / block);
  L.BP = (block + AP_TILE - 1) / AP_TILE * AP_TILE;
  L.batch = L.nb < AP_FACTOR_BATCH ? L.nb : AP_FACTOR_BATCH;
  L.ld = (ctx->n + 31) / 32 * 32;
  L.win_chunks = (block + 31 + 31) / 32;           // a block that starts inside a chunk touches one more
  if (L.win_chunks > L.ld / 32) L.win_chunks = (int)(L.ld / 32);
  L.units = gp_packed_units(t, L.ld / 32);
  // Parts of a column in the update, each with a whole number of blocks: as many workgroups as there are compute units, or
  // fewer.  A few more than that run behind the others: t = 65, 4 parts (260 workgroups) -> 3, per block update,
  // n = 8192 block 500 51.9 -> 45.8 us, n = 16384 block 2000 70.5 -> 64.7 us, n = 65536 block 500 98.6 -> 88.5 us.
  L.parts = ctx->num_cu / t > 0 ? ctx->num_cu / t : 1;
  if (L.parts > L.nb) L.parts = L.nb;
  const size_t bp2 = (size_t)L.BP * L.BP;
  const size_t arr = align_up((size_t)L.ld * t * sizeof(float), 256);
  size_t o = 0;
  L.off_hinv = o; o += align_up((size_t)L.nb * bp2 * sizeof(float), 256);
  L.off_A = o; o += align_up((size_t)L.batch * bp2 * sizeof(double), 256);
  L.off_W = o; o += align_up((size_t)L.batch * bp2 * sizeof(double), 256);
  L.off_T = o; o += align_up((size_t)L.batch * bp2 * sizeof(double), 256);
  L.off_DI = o; o += align_up((size_t)L.batch * L.BP * AP_TILE * sizeof(double), 256);
  L.off_V = o; o += arr;
  L.off_R = o; o += arr + 256;      // block solves read up to 16 floats past a column's end
  L.off_D = o; o += align_up((size_t)SOLVE_KS * L.BP * t * sizeof(float), 256);
  L.off_VY = o; o += align_up((size_t)L.win_chunks * 32 * sizeof(float), 256);
  L.off_bnorm = o; o += align_up((size_t)L.nb * t * sizeof(double), 256);
  L.off_bpart = o; o += align_up((size_t)L.parts * t * sizeof(double), 256);
  L.off_state = o; o += align_up(sizeof(ColFlags) + 16 + (size_t)t * (sizeof(double) + 2 * sizeof(float) + 3 * sizeof(int)), 256);
  L.off_VP = o; o += align_up((size_t)L.units * 16, 256);
  const int square = gp_packed_images(ctx, t, ctx->n), window = gp_packed_images(ctx, t, ctx->n, L.win_chunks);
  L.off_images = o; o += arr * (size_t)(square > window ? square : window);
  L.total = o;
  return L;
}

}  // namespace

bool gp_ap_by_columns(const gp_ctx* ctx, int block) {
  return ctx->n <= AP_COLUMNS_MAX_N && (ctx->n + block - 1) / block <= AP_COLUMNS_MAX_BLOCKS;
}
size_t gp_ap_columns_workspace_bytes(const gp_ctx* ctx, int t, int block) { return layout(ctx, t, block).total; }

int gp_ap_columns_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
                      const float* h_tol, int block, int max_iters, void* dWork, int* h_iters, int* h_kmv_count,
                      float* h_relres, int* h_picks) {
  const Layout L = layout(ctx, t, block);
  hipStream_t st = ctx->stream;
  char* w = (char*)dWork;
  ApCols s;
  int* fac_breakdown;
  {
    char* q = w + L.off_state;
    s.flags = (ColFlags*)q; q += sizeof(ColFlags);
    fac_breakdown = (int*)q; q += 16;
    s.bn2 = (double*)q; q += sizeof(double) * t;
    s.tol = (float*)q; q += sizeof(float) * t;
    s.relres = (float*)q; q += sizeof(float) * t;
    s.frozen = (int*)q; q += sizeof(int) * t;
    s.zero_rhs = (int*)q; q += sizeof(int) * t;
    s.colmax = (unsigned*)q;
  }
  s.fac_breakdown = fac_breakdown;
  s.Hinv = (const float*)(w + L.off_hinv);
  s.V = (float*)(w + L.off_V);
  s.R = (float*)(w + L.off_R);
  s.D = (float*)(w + L.off_D);
  s.VY = (float*)(w + L.off_VY);
  s.bnorm = (double*)(w + L.off_bnorm);
  s.bpart = (double*)(w + L.off_bpart);
  s.VP = (u32x4*)(w + L.off_VP);
  s.images = (const float*)(w + L.off_images);
  s.JS = 1;
  s.stride = L.ld * (int64_t)t;
  s.n = ctx->n;
  s.ld = L.ld;
  s.t = t;
  s.block = block;
  s.nb = L.nb;
  s.BP = L.BP;
  s.win_chunks = L.win_chunks;
  s.sigma2 = (float)(ctx->sigma * ctx->sigma);

  // Pinned staging: tolerances in, flags and residuals out.  Written by the host only here; every solver
  // synchronises the stream before it returns, so the copy a previous call queued from it has run.
  if (sizeof(ColFlags) + sizeof(float) * t * 2 > GP_PIN_THETA)
    return gp_fail(ctx, GP_ERR_ARG, "gp_ap_solve: t too large for the pinned staging block");
  ColFlags* hflags = (ColFlags*)((char*)ctx->hPinned + GP_PIN_SOLVER);
  float* htol = (float*)(hflags + 1);
  float* hrel = htol + t;
  for (int c = 0; c < t; ++c) htol[c] = h_tol[c];
  volatile unsigned long long* hpost = (volatile unsigned long long*)((char*)ctx->hPinned + GP_PIN_POST);
  s.post = (unsigned long long*)((char*)ctx->dPinned + GP_PIN_POST);
  for (int k = 0; k < POSTS; ++k) hpost[k] = 0;

  // an error return leaves nothing of this solve running: queued kernels would post into the next solve
  auto drained = [&](int rc) -> int {
    (void)hipStreamSynchronize(st);
    return rc;
  };
  auto failed = [&](hipError_t e) -> bool {
    if (e != hipSuccess) (void)drained(gp_fail(ctx, GP_ERR_HIP, "gp_ap_solve: %s", hipGetErrorString(e)));
    return e != hipSuccess;
  };

  const dim3 grid(column_blocks(t)), cblock(CT);
  if (failed(hipMemcpyAsync(s.tol, htol, sizeof(float) * t, hipMemcpyHostToDevice, st))) return GP_ERR_HIP;
  auto clear = [&](void* p, size_t bytes) {
    const int64_t units = (int64_t)(bytes / 16);
    int blocks = (int)((units + 255) / 256);
    if (blocks > 4 * ctx->num_cu) blocks = 4 * ctx->num_cu;
    if (blocks > 0) hipLaunchKernelGGL(clear_units_kernel, dim3(blocks), dim3(256), 0, st, (u32x4*)p, units);
  };
  clear(s.flags, sizeof(ColFlags) + 16);
  clear(s.VP, (size_t)L.units * 16);   // columns that pad the last tile, and stopped columns, are never written
  clear(s.D, L.off_bnorm - L.off_D);   // D and VY
  hipLaunchKernelGGL(to_columns_kernel, transpose_grid(L.ld, t, 2), dim3(256), 0, st, dB, ldb, s.R, dX0, ldv, s.V, ctx->n, L.ld, t);
  if (failed(hipGetLastError())) return GP_ERR_HIP;
  int rc = gp_ap_inverses(ctx, block, L.nb, L.BP, L.batch, (float*)(w + L.off_hinv), (double*)(w + L.off_A), (double*)(w + L.off_W),
                          (double*)(w + L.off_T), (double*)(w + L.off_DI), fac_breakdown);
  if (rc < 0) return drained(rc);

  KmvPacked pk;
  pk.VP = s.VP;
  pk.VY = s.V;
  pk.colmax = s.colmax;
  pk.images = (float*)(w + L.off_images);
  pk.ld = L.ld;
  pk.done = nullptr;
  int kmv_count = 0;
  if (dX0) {
    hipLaunchKernelGGL(pack_columns_kernel, grid, cblock, 0, st, (const float*)s.V, s.VP, s.colmax, t, L.ld);
    rc = gp_kmv_packed(ctx, t, pk, nullptr, 0, nullptr, &s.JS);
    if (rc < 0) return drained(rc);
    ++kmv_count;
  }
  const dim3 ugrid(L.parts, t);
  const bool small = (int64_t)((L.nb + L.parts - 1) / L.parts) * block <= 2 * CROWS;   // rows of a part
  hipLaunchKernelGGL((small ? apc_update_kernel<2, true> : apc_update_kernel<4, true>), ugrid, cblock, 0, st, s, dX0 ? 1 : 0);
  if (dX0 && padded_tiles(t)) clear(s.VP, (size_t)L.units * 16);   // the windows' operands are laid out anew
  if (failed(hipGetLastError())) return GP_ERR_HIP;

  const KmvBlock win = {&s.flags->pad, block, L.win_chunks};
  pk.VY = s.VY;
  pk.done = &s.flags->all_done;
  const int rt = (int)(((ctx->n < block ? ctx->n : block) + 31) / 32) * SOLVE_KS;
  const int ct = (t + 15) / 16;
  auto* solve = ct == 1 ? apc_solve_kernel<1> : ct <= 3 ? apc_solve_kernel<3> : apc_solve_kernel<5>;
  const dim3 solve_grid(rt, ct == 1 ? 1 : ct <= 3 ? 1 : (ct + 4) / 5);
  auto* update = small ? apc_update_kernel<2, false> : apc_update_kernel<4, false>;
  // Steps queued ahead of the flags the host has seen; kernels queued past the end return at once.
  const int ahead = ctx->prof_mask ? 0 : 3;
  bool done = false;
  int sel = 0;
  auto wait_steps = [&](int steps) -> int {      // and the block chosen at the end of them
    unsigned long long seen = 0;
    const int r = wait_post(ctx, "gp_ap_solve", hpost + steps % POSTS, (unsigned)steps + 1, &seen);
    done = ((seen >> 32) & COL_DONE) != 0;
    sel = (int)((seen >> 33) & 0x7FFFFFFFu);
    return r;
  };
  rc = wait_steps(0);
  if (rc < 0) return drained(rc);
  for (int finished = 0, queued = 0; !done && finished < max_iters; ++finished) {
    for (; queued < max_iters && queued <= finished + ahead; ++queued) {
      hipLaunchKernelGGL(solve, solve_grid, dim3(64 * SOLVE_WAVES), 0, st, s);
      hipLaunchKernelGGL(apc_pack_kernel, grid, cblock, 0, st, s);
      rc = gp_kmv_packed(ctx, t, pk, nullptr, 0, &win, &s.JS);
      if (rc < 0) return drained(rc);
      hipLaunchKernelGGL(update, ugrid, cblock, 0, st, s, 0);
      if (failed(hipGetLastError())) return GP_ERR_HIP;
    }
    if (h_picks) h_picks[finished] = sel;
    rc = wait_steps(finished + 1);
    if (rc < 0) return drained(rc);
  }

  hipLaunchKernelGGL(from_columns_kernel, transpose_grid(L.ld, t, 1), dim3(256), 0, st, (const float*)s.V, L.ld, ctx->n, t,
                     (const int*)s.zero_rhs, dV, ldv);
  if (failed(hipGetLastError())) return GP_ERR_HIP;
  if (failed(hipMemcpyAsync(hrel, s.relres, sizeof(float) * t, hipMemcpyDeviceToHost, st))) return GP_ERR_HIP;
  if (failed(hipMemcpyAsync(hflags, s.flags, sizeof(ColFlags), hipMemcpyDeviceToHost, st))) return GP_ERR_HIP;
  if (failed(hipStreamSynchronize(st))) return GP_ERR_HIP;
  if (h_iters) *h_iters = hflags->iters;
  if (h_kmv_count) *h_kmv_count = kmv_count;
  if (h_relres)
    for (int c = 0; c < t; ++c) h_relres[c] = hrel[c];
  if (hflags->bad)
    return gp_fail(ctx, GP_ERR_BREAKDOWN, "gp_ap_solve: a diagonal block is not positive definite in fp64, or a non-finite residual (step %d)", hflags->iters);
  return hflags->all_done ? GP_OK : GP_NOT_CONVERGED;
}
