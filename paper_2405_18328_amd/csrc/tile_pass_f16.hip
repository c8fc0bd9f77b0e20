// Matrix-free product OUT = K V (+ sigma^2 V), split-fp16 matrix-core path.
//
// On gfx950 the fp32 MFMA shares the SIMD's FMA lanes with the VALU (measured: VALU work adds to
// fp32-MFMA time instead of hiding under it), while the fp16 MFMA runs on the matrix cores at 16x the
// rate and overlaps with VALU work.  This path therefore evaluates both contractions of the tile pass
// with v_mfma_f32_32x32x16_f16 on operands split into fp16 pieces, fp32 accumulation:
//   x = hi + mid (+ lo), each piece an 11-bit fp16 mantissa, so
//   a.b ~ ah.bh + ah.bm + am.bh (+ ah.bl + al.bh + am.bm): relative error 2^-22 (2^-33), i.e. fp32-class.
// The VALU keeps what needs fp32: the kernel function (exp2 / sqrt) and the split of phi.
//
// Per 32x32 tile of pairs (j, i), one wavefront:
//   1. S[j][i] = XA_j . XB_i     3 (or 6) MFMAs per 16 components      (= g r^2_ij [+ 15 for SE])
//   2. phi' = 2^15 phi(S)        VALU; hi = phi' cut to fp16, lo = phi' - hi rounded; packed to fp16 pairs
//   3. OUT_i += phi'[i][j] V'_j  2 k-steps x NT x 3 MFMAs; V' = V scaled per column by a power of two
//                                so that max |V'_c| is in [2^13, 2^14), pre-split and pre-packed
// The accumulator layout of step 1 (lane = i, register r <-> j = 8(r/4) + 4(lane/32) + r%4) gives each lane
// eight consecutive registers per k-step that are exactly its eight A-operand elements, provided the
// V' rows are packed in that order; phi never leaves registers, K is never stored.
#include <cstdlib>

#include "gpws_internal.h"
#include "split_f16.h"

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

namespace {

struct TileArgsH {
  const u32x4* XA[3];     // column-side pieces, 16-byte units [(chunk*KH + kh)*64 + lane]
  const u32x4* XB[3];     // row-side pieces
  const u32x4* VP;        // packed V' images of this pass, [chunk][mh][nt][part][lane]
  const float* VY;        // [n_pad] the VALU column, unscaled (zeros when unused)
  const float* V;         // the caller's V (noise term in the epilogue)
  int64_t ldv;
  const unsigned* colmax; // [t] bit patterns of max_i |V_ic|
  float* OUT;
  int64_t ldo;
  int64_t split_stride;
  int64_t n;               // rows of the output (the context's n, or m for a rectangular product)
  int diag;                // square product: the pair (i, i) gets r^2 = 0 exactly
  int diag_shift;          // chunk of the first row minus the first chunk of the contraction
  int nchunks;             // column chunks (always the context's points)
  int col0, ncols, vcol;
  int JS, cps;             // column-range splits inside this launch, chunks per split
  float a2, sigma2;
  int add_noise;
  unsigned* clear;         // column maxima in accumulation: everyone has read them, workgroup 0 zeroes them (clear_n words); NULL: none
  int clear_n;
  const int* win_sel;      // contraction over the columns of block *win_sel (win_block points each): XA starts at that block's
  int win_block;           // first chunk, and chunks past the last one are not there; NULL: XA as it is
  const int* gather;       // row i of the output is the context's point gather[i] (an index outside [0, npoints) reads point 0); NULL: i
  int64_t npoints;
  int64_t cm_ld;           // > 0: images are column-major with this many rows per column (a multiple of 32)
  const int* done;         // a non-zero value there turns the launch into a no-op; NULL: always runs
};

// What a tile kernel is compiled for, besides the row-major product of gp_kmv and gp_predict (FORM_PLAIN).  The shapes
// that fill the register file are built once per form: with all options in one kernel, KH = 1 NT = 2 MI = 2
// kept 65 registers in scratch memory (now 2) and the wide kernel 15 (none; FORM_PLAIN 7).  Before -> after:
// a CG iteration, d = 11, t = 65, n = 16384 201 -> 161 us, n = 65536 2428 -> 2105 us; a block update of alternating
// projections, n = 16384 d = 5 t = 65, block 2000, 97 -> 71 us.
enum {
  FORM_PLAIN,
  FORM_COLUMNS,   // the solvers' products: column-major images, early return
  FORM_GATHER,    // and rows gathered from the context's points
  FORM_WINDOW,    // and a column window chosen on the device
  FORM_ANY        // all of it, chosen by the arguments
};
constexpr bool has_gather(int form) { return form == FORM_GATHER || form == FORM_ANY; }
constexpr bool has_window(int form) { return form == FORM_WINDOW || form == FORM_ANY; }

// where this lane's row operands of sub-tile `sub` start (units; + kh * 64 per distance step)
template <int KH>
__device__ __forceinline__ int64_t row_operand(const TileArgsH& p, int64_t sub, int lane) {
  if (!p.gather) return sub * KH * 64 + lane;
  const int64_t slot = sub * 32 + (lane & 31);
  const int64_t v = p.gather[slot < p.n ? slot : 0];
  const int64_t i = v >= 0 && v < p.npoints ? v : 0;
  return (i >> 5) * KH * 64 + (lane & 32) + (i & 31);
}

// first chunk of the column side (0 unless the launch works on a block chosen on the device)
__device__ __forceinline__ int64_t window_chunk(const TileArgsH& p) {
  return p.win_sel ? ((int64_t)*p.win_sel * p.win_block) >> 5 : 0;
}

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// one lane's 16 accumulators of a column: four runs of four rows, eight rows apart, as 16-byte stores (a lane pair
// covers 32 consecutive bytes); the accumulators are cleared
__device__ __forceinline__ void store_column_quads(float* dst, bool ok, bool first, float scale, f32x16& acc) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    f32x4 v = scale * f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    if (ok) {
      f32x4* d = reinterpret_cast<f32x4*>(dst + 8 * g);
      if (!first) v += *d;
      *d = v;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[4 * g + q] = 0.0f;
  }
}

// One lane's 16 accumulators of a column into a row-major output: first stores, later adds to what is there; noise adds
// sigma^2 V.  All loads go out before the first value is used, with clamped indices instead of a branch around each, behind which they
// were waited for one by one; the branches also kept 27 registers of the KH = 1, NT = 2, MI = 2 kernel in scratch memory (now 2).
// gp_kmv n = 16384, d = 11, t = 65 (SE) 149 -> 139 us; d = 26 (Matern) 187 -> 186 us.
__device__ __forceinline__ void store_row_elements(const TileArgsH& p, float* out, int64_t ibase, int h, int c, bool first, bool noise,
                                                   float scale, f32x16& acc) {
  const bool cok = c < p.ncols;
  const int64_t col = p.col0 + (cok ? c : 0);
  auto row = [&](int r) { return ibase + 8 * (r >> 2) + 4 * h + (r & 3); };
  float v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    v[r] = scale * acc[r];
    acc[r] = 0.0f;
  }
  if (noise) {
    float w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) w[r] = p.V[min(row(r), p.n - 1) * p.ldv + col];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = fmaf(p.sigma2, w[r], v[r]);
  }
  if (!first) {
    float w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) w[r] = out[min(row(r), p.n - 1) * p.ldo + col];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] += w[r];
  }
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (cok && row(r) < p.n) out[row(r) * p.ldo + col] = v[r];
}

// Two waves per SIMD with two software pipelines.  Four wavefronts per workgroup: every workgroup streams all
// of V' and XA through its LDS, so the L2-to-LDS traffic of a launch is inversely proportional to the
// rows a workgroup owns (128 MI; eight waves halve the traffic and measured no faster).
template <int KIND, int KH, int XP, int NT, int MI, bool Y, int FORM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void kmv_tile_f16_kernel(TileArgsH p) {
  // One pipeline stage in LDS, in 16-byte units: G groups of 64 units (one wave-wide 16-byte load
  // each): XP*KH groups of XA pieces, then 4*NT groups of V' images; then one 8-unit y slot per wave.
  constexpr int W = 4;
  constexpr int XA_G = XP * KH;
  constexpr int V_G = 4 * NT;
  constexpr int G = XA_G + V_G;
  constexpr int V_OFF = XA_G * 64;
  constexpr int V_U = V_G * 64;
  constexpr int VY_OFF = G * 64;
  constexpr int STAGE = VY_OFF + (Y ? 8 * W : 0);
  constexpr int NS = G > 12 ? 3 : 4;               // stages: chunks up to ch + NS - 1 are in flight while ch is consumed
  constexpr int DEPTH = NS - 1;
  constexpr int LPW = (G + W - 1) / W;             // group loads per wave per chunk
  constexpr int LPC = LPW + (Y ? 1 : 0);           // + the y slot
  static_assert((DEPTH - 1) * LPC < 64, "vmcnt cannot express the pipeline depth");
  __shared__ u32x4 lds[NS][STAGE];

  constexpr bool CM = FORM != FORM_PLAIN;
  const int over = CM && p.done ? *p.done : 0;   // looked at only once the first loads are on their way
  if (p.clear && blockIdx.x == 0)
    for (int c = threadIdx.x; c < p.clear_n; c += blockDim.x) p.clear[c] = 0u;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction: lets the compiler branch on it
  const int h = lane >> 5;
  const int li = lane & 31;
  const int js = blockIdx.x % p.JS;
  const int rb = blockIdx.x / p.JS;
  const int sub0 = (rb * W + wave) * MI;
  const int diag_at = p.diag ? sub0 + p.diag_shift : -MI;     // the chunk that holds the first sub-tile's own points
  // The workgroup's column range [r_begin, r_end) is walked in segments [c_begin, c_end) of at most
  // GP_FLUSH_CHUNKS chunks; the accumulators are added into OUT after each segment (see flush below).
  const int64_t chunk0 = has_window(FORM) ? window_chunk(p) : 0;
  const int r_begin = js * p.cps;
  const int r_end = has_window(FORM) ? (int)min((int64_t)min(p.nchunks, r_begin + p.cps), (p.npoints + 31) / 32 - chunk0) : min(p.nchunks, r_begin + p.cps);
  int c_begin = r_begin;
  int c_end = min(r_end, c_begin + GP_FLUSH_CHUNKS);

  // row-side operands: registers for the whole pass
  f16x8 xb[MI][XP][KH];
#pragma unroll
  for (int m = 0; m < MI; ++m) {
    const int64_t at = has_gather(FORM) ? row_operand<KH>(p, sub0 + m, lane) : (int64_t)(sub0 + m) * KH * 64 + lane;
#pragma unroll
    for (int pc = 0; pc < XP; ++pc)
#pragma unroll
      for (int kh = 0; kh < KH; ++kh) xb[m][pc][kh] = as_f16x8(p.XB[pc][at + kh * 64]);
  }

  f32x16 acc[MI][NT];
  float accv[MI];
#pragma unroll
  for (int m = 0; m < MI; ++m) {
    accv[m] = 0.0f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][nt][r] = 0.0f;
  }

  // Staging goes global -> LDS directly (global_load_lds_dwordx4: lane L of a wave lands at the
  // wave's LDS base + 16 L), NS - 1 chunks ahead of the chunk being consumed, so no registers are held
  // and the L2/HBM latency is spread over several chunks of work.  Every wave issues the same number of
  // loads per chunk (its groups wave, wave + W, ..; surplus slots repeat the last group, which rewrites
  // identical bytes), so one vmcnt value tells each wave when its part of a chunk has landed; the
  // barrier that follows makes the whole chunk visible.
  const u32x4* g_src[LPW];
  int g_stride[LPW], g_off[LPW];
#pragma unroll
  for (int x = 0; x < LPW; ++x) {
    const int g = min(wave + W * x, G - 1);
    if (g < XA_G) {
      g_src[x] = p.XA[g / KH] + (chunk0 * KH + g % KH) * 64 + lane;
      g_stride[x] = KH * 64;
    } else {
      g_src[x] = p.VP + (g - XA_G) * 64 + lane;
      g_stride[x] = V_U;
    }
    g_off[x] = g * 64;
  }
  // The loads are issued through inline assembly on purpose: the compiler's wait-count pass treats an
  // LDS-DMA load as aliasing every later LDS read and would drain all chunks in flight (vmcnt(0)) at
  // each barrier.  Here the ordering is explicit instead: s_waitcnt vmcnt(WAIT_N), then the barrier.
  const bool vy_lane = lane < 8;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)&lds[0][0];
  unsigned g_lds[LPW];
#pragma unroll
  for (int x = 0; x < LPW; ++x) g_lds[x] = __builtin_amdgcn_readfirstlane(lds_base + 16u * (unsigned)g_off[x]);
  const unsigned vy_lds = __builtin_amdgcn_readfirstlane(lds_base + 16u * (unsigned)(VY_OFF + 8 * wave));
  auto dma16 = [](const u32x4* src, unsigned lds_addr) {
    // m0 carries the LDS address of the load; it is declared clobbered, so the compiler keeps nothing in it
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds_addr) : "memory", "m0");
  };
  auto issue_chunk = [&](int ch_target) {
    const int ch = min(ch_target, c_end - 1);           // past the end: harmless reload of the last chunk
    const unsigned stage_off = (unsigned)((ch_target - c_begin) % NS) * (unsigned)(STAGE * 16);
#pragma unroll
    for (int x = 0; x < LPW; ++x) dma16(g_src[x] + (int64_t)ch * g_stride[x], __builtin_amdgcn_readfirstlane(g_lds[x] + stage_off));
    if (Y && vy_lane) dma16(reinterpret_cast<const u32x4*>(p.VY + (int64_t)ch * 32) + lane, __builtin_amdgcn_readfirstlane(vy_lds + stage_off));
  };
  // vmcnt <= (DEPTH-1)*LPC: everything but the newest DEPTH-1 chunks has landed (loads retire in order)
  constexpr int WAIT_N = (DEPTH - 1) * LPC;

  // distance chain of one chunk: S[j][i] = XA_j . XB_i, with the pair (i, i) forced to r^2 = 0
  auto distance = [&](int ch, f32x16 (&S)[MI]) {
    const u32x4* s = lds[(ch - c_begin) % NS];
#pragma unroll
    for (int m = 0; m < MI; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) S[m][r] = 0.0f;
#pragma unroll
    for (int kh = 0; kh < KH; ++kh) {
      f16x8 xa[XP];
#pragma unroll
      for (int pc = 0; pc < XP; ++pc) xa[pc] = as_f16x8(s[(pc * KH + kh) * 64 + lane]);
#pragma unroll
      for (int m = 0; m < MI; ++m) {
        // smallest terms first
        if constexpr (XP == 3) {
          S[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[1], xb[m][1][kh], S[m], 0, 0, 0);
          S[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[2], xb[m][0][kh], S[m], 0, 0, 0);
          S[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[0], xb[m][XP - 1][kh], S[m], 0, 0, 0);
        }
        S[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[1], xb[m][0][kh], S[m], 0, 0, 0);
        S[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[0], xb[m][1][kh], S[m], 0, 0, 0);
        S[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[0], xb[m][0][kh], S[m], 0, 0, 0);
      }
    }
#pragma unroll
    for (int m = 0; m < MI; ++m) {
      if (ch == diag_at + m) {
        // one chunk in thousands: an opaque statement keeps this a real (wave-uniform) branch instead of
        // sixteen selects executed on every chunk
        asm volatile("" ::: "memory");
        const float s0 = KIND == GP_SE_ARD ? (float)PHI_SHIFT : 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r >> 2) + 4 * h + (r & 3) == li) S[m][r] = s0;
      }
    }
  };

  // ---- main loop ---------------------------------------------------------------------------------
  // A chunk is worked through in NG = 2 MI groups of 8 values per lane (group g = (mh, m): the k-step
  // mh of sub-tile m).  Two software pipelines keep the matrix core and the VALU busy together:
  //   * the distance chain runs one chunk ahead (S of chunk ch + 1 while chunk ch is consumed);
  //   * the phi/split stage runs one group ahead of the contraction, and the two are emitted as
  //     bundles "one MFMA, then the VALU work of one value pair".  The matrix pipe accepts an MFMA only
  //     when it is free; a wave that reaches its next MFMA early stalls there with its VALU work
  //     undone, so MFMAs are spaced by at least their own duration of VALU instructions.
  constexpr int NG = 2 * MI;
  constexpr int MPG = 3 * NT;        // contraction MFMAs per group

  // phi and its split for values 2 e2, 2 e2 + 1 of group (mh, m); vy = the lane's y values for that mh
  auto phi_pair = [&](const f32x16& Sv, int mh, int e2, const f32x4 (&vy)[2], float& av, unsigned& oh, unsigned& ol) {
    float f[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      const int e = 2 * e2 + z;
      const float sv = Sv[8 * mh + e];
      if (KIND == GP_SE_ARD) {
        f[z] = __builtin_amdgcn_exp2f(sv);                 // sv = -log2(e)/2 r^2 + 15
      } else {
        // sv = 3 r^2; a rounding-level negative value is mirrored instead of clamped (|.| is a free
        // source modifier), the pair (i, i) was set to exactly 0 above
        const float u = __builtin_amdgcn_sqrtf(__builtin_fabsf(sv));
        const float ex = __builtin_amdgcn_exp2f(fmaf(u, -LOG2E, (float)PHI_SHIFT));
        f[z] = fmaf(u, ex, ex);
      }
      if (Y) av = fmaf(f[z], vy[e >> 2][e & 3], av);
    }
    split_pair_positive(f[0], f[1], oh, ol);
  };
  auto load_vy = [&](const u32x4* s, int mh, f32x4 (&vy)[2]) {
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2) vy[g2] = __builtin_bit_cast(f32x4, s[VY_OFF + 8 * wave + 2 * (2 * mh + g2) + h]);
  };

  f32x16 S0[MI], S1[MI];             // S of the chunk being consumed / of the next chunk, roles alternate
  unsigned ph[4], pl[4];             // packed A operands of the group about to be contracted
  f32x4 vy0[2];                      // y values of k-step 0 of the chunk being consumed
  // fills the pipelines at the start of a segment: DEPTH chunks in flight, S and the first phi group of
  // the first chunk ready
  auto segment_prologue = [&]() {
#pragma unroll
    for (int d0 = 0; d0 < DEPTH; ++d0) issue_chunk(c_begin + d0);
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(WAIT_N) : "memory");
    __syncthreads();
    distance(c_begin, S0);
    if (Y) load_vy(lds[0], 0, vy0);
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) phi_pair(S0[0], 0, e2, vy0, accv[0], ph[e2], pl[e2]);
  };

  // one chunk: S = its distances (ready), Sn = receives the next chunk's
  auto chunk_body = [&](int ch, f32x16 (&S)[MI], f32x16 (&Sn)[MI]) {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(WAIT_N - LPC) : "memory");
    __syncthreads();            // chunks <= ch + 1 are complete in LDS; every wave is done with chunk ch - 1
    issue_chunk(ch + DEPTH);    // refills the stage chunk ch - 1 occupied
    const u32x4* s = lds[(ch - c_begin) % NS];
    const u32x4* s_next = lds[(ch + 1 - c_begin) % NS];
    // every LDS operand of the chunk is fetched here, ahead of the distance chain, so that no MFMA or
    // VALU instruction further down waits on LDS latency
    f16x8 bh[2][NT], bl[2][NT];
#pragma unroll
    for (int mh = 0; mh < 2; ++mh)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        bh[mh][nt] = as_f16x8(s[V_OFF + ((mh * NT + nt) * 2 + 0) * 64 + lane]);
        bl[mh][nt] = as_f16x8(s[V_OFF + ((mh * NT + nt) * 2 + 1) * 64 + lane]);
      }
    f32x4 vy1[2], vy0n[2];
    if (Y) {
      load_vy(s, 1, vy1);
      load_vy(s_next, 0, vy0n);
      // past the last chunk the look-ahead group must not reach the y accumulator
      const float keep = ch + 1 < c_end ? 1.0f : 0.0f;
      vy0n[0] *= keep;
      vy0n[1] *= keep;
    }
    distance(ch + 1, Sn);       // past the last chunk this reads a harmless reload of it

#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int mh = g / MI, m = g % MI;
      // the group whose phi stage rides along: g + 1 of this chunk, or group 0 of the next chunk
      const bool wrap = g + 1 == NG;
      const int gn = wrap ? 0 : g + 1;
      const int mhn = gn / MI, mn = gn % MI;
      const f32x4 (&vyn)[2] = wrap ? vy0n : (mhn == 0 ? vy0 : vy1);
      const f16x8 ah = as_f16x8(u32x4{ph[0], ph[1], ph[2], ph[3]}), al = as_f16x8(u32x4{pl[0], pl[1], pl[2], pl[3]});
      unsigned nh[4], nl[4];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < MPG; ++k) {
        const int nt = k / 3, term = k % 3;      // smallest terms first: lo*hi, hi*lo, hi*hi
        acc[m][nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(term == 0 ? al : ah, term == 1 ? bl[mh][nt] : bh[mh][nt],
                                                            acc[m][nt], 0, 0, 0);
        // the 4 value pairs of the next group, spread over the MPG bundles
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2)
          if ((e2 * MPG) / 4 == k) phi_pair(wrap ? Sn[mn] : S[mn], mhn, e2, vyn, accv[mn], nh[e2], nl[e2]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        ph[e2] = nh[e2];
        pl[e2] = nl[e2];
      }
    }
    if (Y) {
      vy0[0] = vy0n[0];
      vy0[1] = vy0n[1];
    }
  };

  // Writes what the accumulators hold to OUT (first: stores, adds the noise term once; later: adds to
  // what is there) and clears them.  Undoes the power-of-two scalings and multiplies by a^2.
  float* out = p.OUT + (int64_t)js * p.split_stride;
  float oscale[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int c = min(li + 32 * nt, p.ncols - 1);
    oscale[nt] = p.a2 * ldexpf(1.0f, column_exponent(p.colmax[p.col0 + c]) - V_TOP - PHI_SHIFT);
  }
  auto flush = [&](bool first) {
    const bool noise = first && p.add_noise && js == 0;
    // an opaque zero keeps the address arithmetic of the flush inside it: hoisted out of the segment
    // loop it would hold dozens of registers across the main loop
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
#pragma unroll
    for (int m = 0; m < MI; ++m) {
      const int64_t ibase = (int64_t)(sub0 + m) * 32 + zero;
      if (FORM == FORM_ANY ? p.cm_ld != 0 : CM) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int c = li + 32 * nt;
          store_column_quads(out + (int64_t)(p.col0 + c) * p.cm_ld + ibase + 4 * h, c < p.ncols && ibase < p.cm_ld, first,
                             oscale[nt], acc[m][nt]);
        }
        if (Y) {
          const float tot = accv[m] + __shfl_xor(accv[m], 32);
          if (h == 0 && ibase < p.cm_ld) {
            float* o = out + (int64_t)p.vcol * p.cm_ld + ibase + li;
            const float v = p.a2 * ldexpf(1.0f, -PHI_SHIFT) * tot;
            *o = first ? v : *o + v;
          }
          accv[m] = 0.0f;
        }
        continue;
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) store_row_elements(p, out, ibase, h, li + 32 * nt, first, noise, oscale[nt], acc[m][nt]);
      if (Y) {
        const float tot = accv[m] + __shfl_xor(accv[m], 32);
        const int64_t i = ibase + li;
        if (h == 0 && i < p.n) {
          float v = p.a2 * ldexpf(1.0f, -PHI_SHIFT) * tot;
          if (noise) v = fmaf(p.sigma2, p.V[i * p.ldv + p.vcol], v);
          if (!first) v += out[i * p.ldo + p.vcol];
          out[i * p.ldo + p.vcol] = v;
        }
        accv[m] = 0.0f;
      }
    }
  };

  // Rounding error of an fp32 accumulator grows with the length of its chain of partial sums, so the
  // accumulators are added into OUT after every segment (the running sum then sees one addition per
  // segment).  The same threads read and write the same elements: no race, fixed order.
  if (over) return;
  bool first = true;
  if (has_window(FORM) && r_begin >= r_end) {   // a block at the end of the points is shorter than the launch
    flush(true);
    return;
  }
  for (;;) {
    segment_prologue();
    for (int ch = c_begin; ch < c_end; ch += 2) {
      chunk_body(ch, S0, S1);
      if (ch + 1 < c_end) chunk_body(ch + 1, S1, S0);
    }
    // no LDS write may be in flight, and no wave still reading, when the ring is refilled or released
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    flush(first);
    first = false;
    if (c_end >= r_end) break;
    c_begin = c_end;
    c_end = min(r_end, c_begin + GP_FLUSH_CHUNKS);
  }
}

// ---- four waves per SIMD ----------------------------------------------------------------------------
// The same tile pass laid out for more waves instead of software pipelines: 128 registers hold one
// sub-tile of 32 rows, and the other three waves of the SIMD are the pipeline.  Eight waves per workgroup
// share a stage of two chunks in LDS, two stages deep, one barrier per two chunks.  NT = 0 is the product
// with a single vector (the mean of a prediction): no contraction tiles at all, phi goes straight into one
// FMA per pair, eight waves per SIMD.
// What bounds it (SQ counters, n = 32768, d = 26, t = 65, Matern): the vector port in use 69 % and the matrix core 60 % of
// the cycles; the two-wave kernel at n = 16384: 62 % and 49 %.
// Measured against the two-wave kernel, same box: n = 16384 d = 26 t = 65 Matern 164 -> 160 us; n = 32768
// d = 26 t = 65 SE 553 -> 516 us; one vector: n = 41157 d = 9 Matern 508 -> 409 us, n = 65536 d = 8 SE 892 -> 564 us.
// With KH = 1 or NT = 1 the two-wave kernel with two sub-tiles per wave reads half the operands from LDS and stays ahead.
constexpr int wide_waves(int KH, int XP, int NT) { return NT ? 4 : KH <= 2 ? 8 : XP * KH <= 16 ? 4 : 2; }   // per SIMD

template <int KIND, int KH, int XP, int NT, bool Y, int FORM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(wide_waves(KH, XP, NT), wide_waves(KH, XP, NT)))) void kmv_tile_f16_wide_kernel(TileArgsH p) {
  constexpr int W = 8;
  constexpr int XA_G = XP * KH;                     // groups of 64 16-byte units per chunk
  constexpr int V_G = 4 * NT;
  constexpr int G = XA_G + V_G;
  constexpr int V_OFF = XA_G * 64;                  // in units, inside a chunk
  constexpr int CH_U = G * 64;                      // units per chunk
  constexpr int VY_OFF = 2 * CH_U;                  // the two chunks' 32 y values each: 16 units
  constexpr int STAGE = 2 * CH_U + (Y ? 16 : 0);
  constexpr int LPW = (2 * G + W - 1) / W;          // group loads per wave and stage; surplus slots repeat the last group
  __shared__ u32x4 lds[2][STAGE];

  constexpr bool CM = FORM != FORM_PLAIN;
  const int over = CM && p.done ? *p.done : 0;   // looked at only once the first loads are on their way
  if (p.clear && blockIdx.x == 0)
    for (int c = threadIdx.x; c < p.clear_n; c += blockDim.x) p.clear[c] = 0u;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5;
  const int li = lane & 31;
  const int js = blockIdx.x % p.JS;
  const int rb = blockIdx.x / p.JS;
  const int sub0 = rb * W + wave;
  const int diag_at = p.diag ? sub0 + p.diag_shift : -1;
  const int64_t chunk0 = has_window(FORM) ? window_chunk(p) : 0;
  const int r_begin = js * p.cps;
  const int r_end = has_window(FORM) ? (int)min((int64_t)min(p.nchunks, r_begin + p.cps), (p.npoints + 31) / 32 - chunk0) : min(p.nchunks, r_begin + p.cps);
  int c_begin = r_begin;
  int c_end = min(r_end, c_begin + GP_FLUSH_CHUNKS);

  f16x8 xb[XP][KH];
  const int64_t row_at = has_gather(FORM) ? row_operand<KH>(p, sub0, lane) : (int64_t)sub0 * KH * 64 + lane;
#pragma unroll
  for (int pc = 0; pc < XP; ++pc)
#pragma unroll
    for (int kh = 0; kh < KH; ++kh) xb[pc][kh] = as_f16x8(p.XB[pc][row_at + kh * 64]);

  static_assert(NT > 0 || Y, "nothing to multiply");
  f32x16 acc[NT > 0 ? NT : 1];
  float accv[2] = {0.0f, 0.0f};
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nt][r] = 0.0f;

  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)&lds[0][0];
  const unsigned lane16 = lane * 16u;
  // group g of a stage: chunk g / G, then XA pieces, then V' images; source = uniform base + 16 lane
  auto dma16 = [](uint64_t base, unsigned off, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
  };
  auto issue_pair = [&](int ch0, int st) {
#pragma unroll
    for (int x = 0; x < LPW; ++x) {
      const int g = min(wave + W * x, 2 * G - 1);
      const int gc = g >= G ? g - G : g;
      const int ch = min(g >= G ? ch0 + 1 : ch0, c_end - 1);     // past the end: harmless reload of the last chunk
      const u32x4* src;
      if (gc < XA_G) src = p.XA[gc / KH] + ((chunk0 + ch) * KH + gc % KH) * 64;
      else src = p.VP + ((int64_t)ch * V_G + (gc - XA_G)) * 64;
      dma16((uint64_t)src, lane16, lds_base + 16u * (unsigned)(st * STAGE + g * 64));
    }
    if (Y) {   // every wave fetches the same 256 bytes to the same place
      const int ch = min(ch0 + (lane >> 3), c_end - 1);
      if (lane < 16) dma16((uint64_t)p.VY, (unsigned)ch * 128u + (lane & 7) * 16u, lds_base + 16u * (unsigned)(st * STAGE + VY_OFF));
    }
  };

  auto phi_pair = [&](float s0, float s1, const f32x4& vy, int q, unsigned& oh, unsigned& ol) {
    float f[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      const float sv = z ? s1 : s0;
      if (KIND == GP_SE_ARD) {
        f[z] = __builtin_amdgcn_exp2f(sv);
      } else {
        const float u = __builtin_amdgcn_sqrtf(__builtin_fabsf(sv));
        const float ex = __builtin_amdgcn_exp2f(fmaf(u, -LOG2E, (float)PHI_SHIFT));
        f[z] = fmaf(u, ex, ex);
      }
      if (Y) accv[z] = fmaf(f[z], vy[q + z], accv[z]);
    }
    if constexpr (NT > 0) {
      split_pair_positive(f[0], f[1], oh, ol);
    }
  };

  auto chunk = [&](int ch, const u32x4* s, const u32x4* sy) {
    f32x16 S;
#pragma unroll
    for (int r = 0; r < 16; ++r) S[r] = 0.0f;
#pragma unroll
    for (int kh = 0; kh < KH; ++kh) {
      f16x8 xa[XP];
#pragma unroll
      for (int pc = 0; pc < XP; ++pc) xa[pc] = as_f16x8(s[(pc * KH + kh) * 64 + lane]);
      // smallest terms first
      if constexpr (XP == 3) {
        S = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[1], xb[1][kh], S, 0, 0, 0);
        S = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[2], xb[0][kh], S, 0, 0, 0);
        S = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[0], xb[XP - 1][kh], S, 0, 0, 0);
      }
      S = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[1], xb[0][kh], S, 0, 0, 0);
      S = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[0], xb[1][kh], S, 0, 0, 0);
      S = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[0], xb[0][kh], S, 0, 0, 0);
    }
    if (ch == diag_at) {
      asm volatile("" ::: "memory");
      const float s0 = KIND == GP_SE_ARD ? (float)PHI_SHIFT : 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + 4 * h + (r & 3) == li) S[r] = s0;
    }
#pragma unroll
    for (int mh = 0; mh < 2; ++mh) {
      u32x4 ph, pl;
      f32x4 vy[2];
      if (Y) {
#pragma unroll
        for (int g2 = 0; g2 < 2; ++g2) vy[g2] = __builtin_bit_cast(f32x4, sy[2 * (2 * mh + g2) + h]);
      }
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        unsigned oh = 0, ol = 0;
        phi_pair(S[8 * mh + 2 * e2], S[8 * mh + 2 * e2 + 1], vy[e2 >> 1], 2 * (e2 & 1), oh, ol);
        ph[e2] = oh;
        pl[e2] = ol;
      }
      if constexpr (NT > 0) {
      const f16x8 ah = as_f16x8(ph), al = as_f16x8(pl);
      f16x8 bh[NT], bl[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        bh[nt] = as_f16x8(s[V_OFF + ((mh * NT + nt) * 2 + 0) * 64 + lane]);
        bl[nt] = as_f16x8(s[V_OFF + ((mh * NT + nt) * 2 + 1) * 64 + lane]);
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[nt], acc[nt], 0, 0, 0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[nt], acc[nt], 0, 0, 0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[nt], acc[nt], 0, 0, 0);
      }
    }
  };

  float* out = p.OUT + (int64_t)js * p.split_stride;
  auto flush = [&](bool first) {
    const bool noise = first && p.add_noise && js == 0;
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    const int64_t ibase = (int64_t)sub0 * 32 + zero;
    if (FORM == FORM_ANY ? p.cm_ld != 0 : CM) {
      if constexpr (NT > 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int c = li + 32 * nt;
          const float oscale = p.a2 * ldexpf(1.0f, column_exponent(p.colmax[p.col0 + min(c, p.ncols - 1)]) - V_TOP - PHI_SHIFT);
          store_column_quads(out + (int64_t)(p.col0 + c) * p.cm_ld + ibase + 4 * h, c < p.ncols && ibase < p.cm_ld, first,
                             oscale, acc[nt]);
        }
      }
      if (Y) {
        const float both = accv[0] + accv[1];
        const float tot = both + __shfl_xor(both, 32);
        if (h == 0 && ibase < p.cm_ld) {
          float* o = out + (int64_t)p.vcol * p.cm_ld + ibase + li;
          const float v = p.a2 * ldexpf(1.0f, -PHI_SHIFT) * tot;
          *o = first ? v : *o + v;
        }
        accv[0] = accv[1] = 0.0f;
      }
      return;
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int c = li + 32 * nt;
      const float oscale = p.a2 * ldexpf(1.0f, column_exponent(p.colmax[p.col0 + min(c, p.ncols - 1)]) - V_TOP - PHI_SHIFT);
      store_row_elements(p, out, ibase, h, c, first, noise, oscale, acc[nt]);
    }
    if (Y) {
      const float both = accv[0] + accv[1];
      const float tot = both + __shfl_xor(both, 32);
      const int64_t i = ibase + li;
      if (h == 0 && i < p.n) {
        float v = p.a2 * ldexpf(1.0f, -PHI_SHIFT) * tot;
        if (noise) v = fmaf(p.sigma2, p.V[i * p.ldv + p.vcol], v);
        if (!first) v += out[i * p.ldo + p.vcol];
        out[i * p.ldo + p.vcol] = v;
      }
      accv[0] = accv[1] = 0.0f;
    }
  };

  if (over) return;
  // The row operands are waited for here, where the compiler sees it: it would otherwise wait for them at their first use,
  // inside the loop, and there drain the stage in flight too, every two chunks.  With the stores above, gp_kmv
  // n = 40000, d = 20, t = 65 (SE) 808 -> 790 us.
  __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
  bool first = true;
  if (has_window(FORM) && r_begin >= r_end) {
    flush(true);
    return;
  }
  for (;;) {
    int st = 0;
    issue_pair(c_begin, 0);
    for (int ch = c_begin; ch < c_end; ch += 2) {
      asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
      __syncthreads();              // this stage is complete in LDS, every wave is done with the other one
      issue_pair(ch + 2, st ^ 1);
      const u32x4* s = lds[st];
      chunk(ch, s, s + VY_OFF);
      if (ch + 1 < c_end) chunk(ch + 1, s + CH_U, s + VY_OFF + 8);
      st ^= 1;
    }
    // no LDS write may be in flight, and no wave still reading, when the ring is refilled or released
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    flush(first);
    first = false;
    if (c_end >= r_end) break;
    c_begin = c_end;
    c_end = min(r_end, c_begin + GP_FLUSH_CHUNKS);
  }
}

// ---- per-call operand preparation -------------------------------------------------------------
// colmax[c] = max_i |V_ic| as a bit pattern (non-negative floats order like unsigned ints)
// blockIdx.y = 1 does the same for a second matrix of the same shape.
__global__ __launch_bounds__(256) void colmax_kernel(const float* __restrict__ V, int64_t ldv,
                                                     const float* __restrict__ V2, int64_t ldv2, int64_t n, int t,
                                                     unsigned* __restrict__ colmax, unsigned* __restrict__ colmax2) {
  if (blockIdx.y) {
    V = V2;
    ldv = ldv2;
    colmax = colmax2;
  }
  // a thread keeps one column (per group of 256 columns) and walks rows: consecutive threads read
  // consecutive columns of a row, the running maximum stays in a register
  extern __shared__ unsigned smax[];   // [t]
  for (int c = threadIdx.x; c < t; c += 256) smax[c] = 0u;
  __syncthreads();
  const int64_t rows_per_block = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
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

// zeroes t words of one or two arrays (a kernel, not a memset command: memset nodes recorded into a
// captured graph have misbehaved on replay, and gp_kmv_static must be capturable)
__global__ __launch_bounds__(256) void clear_words_kernel(unsigned* __restrict__ a, unsigned* __restrict__ b, int t) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c < t) {
    a[c] = 0u;
    if (b) b[c] = 0u;
  }
}

// V' images of one column pass: unit u = ((chunk*2 + mh)*NT + nt)*2 + part, lane l: element e is
// V'[32 chunk + 16 mh + 8 (e/4) + 4 (l/32) + e%4][col0 + 32 nt + l%32]; rows >= n and columns past the pass are zero.
__global__ __launch_bounds__(256) void pack_v_kernel(const float* __restrict__ V, int64_t ldv, int64_t n, int nchunks,
                                                     int NT, int col0, int ncols, int vcol,
                                                     const unsigned* __restrict__ colmax, u32x4* __restrict__ VP,
                                                     float* __restrict__ VY, unsigned* __restrict__ copy, int copy_n) {
  if (copy && blockIdx.x == 0)      // the maxima as the tile kernel and later passes read them
    for (int c = threadIdx.x; c < copy_n; c += 256) copy[c] = colmax[c];
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t total = (int64_t)nchunks * 2 * NT * 64;
  if (gid < total) {
    const int lane = (int)(gid & 63);
    int64_t q = gid >> 6;
    const int nt = (int)(q % NT); q /= NT;
    const int mh = (int)(q & 1);
    const int64_t chunk = q >> 1;
    const int hh = lane >> 5;
    const int cc = 32 * nt + (lane & 31);
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
        const int64_t j = chunk * 32 + 16 * mh + 8 * (e >> 2) + 4 * hh + (e & 3);
        f[z] = (cok && j < n) ? V[j * ldv + col] * scale : 0.0f;
      }
      unsigned fh, fl;
      split_pair(f[0], f[1], fh, fl);
      hi[e2] = fh;
      lo[e2] = fl;
    }
    u32x4* dst = VP + ((chunk * 2 + mh) * NT + nt) * 2 * 64;
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
  if (cc >= 32 * NT) return;
  const float scale = cc < 0 ? 1.0f : ldexpf(1.0f, V_TOP - column_exponent(__float_as_uint(mx)));
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int k = ql + 128 * j;
    if (k >= nk) break;                  // whole groups of eight quads
    unsigned hi[2], lo[2];
    split_quad(v[j] * scale, hi, lo);
    const bool up = (k & 2) != 0;        // quads k and k + 2 (sixteen lanes on) make up one high and one low unit
    const unsigned x0 = (unsigned)__shfl_xor((int)(up ? hi[0] : lo[0]), 16);
    const unsigned x1 = (unsigned)__shfl_xor((int)(up ? hi[1] : lo[1]), 16);
    if (cc < 0) {
      *reinterpret_cast<f32x4*>(VY + 4 * k) = v[j];
    } else {
      const u32x4 unit = up ? u32x4{x0, x1, lo[0], lo[1]} : u32x4{hi[0], hi[1], x0, x1};
      VP[((int64_t)((k >> 2) * NT + (cc >> 5)) * 2 + (up ? 1 : 0)) * 64 + (cc & 31) + 32 * (k & 1)] = unit;
    }
  }
}

// OUT = (add: OUT +) sum of the partial images, in order.  A chain of dependent loads bounded it (one element per thread, one image
// after the other); now four consecutive elements per thread, eight images fetched at a time.  With the clearing launch
// of the column maxima gone, gp_predict n = 13500, m = 1500, t = 65: 79 -> 70 us; n = 41157, m = 4573, t = 1: 85 -> 78 us.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void kmv_reduce_f16_kernel(const float* __restrict__ part, int64_t split_stride, int JS, int64_t n,
                                                             int t, int add, float* __restrict__ out, int64_t ldo) {
  const int64_t total = n * t;
  for (int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; e < total; e += (int64_t)gridDim.x * 1024) {
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
    if (add) each([&](int q, const float* o) { s[q] = *o; });
    if (total >= 4) {
      for (int k = 0; k < JS; k += 8) {
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f4u*>(part + (int64_t)min(k + u, JS - 1) * split_stride + at);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (k + u < JS) s += v[u];
      }
    } else {
      for (int q = 0; q < (int)total; ++q)
        for (int k = 0; k < JS; ++k) s[q] += part[(int64_t)k * split_stride + q];
    }
    each([&](int q, float* o) { *o = s[q]; });
  }
}

typedef void (*tileh_fn)(TileArgsH);

template <int KIND, int KH, int XP, int NT, int MI, bool Y>
tileh_fn pick_form(int form) {
  switch (form) {
    case FORM_PLAIN: return kmv_tile_f16_kernel<KIND, KH, XP, NT, MI, Y, FORM_PLAIN>;
    case FORM_COLUMNS: return kmv_tile_f16_kernel<KIND, KH, XP, NT, MI, Y, FORM_COLUMNS>;
    case FORM_GATHER: return kmv_tile_f16_kernel<KIND, KH, XP, NT, MI, Y, FORM_GATHER>;
  }
  return kmv_tile_f16_kernel<KIND, KH, XP, NT, MI, Y, FORM_WINDOW>;
}

template <int KIND, int XP, bool Y>
tileh_fn pick_wide_form(int form) {
  switch (form) {
    case FORM_PLAIN: return kmv_tile_f16_wide_kernel<KIND, 2, XP, 2, Y, FORM_PLAIN>;
    case FORM_COLUMNS: return kmv_tile_f16_wide_kernel<KIND, 2, XP, 2, Y, FORM_COLUMNS>;
    case FORM_GATHER: return kmv_tile_f16_wide_kernel<KIND, 2, XP, 2, Y, FORM_GATHER>;
  }
  return kmv_tile_f16_wide_kernel<KIND, 2, XP, 2, Y, FORM_WINDOW>;
}

template <int KIND, int KH, int XP, bool Y>
tileh_fn pick_h_nt_mi(int NT, int MI, int form) {
  if constexpr (KH == 1) {
    if (MI == 2) return NT == 1 ? pick_form<KIND, KH, XP, 1, 2, Y>(form) : pick_form<KIND, KH, XP, 2, 2, Y>(form);
  }
  if constexpr (KH == 2) {
    if (MI == 2 && NT == 1) return pick_form<KIND, KH, XP, 1, 2, Y>(form);
  }
  return NT == 1 ? kmv_tile_f16_kernel<KIND, KH, XP, 1, 1, Y, FORM_ANY> : kmv_tile_f16_kernel<KIND, KH, XP, 2, 1, Y, FORM_ANY>;
}

template <int KIND, int XP, bool Y>
tileh_fn pick_h_kh(int KH, int NT, int MI, int form) {
  switch (KH) {
    case 1: return pick_h_nt_mi<KIND, 1, XP, Y>(NT, MI, form);
    case 2: return pick_h_nt_mi<KIND, 2, XP, Y>(NT, MI, form);
    case 3: return pick_h_nt_mi<KIND, 3, XP, Y>(NT, MI, form);
    case 4: return pick_h_nt_mi<KIND, 4, XP, Y>(NT, MI, form);
    case 6: return pick_h_nt_mi<KIND, 6, XP, Y>(NT, MI, form);
    case 8: return pick_h_nt_mi<KIND, 8, XP, Y>(NT, MI, form);
  }
  return nullptr;
}

template <int KIND, int XP>
tileh_fn pick_vec_kh(int KH) {
  switch (KH) {
    case 1: return kmv_tile_f16_wide_kernel<KIND, 1, XP, 0, true, FORM_ANY>;
    case 2: return kmv_tile_f16_wide_kernel<KIND, 2, XP, 0, true, FORM_ANY>;
    case 3: return kmv_tile_f16_wide_kernel<KIND, 3, XP, 0, true, FORM_ANY>;
    case 4: return kmv_tile_f16_wide_kernel<KIND, 4, XP, 0, true, FORM_ANY>;
    case 6: return kmv_tile_f16_wide_kernel<KIND, 6, XP, 0, true, FORM_ANY>;
    case 8: return kmv_tile_f16_wide_kernel<KIND, 8, XP, 0, true, FORM_ANY>;
  }
  return nullptr;
}

template <int KIND, int XP>
tileh_fn pick_h(int KH, int NT, int MI, bool wide, bool y, int form) {
  if (NT == 0) return pick_vec_kh<KIND, XP>(KH);
  if (wide) return y ? pick_wide_form<KIND, XP, true>(form) : pick_wide_form<KIND, XP, false>(form);
  return y ? pick_h_kh<KIND, XP, true>(KH, NT, MI, form) : pick_h_kh<KIND, XP, false>(KH, NT, MI, form);
}

// The kernel of one column pass of NT tiles (y: with the extra vector-ALU column).
struct TileKernelH {
  tileh_fn fn;
  int rows_per_wg, threads;
  int per_cu;              // workgroups that share a compute unit
  double chunk_us;         // about what a chunk takes one of them
};

// form: FORM_PLAIN .. FORM_WINDOW (the shape does not depend on it)
TileKernelH tile_kernel_h(const gp_ctx* ctx, int64_t rows, int XP, int NT, bool y, int form) {
  TileKernelH k;
  const int KH = ctx->KH;
  // The wide kernel where it is ahead (see there) and has rows enough: it takes twice the waves to fill the chip, so
  // below 32768 rows twice the column splits, whose images cost what it gains (n = 16384: 6 us against 4).  Two
  // sub-tiles per wave halve the LDS operand traffic; past one k-step of distance operands (two with a
  // single contraction tile) the second sub-tile no longer fits the register file.  Registers kept in scratch memory
  // with two: KH = 1 NT = 2 2 on two pieces, 8 on three; KH = 2 NT = 1 none.
  const bool wide = NT == 0 || (NT == 2 && KH == 2 && rows >= 32768);
  const int MI = !wide && rows >= 8192 && (KH == 1 || (KH == 2 && NT == 1)) ? 2 : 1;
  if (ctx->kernel == GP_SE_ARD) k.fn = XP == 2 ? pick_h<GP_SE_ARD, 2>(KH, NT, MI, wide, y, form) : pick_h<GP_SE_ARD, 3>(KH, NT, MI, wide, y, form);
  else k.fn = XP == 2 ? pick_h<GP_MATERN32_ARD, 2>(KH, NT, MI, wide, y, form) : pick_h<GP_MATERN32_ARD, 3>(KH, NT, MI, wide, y, form);
  k.rows_per_wg = wide ? 256 : 128 * MI;
  k.threads = wide ? 512 : 256;
  if (wide) {
    k.per_cu = wide_waves(KH, XP, NT) / 2;
    k.chunk_us = NT ? 2.5 : 0.3 * wide_waves(KH, XP, NT);
  } else {
    // two workgroups of one wave per SIMD, where their LDS rings fit
    const int G = XP * KH + 4 * NT, NS = G > 12 ? 3 : 4;
    const size_t lds = ((size_t)NS * (G * 64 + (y ? 8 * 4 : 0)) * 16 + 1279) / 1280 * 1280;
    k.per_cu = 2 * lds <= 160 * 1024 ? 2 : 1;
    k.chunk_us = 1.2 * MI;
  }
  return k;
}

struct PlanH {
  int JS, cps;     // column-range splits, chunks per split
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
  L.off_vp = o; o += align_up((size_t)nchunks * 2 * 2 * 2 * 64 * 16, 256);      // NT = 2 images
  L.off_part = o;
  if (JS > 1) o += align_up((size_t)JS * rows * t * sizeof(float), 256);
  L.total = o;
  return L;
}

// tiles of the first (widest) column pass, and whether the vector-ALU column rides along with it: a lone
// column past a multiple of 32 goes there, whose tile would be used for 1/32 of its width
bool has_vec_column(int t) { return t % 32 == 1; }
int pass_tiles(int rem) { return rem > 32 ? 2 : rem > 0 ? 1 : 0; }

PlanH plan_h(const gp_ctx* ctx, int64_t rows, int64_t col_chunks, int t, int XP) {
  PlanH pl;
  const int64_t chunks = col_chunks > 0 ? col_chunks : (ctx->n + 31) / 32;
  for (const SplitMemo& m : ctx->split_memo)
    if (m.JS && m.rows == rows && m.chunks == chunks && m.t == t && m.XP == XP) {
      pl.JS = m.JS;
      pl.cps = (int)((chunks + pl.JS - 1) / pl.JS);
      return pl;
    }
  const bool y = has_vec_column(t);
  const TileKernelH k = tile_kernel_h(ctx, rows, XP, pass_tiles(y ? t - 1 : t), y, FORM_PLAIN);
  const int row_blocks = (int)((rows + k.rows_per_wg - 1) / k.rows_per_wg);
  // a partial image is written and read once, at about 4 TB/s
  const double image = (double)rows * t * sizeof(float);
  // images of more than 2 GB in all would not pay for their memory
  int max_js = image * 64.0 > 2.0e9 ? (int)(2.0e9 / image) : 64;
  if (max_js < 1) max_js = 1;
  pl.JS = gp_column_splits(row_blocks, chunks, k.per_cu * ctx->num_cu, 2.0 * image / 4.0e6 / k.chunk_us, max_js);
  pl.cps = (int)((chunks + pl.JS - 1) / pl.JS);
  gp_ctx* memo = const_cast<gp_ctx*>(ctx);   // a context belongs to one host thread at a time
  memo->split_memo[memo->split_next] = SplitMemo{rows, chunks, t, XP, pl.JS};
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
constexpr int PANEL_ROWS = 256;     // a multiple of every kernel's rows per workgroup

size_t panel_images_at(const ScratchH& L, int group, const PlanH& pl) {
  return L.off_vp + align_up((size_t)group * pl.cps * 2 * 2 * 2 * 64 * 16, 256);
}

// Smaller groups leave room for larger panels.  A launch takes about one unit of time per generation of workgroups, 0.55 where
// there is at most one per compute unit.  gp_kmv_static, Matern-3/2, t = 65, every row's column range in one image -> panels
// (gp_kmv, all images at once): n = 70001 d = 26 4.29 -> 2.86 ms (2.76), n = 150000 d = 5 14.0 -> 11.8 ms (10.6),
// n = 200000 d = 5 24.2 -> 20.7 ms (19.6), n = 240000 d = 5 28.4 -> 29.8 ms (26.8).
PanelsH plan_panels(const gp_ctx* ctx, int64_t nrows, int t, int XP, const PlanH& pl, const ScratchH& L, size_t scratch_bytes) {
  const bool y = has_vec_column(t);
  const TileKernelH k = tile_kernel_h(ctx, nrows, XP, pass_tiles(y ? t - 1 : t), y, FORM_PLAIN);
  const int64_t unit = PANEL_ROWS / k.rows_per_wg, slots = (int64_t)k.per_cu * ctx->num_cu;
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

// A launch runs in generations of `slots` workgroups, and a last generation of a few row blocks costs as much as a
// full one: the time is about generations x (chunks per workgroup + what its prologue and flush cost), and
// every further cut adds one partial image of the output to write and read (image_cost, in units of a
// workgroup's chunk).  Measured on MI355X (gp_predict, n = 41157 and 4573 test points, t = 1: 36 row
// blocks of 128 rows): 15 ranges, 540 workgroups, 149.8 us; 14 ranges, 504 workgroups, 121.9 us.
int gp_column_splits(int row_blocks, int64_t chunks, int slots, double image_cost, int max_splits) {
  constexpr double FIXED = 4.0;       // prologue and flush of a workgroup, in chunks
  constexpr int MIN_CHUNKS = 4;
  // Past four generations the workgroups have drifted apart, which fills the last one by itself, and column ranges only
  // cost locality: 3.1 generations (n = 400000 d = 3 t = 65) split 450 -> 424 ms a CG step; 7.6 (n = 500000 d = 90) 221 ->
  // 225 ms, 15.3 (n = 2000000 d = 11) 1590 -> 1690 ms a product.
  if (row_blocks > 4 * slots) return 1;
  int best = 1;
  double best_cost = 1e300;
  for (int js = 1; js <= max_splits; ++js) {
    const int64_t cps = (chunks + js - 1) / js;
    if (js > 1 && cps < MIN_CHUNKS) break;
    const int parts = (int)((chunks + cps - 1) / cps);
    const int64_t gens = ((int64_t)row_blocks * parts + slots - 1) / slots;
    const double cost = (double)gens * ((double)cps + FIXED) + (parts > 1 ? image_cost * parts : 0.0);
    if (cost < best_cost * (1.0 - 1e-9)) {
      best_cost = cost;
      best = parts;
    }
  }
  return best;
}

int gp_launch_colmax(gp_ctx* ctx, const float* dV, int64_t ldv, int t, unsigned* cm, const float* dV2, int64_t ldv2,
                     unsigned* cm2, bool cleared) {
  if (!cleared) {
    hipLaunchKernelGGL(clear_words_kernel, dim3((t + 255) / 256), dim3(256), 0, ctx->stream, cm, dV2 ? cm2 : nullptr, t);
    GP_HIP(ctx, hipGetLastError());
  }
  // few workgroups: every one ends with t atomic maxima on the same t words
  int blocks = (int)((ctx->n * (int64_t)t + 8191) / 8192);
  if (blocks > 2 * ctx->num_cu) blocks = 2 * ctx->num_cu;
  if (blocks < 1) blocks = 1;
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
  const bool y = has_vec_column(t);
  const bool small = !colmax_ready && !win && t > 1 && ctx->n <= 8192 && t - (y ? 1 : 0) <= 64;
  const bool maxima = !colmax_ready && t > 1 && !small;       // a single vector is not scaled
  const bool accumulate = maxima && scratch != ctx->static_scratch;
  if (maxima) {
    if (accumulate) {
      if (ctx->colmax_dirty) {
        hipLaunchKernelGGL(clear_words_kernel, dim3((ctx->colmax_dirty + 255) / 256), dim3(256), 0, st, ctx->dColmax, nullptr, ctx->colmax_dirty);
        GP_HIP(ctx, hipGetLastError());
      }
      if (ctx->colmax_dirty < t) ctx->colmax_dirty = t;     // until the launch that clears them is on the stream
    }
    const int rc = gp_launch_colmax(ctx, dV, ldv, t, accumulate ? ctx->dColmax : (unsigned*)(w + L.off_colmax), nullptr, 0, nullptr, accumulate);
    if (rc < 0) return rc;
  }

  // operands of one column pass, chunks c0 .. c0 + chunks - 1
  auto pack = [&](int c0, int chunks, int NT, int col0, int ncols, int vc, bool first_pass) {
    const int64_t threads = (int64_t)chunks * 2 * NT * 64;
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
      hipLaunchKernelGGL(pack_small, dim3((unsigned)((col0 + 32 * NT + 7) / 8)), dim3(1024), 0, st, dV, ldv, (int)ctx->n, nchunks, NT, col0, t,
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
    int rc = pack_pass(NT, c, t - c < 32 * NT ? t - c : 32 * NT, y ? 0 : -1, true);
    if (rc < 0 || (rc = gp_rows_path(ctx, rows)) < 0) return rc;
    if (rows->path == GP_PATH_FP32) return GP_TO_FP32;
    packed = true;
  }

  const int XP = rows ? (rows->path == GP_PATH_F16X3 ? 3 : 2) : ctx->XP;
  PlanH pl = plan_h(ctx, nrows, win ? win->nchunks : 0, t, XP);
  L = scratch_layout(ctx, t, pl.JS, nrows);
  const PanelsH pn = scratch_bytes < L.total && pl.JS > 1 && !defer && !win && !rows ? plan_panels(ctx, nrows, t, XP, pl, L, scratch_bytes) : PanelsH{0, pl.JS};
  if (pn.rows) L = scratch_layout(ctx, t, 1, nrows), L.off_part = panel_images_at(L, pn.group, pl), L.total = scratch_bytes;
  if (scratch_bytes < L.total)
    return gp_fail(ctx, GP_ERR_WORKSPACE, "gp_kmv: scratch %zu < %zu bytes", scratch_bytes, L.total);
  float* part = (float*)(w + L.off_part);
  const bool split = pl.JS > 1;

  TileArgsH a;
  for (int pc = 0; pc < 3; ++pc) {
    a.XA[pc] = (const u32x4*)ctx->dXAh[pc] + (win ? (int64_t)win->chunk0 * ctx->KH * 64 : 0);
    a.XB[pc] = (const u32x4*)(rows ? rows->XBh[pc] : ctx->dXBh[pc]);
  }
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
  a.a2 = (float)(ctx->a * ctx->a);
  a.sigma2 = (float)(ctx->sigma * ctx->sigma);
  a.add_noise = add_noise;
  a.win_sel = nullptr;
  a.win_block = 0;
  a.gather = nullptr;
  a.npoints = ctx->n - first;
  a.cm_ld = 0;
  a.done = nullptr;
  a.diag_shift = 0;

  auto sum_images_of = [&](int64_t m, int width, bool add, float* out) {     // out = the sum of the images of m rows
    int blocks = (int)((m * width + 1023) / 1024);
    if (blocks > 8 * ctx->num_cu) blocks = 8 * ctx->num_cu;
    hipLaunchKernelGGL(kmv_reduce_f16_kernel, dim3(blocks), dim3(256), 0, st, (const float*)part, a.split_stride, a.JS, m, width, add ? 1 : 0,
                       out, ldo);
  };
  int vcol = y ? 0 : -1;
  int c = vcol >= 0 ? 1 : 0;
  bool first_pass = true;
  do {
    const int rem = t - c;
    const int NT = pass_tiles(rem);
    a.col0 = c;
    a.ncols = rem < 32 * NT ? rem : 32 * NT;
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
    const TileKernelH k = tile_kernel_h(ctx, nrows, XP, NT, a.vcol >= 0, FORM_PLAIN);
    if (!k.fn) return gp_fail(ctx, GP_ERR_ARG, "gp_kmv: no fp16 kernel for KH=%d", ctx->KH);
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
          a.VP = VP + (pn.group < pl.JS ? 0 : (int64_t)c0 * 4 * NT * 64);
          for (int pc = 0; pc < 3; ++pc) {
            a.XA[pc] = (const u32x4*)ctx->dXAh[pc] + (int64_t)c0 * ctx->KH * 64;
            a.XB[pc] = (const u32x4*)ctx->dXBh[pc] + (r0 / 32) * ctx->KH * 64;
          }
          a.ldo = width;
          a.split_stride = m * width;
          a.OUT = part - col;
          if (pn.group < pl.JS) pack(c0, a.nchunks, NT, a.col0, a.ncols, vc, first_pass);
        }
        const dim3 grid((unsigned)((m + k.rows_per_wg - 1) / k.rows_per_wg) * a.JS);
        const bool prof = gp_prof_begin(ctx, GP_PROF_TILE);
        hipLaunchKernelGGL(k.fn, grid, dim3(k.threads), 0, st, a);
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
  for (int c = has_vec_column(t) ? 1 : 0; c < t;) {
    const int NT = pass_tiles(t - c);
    u += nchunks * 4 * NT * 64;
    c += 32 * NT;
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
  for (int pc = 0; pc < 3; ++pc) {
    a.XA[pc] = (const u32x4*)ctx->dXAh[pc];
    a.XB[pc] = (const u32x4*)ctx->dXBh[pc];
  }
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
  a.a2 = (float)(ctx->a * ctx->a);
  a.sigma2 = 0.0f;
  a.add_noise = 0;
  a.cm_ld = pk.ld;
  a.done = pk.done;
  a.diag_shift = 0;
  const u32x4* VP = (const u32x4*)pk.VP;
  int vcol = has_vec_column(t) ? 0 : -1;
  int c = vcol >= 0 ? 1 : 0;
  do {
    const int rem = t - c, NT = pass_tiles(rem);
    a.VP = VP;
    a.col0 = c;
    a.ncols = rem < 32 * NT ? rem : 32 * NT;
    a.vcol = vcol;
    vcol = -1;
    const TileKernelH k = tile_kernel_h(ctx, nrows, ctx->XP, NT, a.vcol >= 0, gather ? FORM_GATHER : win ? FORM_WINDOW : FORM_COLUMNS);
    if (!k.fn) return gp_fail(ctx, GP_ERR_ARG, "gp_kmv: no fp16 kernel for KH=%d", ctx->KH);
    const dim3 grid((unsigned)((nrows + k.rows_per_wg - 1) / k.rows_per_wg) * pl.JS);
    const bool prof = gp_prof_begin(ctx, GP_PROF_TILE);
    hipLaunchKernelGGL(k.fn, grid, dim3(k.threads), 0, ctx->stream, a);
    GP_HIP(ctx, hipGetLastError());
    gp_prof_end(ctx, prof);
    VP += (int64_t)nchunks * 4 * NT * 64;
    c += a.ncols;
  } while (c < t);
  *images = pl.JS;
  return GP_OK;
}
