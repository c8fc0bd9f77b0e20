// Marginal-likelihood gradient estimator (paper Section 2 gradient equation with the Section 2.1
// trace estimator), split-fp16 matrix-core tile pass.  Same mathematics as the fp32 pass:
//   g_k = sum_ij w_ij (dH/dtheta_k)_ij,  w_ij = A_i . C_j,  G = w .* psi,  row sums of G Q with
//   Q = [xs, xs^2, 1], plus one vector-ALU column sum_j w_ij K_ij / a^2 for the amplitude.
// dH/dtheta_k is symmetric, so only the tiles on and above the diagonal are worked on, with the weights of both
// halves: u_ij = w_ij + w_ji.  The y column's term is symmetric by itself (v_i v_j, one FMA per pair on the vector
// ALU); a probe's becomes two, a_i z_j + z_i a_j with a = -v / (2s).  A square expanded as
// (xs_i - xs_j)^2 = xs_i^2 + xs_j^2 - 2 xs_i xs_j needs the sums over j of one row only, never those of a column, so
// half a matrix of pairs is all there is to it.
// All three contractions of a 32x32 tile of pairs run on v_mfma_f32_32x32x16_f16 with operands split
// into two fp16 pieces rounded to nearest (three products per fp32 product, fp32 accumulation):
//   1. S[j][i]  = XA_j . XB_i        the distance chain, on operands of its own (the K V pass packs its slots otherwise: dist_f16.h)
//   2. U'[j][i] = C'_j . A'_i        the probes' part of u; every column-side component is scaled to max in [2^6, 2^7),
//                                    the row side carries the inverse scales and a global power of two alpha chosen so
//                                    that |U' psi| < 2^15 (from the sum over the components of max|row| max|column| >= |u_ij|)
//   3. OUT_i   += G'[i][j] Q'_j      G' = U' psi split on the VALU, Q' = 2^qshift Q pre-split
// The epilogue removes alpha and 2^qshift.  K and u are never stored.
// Matrix instructions per pair of mirrored tiles, d = 26, t = 65: 42 instead of 66 (6 + 24 + 12 against twice 6 + 15 + 12), and half
// the vector work; the matrix core and the vector port together bound it (56 % and 39 % of the cycles at n = 43945, d = 26, t = 65, at 1.89 GHz).
// A gradient, all pairs -> half: n = 16384, d = 26, t = 65 (Matern) 320 -> 234 us, d = 60 692 -> 471 us; n = 43945, d = 20, t = 17
// 1468 -> 832 us; n = 140000, d = 3, t = 65 (SE) 14.0 -> 9.3 ms.  Error against 64 bits, V a solution:
// n = 8192, d = 26, t = 65 1.05e-6 -> 2.3e-7; n = 8000, d = 9, t = 33 1.8e-6 -> 3.3e-7.
#include <cstdlib>

#include "gpws_internal.h"
#include "split_f16.h"

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

namespace {

constexpr int C_TOP = 7;                    // max |C'_c| in [2^6, 2^7)
constexpr int U_TOP = 13;                   // alpha |u_ij| <= 2^13, so |U' psi| <= 3 2^13 < 2^15
constexpr int PROBE_BLOCK = 80;             // most probe columns per tile pass (two times 5 k-steps of 16)
constexpr int SCALE_THREADS = 128;          // of the kernel that scales them, a thread per probe
static_assert(PROBE_BLOCK <= SCALE_THREADS, "a thread per probe");
// Rows of all images together, where they are more than one: 407 MB at d = 96.  Every row in pieces, n = 100000 would take 850000.
// With half as many n = 43945 .. 125000 takes up to 10 % longer (d = 96, t = 65, n = 100000 33.6 -> 36.9 ms), with these 3 % at most.
constexpr int64_t IMAGE_ROWS = 1 << 19;
// the same, and probes per pass, of a context whose device did not have the memory
constexpr int64_t IMAGE_ROWS_TIGHT = 1 << 17;
constexpr int PROBE_BLOCK_TIGHT = 32;
// A workgroup's waves, 32 rows each.  Two workgroups of four run past each other's barriers; from six k-steps of probes on a chunk's
// operands are so many that eight waves should share them.  n = 16384, d = 26: t = 65 (8 k-steps) 250 us a gradient with four
// waves, 234 with eight; n = 43945, d = 20, t = 17 (2 k-steps) 839 and 915.  Not while there are too few rows for that: up to about
// five workgroups of four waves to four compute units a gradient is the time of its chains, and those are shorter in a kernel that
// may have 512 registers to a wave: of the eight-wave kernels with many distance operands, 37 of 144 keep some in scratch memory
// (4 XP KH + 8 KT + 16 NT above 140).  Four and eight waves, t = 65: n = 2048, d = 60 86 and 90 us, d = 96 124 and 144,
// with three pieces 135 and 186; n = 3500, d = 60 115 and 100, d = 96 191 and 170; n = 43945, d = 96 8.1 and 6.6 ms.
int grad_waves(int KT, int64_t chunks, int cus) {
  return KT >= 6 && chunks * (chunks + 4) / 32 > cus + cus / 4 ? 8 : 4;      // workgroups of four waves and four chunks
}

struct GradArgsH {
  const u32x4* XA[3];     // column-side distance pieces [(chunk*KH + kh)*64 + lane]
  const u32x4* XB[3];     // row-side distance pieces
  const u32x4* CA;        // C' images, column side: [((chunk*2 + part)*KT + kt)*64 + lane]
  const u32x4* AB;        // A' images, row side, same indexing by sub-tile
  const u32x4* QP;        // Q' images of this column pass: [(((chunk*2 + mh)*NT + nt)*2 + part)*64 + lane]
  const float* VY;        // the y column, zero from n up to the end of its chunk; all zero in later blocks of probes
  const int* scales;      // [0] = exponent of alpha
  float* OUT;             // [workgroup][32 W][ldo]: an image per piece of a row, of the rows that have the piece
  int64_t ldo;
  int64_t n;
  int nchunks;
  int col0, ncols;        // Q columns of this pass
  int vcol;               // output column of sum_j u_ij K_ij / a^2, or -1
  int cps;                // most chunks one workgroup takes of its rows' columns
  int qshift;             // Q' = 2^qshift Q
  int slot_kh, slot_h, slot_e;   // where the row-side operand carries the SE exponent shift, or -1
};

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// A workgroup takes piece js of the columns of row block rb, from the row block's first chunk on.  Only pieces that are there
// have a workgroup: with the others returning at once, as many pieces as compute units did not run side by side, the hardware
// dealing workgroups to the eight dies in turn (n = 16384, d = 26, t = 65: compute units busy 46 % of the launch).
template <int KIND, int KH, int XP, int KT, int NT, int W>
__global__ __launch_bounds__(64 * W) void grad_tile_f16_kernel(GradArgsH p) {
  constexpr int XA_G = XP * KH;          // groups of 64 16-byte units per stage
  constexpr int C_G = 2 * KT;
  constexpr int Q_G = 4 * NT;
  constexpr int G = XA_G + C_G + Q_G;
  constexpr int C_OFF = XA_G * 64;
  constexpr int Q_OFF = (XA_G + C_G) * 64;
  constexpr int Y_OFF = G * 64;          // then the chunk's 32 y values: 8 units
  constexpr int STAGE = G * 64 + 8;
  constexpr int NS = 3 * STAGE <= 5120 ? 3 : 2;    // LDS ring (two workgroups share 160 KB): chunks up to ch + NS - 1 in flight while ch is consumed
  constexpr int DEPTH = NS - 1;
  constexpr int LPW = (G + W - 1) / W;   // group loads per wave per chunk
  constexpr int LPC = LPW + 1;           // + the y values (every wave fetches the same 128 bytes to the same place)
  static_assert(DEPTH * LPC < 64, "vmcnt cannot express the pipeline depth");
  __shared__ u32x4 lds[NS][STAGE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction: lets the compiler branch on it
  const int h = lane >> 5;
  const int li = lane & 31;
  int js = 0, rb = blockIdx.x;
  for (int rows; rb >= (rows = gp_grad_rows_with_piece(js, p.nchunks, p.cps, W)); ++js) rb -= rows;
  const int sub0 = rb * W + wave;
  // The workgroup's column range [r_begin, r_end) is walked in segments [c_begin, c_end) of at most
  // GP_FLUSH_CHUNKS chunks; the accumulators are added into OUT after each segment (see flush below).
  const int len = p.nchunks - rb * W;
  const int pieces = (len + p.cps - 1) / p.cps;
  const int per = (len + pieces - 1) / pieces;
  const int r_begin = rb * W + js * per;
  const int r_end = min(p.nchunks, r_begin + per);
  int c_begin = r_begin;
  int c_end = min(r_end, c_begin + GP_FLUSH_CHUNKS);

  // row-side operands stay in registers for the whole pass
  f16x8 xb[XP][KH], abh[KT], abl[KT];
#pragma unroll
  for (int pc = 0; pc < XP; ++pc)
#pragma unroll
    for (int kh = 0; kh < KH; ++kh) xb[pc][kh] = as_f16x8(p.XB[pc][((int64_t)sub0 * KH + kh) * 64 + lane]);
  if (KIND == GP_SE_ARD) {
    // the K V pass carries phi as 2^15 phi through one extra operand component; psi is used unshifted here
#pragma unroll
    for (int kh = 0; kh < KH; ++kh)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (kh == p.slot_kh && e == p.slot_e && h == p.slot_h) xb[0][kh][e] = (_Float16)0.0f;
  }
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    abh[kt] = as_f16x8(p.AB[((int64_t)(sub0 * 2 + 0) * KT + kt) * 64 + lane]);
    abl[kt] = as_f16x8(p.AB[((int64_t)(sub0 * 2 + 1) * KT + kt) * 64 + lane]);
  }

  f32x16 acc[NT];
  float accv = 0.0f;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nt][r] = 0.0f;

  // global -> LDS staging without registers (global_load_lds_dwordx4), DEPTH chunks ahead; every wave
  // issues LPW loads per chunk (surplus slots repeat the last group) so one vmcnt value per wave tells
  // when its share of a chunk has landed, and the barrier that follows publishes the whole chunk.
  const u32x4* g_src[LPW];
  int g_stride[LPW];
  unsigned g_lds[LPW];
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)&lds[0][0];
#pragma unroll
  for (int x = 0; x < LPW; ++x) {
    const int g = min(wave + W * x, G - 1);
    if (g < XA_G) {
      g_src[x] = p.XA[g / KH] + (g % KH) * 64 + lane;
      g_stride[x] = KH * 64;
    } else if (g < XA_G + C_G) {
      g_src[x] = p.CA + (g - XA_G) * 64 + lane;
      g_stride[x] = C_G * 64;
    } else {
      g_src[x] = p.QP + (g - XA_G - C_G) * 64 + lane;
      g_stride[x] = Q_G * 64;
    }
    g_lds[x] = __builtin_amdgcn_readfirstlane(lds_base + 16u * (unsigned)(g * 64));
  }
  const unsigned vy_lds = lds_base + 16u * (unsigned)Y_OFF;
  // inline assembly keeps the ordering explicit (s_waitcnt vmcnt(N) + barrier) instead of the
  // compiler's conservative drain of all LDS-DMA loads at every barrier
  auto dma16 = [](const u32x4* src, unsigned lds_addr) {
    // m0 carries the LDS address of the load; it is declared clobbered, so the compiler keeps nothing in it
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds_addr) : "memory", "m0");
  };
  auto issue_chunk = [&](int ch_target) {
    const int ch = min(ch_target, c_end - 1);           // past the end: harmless reload of the last chunk
    const unsigned stage_off = (unsigned)((ch_target - c_begin) % NS) * (unsigned)(STAGE * 16);
#pragma unroll
    for (int x = 0; x < LPW; ++x) dma16(g_src[x] + (int64_t)ch * g_stride[x], __builtin_amdgcn_readfirstlane(g_lds[x] + stage_off));
    if (lane < 8) dma16(reinterpret_cast<const u32x4*>(p.VY + (int64_t)ch * 32) + lane, __builtin_amdgcn_readfirstlane(vy_lds + stage_off));
  };
  constexpr int WAIT_N = (DEPTH - 1) * LPC;   // all but the newest DEPTH - 1 chunks have landed

  // Writes the accumulators to OUT (first: stores; later: adds to what is there) without alpha and
  // 2^qshift, and clears them.  Doing so after every segment keeps the chains of fp32 partial sums
  // short; the same threads read and write the same elements, in a fixed order.
  // The weights of odd row sub-tiles are packed with their sign flipped (grad_pack_ac_f16_kernel) and the
  // flip is undone here: what is left of the one-sided rounding described at the weight chain below
  // then enters the sums over rows with alternating sign instead of adding up.
  const int alpha_exp = p.scales[0];
  const float row_sign = (sub0 & 1) ? -1.0f : 1.0f;
  const float oscale = row_sign * (KIND == GP_SE_ARD ? 1.0f : 3.0f) * ldexpf(1.0f, -alpha_exp - p.qshift);   // psi = 3 exp(-u) for Matern: the 3 is applied here
  const float vscale = row_sign * ldexpf(1.0f, -alpha_exp);
  const float yi = row_sign * ldexpf(sub0 < p.nchunks ? p.VY[(int64_t)sub0 * 32 + li] : 0.0f, alpha_exp);
  float* out = p.OUT + (int64_t)(blockIdx.x - rb) * (32 * W) * p.ldo;      // this piece's image
  auto flush = [&](bool first) {
    // an opaque zero keeps the address arithmetic of the flush inside it: hoisted out of the segment
    // loop it would hold dozens of registers across the main loop
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    const int64_t ibase = (int64_t)sub0 * 32 + zero;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int c = li + 32 * nt;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t i = ibase + 8 * (r >> 2) + 4 * h + (r & 3);
        if (i < p.n && c < p.ncols) {
          float v = oscale * acc[nt][r];
          if (!first) v += out[i * p.ldo + p.col0 + c];
          out[i * p.ldo + p.col0 + c] = v;
        }
        acc[nt][r] = 0.0f;
      }
    }
    if (p.vcol >= 0) {
      const float tot = accv + __shfl_xor(accv, 32);
      const int64_t i = ibase + li;
      if (h == 0 && i < p.n) {
        float v = vscale * tot;
        if (!first) v += out[i * p.ldo + p.vcol];
        out[i * p.ldo + p.vcol] = v;
      }
      accv = 0.0f;
    }
  };

  auto chunk = [&](int ch, const u32x4* s) {
    f32x16 S, U;
#pragma unroll
    for (int r = 0; r < 16; ++r) { S[r] = 0.0f; U[r] = 0.0f; }
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
    // Per k-step the hi*hi products first, on purpose.  This matrix instruction rounds to nearest when
    // its accumulator input is the largest addend, but an accumulator input smaller than the products is
    // cut off below half a unit in the last place of the result toward minus infinity (measured on
    // MI355X).  Small cross terms summed first and the hi*hi products added on top of them would give
    // every weight a bias of about -2^-25 of its size of one sign, which the sum over all pairs does not average
    // out while the terms themselves cancel (V nearly orthogonal to K's large eigenvectors, as after a solve).
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const f16x8 ch_ = as_f16x8(s[C_OFF + (0 * KT + kt) * 64 + lane]);
      const f16x8 cl_ = as_f16x8(s[C_OFF + (1 * KT + kt) * 64 + lane]);
      U = __builtin_amdgcn_mfma_f32_32x32x16_f16(ch_, abh[kt], U, 0, 0, 0);
      U = __builtin_amdgcn_mfma_f32_32x32x16_f16(ch_, abl[kt], U, 0, 0, 0);
      U = __builtin_amdgcn_mfma_f32_32x32x16_f16(cl_, abh[kt], U, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 yj = __builtin_bit_cast(f32x4, s[Y_OFF + 2 * q + h]);
#pragma unroll
      for (int e = 0; e < 4; ++e) U[4 * q + e] = fmaf(yi, yj[e], U[4 * q + e]);
    }
    if (ch == sub0) {   // the tile on the diagonal holds both halves already; the pair (i, i): r^2 = 0 exactly
      asm volatile("" ::: "memory");   // keeps this a real (wave-uniform) branch instead of selects on every chunk
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        U[r] *= 0.5f;
        if (8 * (r >> 2) + 4 * h + (r & 3) == li) S[r] = 0.0f;
      }
    }

#pragma unroll
    for (int mh = 0; mh < 2; ++mh) {
      u32x4 gh, gl;
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        float g[2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          const int r = 8 * mh + 2 * e2 + z;
          float psi, kval;
          if (KIND == GP_SE_ARD) {
            psi = __builtin_amdgcn_exp2f(S[r]);                 // S = -log2(e)/2 r^2
            kval = psi;
          } else {
            // S = 3 r^2; rounding-level negatives are mirrored (free source modifier), (i, i) is exactly 0
            const float u = __builtin_amdgcn_sqrtf(__builtin_fabsf(S[r]));
            psi = __builtin_amdgcn_exp2f(-LOG2E * u);
            kval = fmaf(u, psi, psi);
          }
          g[z] = U[r] * psi;
          accv = fmaf(U[r], kval, accv);
        }
        unsigned hi, lo;
        split_pair(g[0], g[1], hi, lo);
        gh[e2] = hi;
        gl[e2] = lo;
      }
      const f16x8 ah = as_f16x8(gh), al = as_f16x8(gl);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const f16x8 bh = as_f16x8(s[Q_OFF + ((mh * NT + nt) * 2 + 0) * 64 + lane]);
        const f16x8 bl = as_f16x8(s[Q_OFF + ((mh * NT + nt) * 2 + 1) * 64 + lane]);
        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, acc[nt], 0, 0, 0);
        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, acc[nt], 0, 0, 0);
        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, acc[nt], 0, 0, 0);
      }
    }
  };

  // The row operands are waited for here, where the compiler sees it: it would otherwise wait for them at their first use,
  // inside the loop, and there drain the ring's loads too, chunk after chunk.
  __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
  bool first = true;
  for (;;) {
#pragma unroll
    for (int d0 = 0; d0 < DEPTH; ++d0) issue_chunk(c_begin + d0);
    for (int ch = c_begin; ch < c_end; ++ch) {
      asm volatile("s_waitcnt vmcnt(%0)" : : "n"(WAIT_N) : "memory");
      __syncthreads();              // chunk ch is complete in LDS; every wave is done with chunk ch - 1
      issue_chunk(ch + DEPTH);      // refills the stage chunk ch - 1 occupied
      if (ch >= sub0) chunk(ch, lds[(ch - c_begin) % NS]);     // the first chunks of a row block lie below the diagonal for its later waves
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

// exponent e with m = f 2^e, f in [0.5, 1), for a positive finite m; of a column of zeros one that takes the other side's
// values to zero too (they are scaled by 2^(alpha + e - C_TOP), alpha <= 113): nothing bounds them where their product is no part of the
// bound alpha is chosen from, and an overflow to infinity would meet the zeros.  Infinities and NaN stay what they are.
constexpr int ZERO_EXP = -400;
__device__ __forceinline__ int exponent_of(float m) {
  if (!(m > 0.0f)) return ZERO_EXP;
  if (!(m < INFINITY)) return 0;
  int e;
  (void)frexpf(m, &e);
  return e;
}

// scales of one block of probe columns [c0, c0 + sb): scales[0] = exponent of alpha, scales[1 + m] = exponent e of
// max |z_m| in [2^(e - 1), 2^e), scales[1 + PROBE_BLOCK + m] = the same of the weighted solutions a_m = probe_w v_m.
// with_y: the y column's weights are in the bound too.  One workgroup, fixed-order sum.
__global__ __launch_bounds__(SCALE_THREADS) void grad_scales_kernel(const unsigned* __restrict__ cmV, const unsigned* __restrict__ cmB,
                                                                  int c0, int sb, int with_y, float half_w, float probe_w,
                                                                  int* __restrict__ scales) {
  __shared__ float bound[SCALE_THREADS];
  const int m = threadIdx.x;
  float b = 0.0f;
  if (m < sb) {
    const float maxA = fabsf(probe_w) * __uint_as_float(cmV[c0 + m]);
    const float maxZ = __uint_as_float(cmB[c0 + m]);
    scales[1 + m] = exponent_of(maxZ);
    scales[1 + PROBE_BLOCK + m] = exponent_of(maxA);
    b = 2.0f * maxA * maxZ;
  }
  bound[m] = b;
  __syncthreads();
  if (m == 0) {
    const float maxY = __uint_as_float(cmV[0]);
    float ub = with_y ? 2.0f * half_w * maxY * maxY : 0.0f;
    for (int k = 0; k < sb; ++k) ub += bound[k];
    // |u_ij| <= ub <= 2^e, so alpha = 2^(U_TOP - e) keeps alpha |u_ij| <= 2^U_TOP; past 2^100 either way its inverse would leave fp32
    scales[0] = (ub > 0.0f && ub < 3.0e38f) ? U_TOP - min(max(exponent_of(ub), -100), 100) : 0;
  }
}

// C' (column side) and A' (row side) images of probe columns [c0, c0 + sb), one thread per (chunk, k-step of 16 probes,
// lane): k-step kt holds z on the column side and a on the row side, k-step KTH + kt the other way round.
// VY: the y column (with_y) or zeros.
__global__ __launch_bounds__(256) void grad_pack_ac_f16_kernel(const float* __restrict__ V, int64_t ldv,
                                                               const float* __restrict__ B, int64_t ldb, int64_t n,
                                                               int64_t nchunks_pad, int c0, int sb, int KTH, int with_y,
                                                               float probe_w, const int* __restrict__ scales,
                                                               u32x4* __restrict__ CA, u32x4* __restrict__ AB,
                                                               float* __restrict__ VY) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (gid < nchunks_pad * 32) VY[gid] = with_y && gid < n ? V[gid * ldv] : 0.0f;
  if (gid >= nchunks_pad * KTH * 64) return;
  const int lane = (int)(gid & 63);
  const int kt = (int)((gid >> 6) % KTH);
  const int64_t chunk = (gid >> 6) / KTH;
  const int64_t row = chunk * 32 + (lane & 31);
  const int alpha_exp = scales[0];
  u32x4 im[8];     // z and a as column side, a and z as row side: high and low pieces
#pragma unroll
  for (int e2 = 0; e2 < 4; ++e2) {
    float x[4][2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int m = 16 * kt + 8 * (lane >> 5) + 2 * e2 + q;
      for (int k = 0; k < 4; ++k) x[k][q] = 0.0f;
      if (row < n && m < sb) {
        const int ez = scales[1 + m], ea = scales[1 + PROBE_BLOCK + m];
        const float a = probe_w * V[row * ldv + c0 + m], z = B[row * ldb + c0 + m];
        x[0][q] = ldexpf(z, C_TOP - ez);
        x[1][q] = ldexpf(a, C_TOP - ea);
        x[2][q] = ldexpf(a, alpha_exp + ez - C_TOP);
        x[3][q] = ldexpf(z, alpha_exp + ea - C_TOP);
        if (chunk & 1) {   // undone by the tile kernel's epilogue (row_sign)
          x[2][q] = -x[2][q];
          x[3][q] = -x[3][q];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      unsigned hi, lo;
      split_pair(x[k][0], x[k][1], hi, lo);
      im[2 * k][e2] = hi;
      im[2 * k + 1][e2] = lo;
    }
  }
  const int KT = 2 * KTH;
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    const int64_t u = ((chunk * 2 + part) * KT + kt) * 64 + lane;
    CA[u] = im[part];
    CA[u + KTH * 64] = im[2 + part];
    AB[u] = im[4 + part];
    AB[u + KTH * 64] = im[6 + part];
  }
}

// Q' images of Q columns [col0, col0 + ncols), Q = [xs (d), xs^2 (d), 1]; one thread per (chunk, mh, nt, lane).
// Element e of lane l is row 32 chunk + 16 mh + 8 (e/4) + 4 (l/32) + e%4 (the register order of the
// accumulator layout that G' comes in), column col0 + 32 nt + l%32.
__global__ __launch_bounds__(256) void grad_pack_q_f16_kernel(const float* __restrict__ Xs, int64_t n, int d,
                                                              int nchunks, int NT, int col0, int ncols, int qshift,
                                                              u32x4* __restrict__ QP) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= (int64_t)nchunks * 2 * NT * 64) return;
  const int lane = (int)(gid & 63);
  int64_t q = gid >> 6;
  const int nt = (int)(q % NT); q /= NT;
  const int mh = (int)(q & 1);
  const int64_t chunk = q >> 1;
  const int hh = lane >> 5;
  const int cc = 32 * nt + (lane & 31);
  const int col = col0 + cc;
  const bool cok = cc < ncols;
  u32x4 hi, lo;
#pragma unroll
  for (int e2 = 0; e2 < 4; ++e2) {
    float f[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      const int e = 2 * e2 + z;
      const int64_t j = chunk * 32 + 16 * mh + 8 * (e >> 2) + 4 * hh + (e & 3);
      float v = 0.0f;
      if (cok && j < n) {
        if (col < d) v = Xs[j * d + col];
        else if (col < 2 * d) { const float x = Xs[j * d + col - d]; v = x * x; }
        else v = 1.0f;
        v = ldexpf(v, qshift);
      }
      f[z] = v;
    }
    unsigned fh, fl;
    split_pair(f[0], f[1], fh, fl);
    hi[e2] = fh;
    lo[e2] = fl;
  }
  u32x4* dst = QP + ((chunk * 2 + mh) * NT + nt) * 2 * 64;
  dst[lane] = hi;
  dst[64 + lane] = lo;
}

typedef void (*gradh_fn)(GradArgsH);

template <int KIND, int KH, int XP, int KT>
gradh_fn pick_nt_w(int NT, int W) {
  if constexpr (KT >= 6) {
    if (W == 8) return NT == 1 ? grad_tile_f16_kernel<KIND, KH, XP, KT, 1, 8> : grad_tile_f16_kernel<KIND, KH, XP, KT, 2, 8>;
  }
  return NT == 1 ? grad_tile_f16_kernel<KIND, KH, XP, KT, 1, 4> : grad_tile_f16_kernel<KIND, KH, XP, KT, 2, 4>;
}

template <int KIND, int KH, int XP>
gradh_fn pick_kt(int KT, int NT, int W) {
  switch (KT) {
    case 2: return pick_nt_w<KIND, KH, XP, 2>(NT, W);
    case 4: return pick_nt_w<KIND, KH, XP, 4>(NT, W);
    case 6: return pick_nt_w<KIND, KH, XP, 6>(NT, W);
    case 8: return pick_nt_w<KIND, KH, XP, 8>(NT, W);
    case 10: return pick_nt_w<KIND, KH, XP, 10>(NT, W);
  }
  return nullptr;
}

template <int KIND, int XP>
gradh_fn pick_kh(int KH, int KT, int NT, int W) {
  switch (KH) {
    case 1: return pick_kt<KIND, 1, XP>(KT, NT, W);
    case 2: return pick_kt<KIND, 2, XP>(KT, NT, W);
    case 3: return pick_kt<KIND, 3, XP>(KT, NT, W);
    case 4: return pick_kt<KIND, 4, XP>(KT, NT, W);
    case 6: return pick_kt<KIND, 6, XP>(KT, NT, W);
    case 8: return pick_kt<KIND, 8, XP>(KT, NT, W);
  }
  return nullptr;
}

gradh_fn pick_gradh(int kind, int KH, int XP, int KT, int NT, int W) {
  if (kind == GP_SE_ARD) return XP == 2 ? pick_kh<GP_SE_ARD, 2>(KH, KT, NT, W) : pick_kh<GP_SE_ARD, 3>(KH, KT, NT, W);
  return XP == 2 ? pick_kh<GP_MATERN32_ARD, 2>(KH, KT, NT, W) : pick_kh<GP_MATERN32_ARD, 3>(KH, KT, NT, W);
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

int grad_probe_steps(int s) { return s > 16 ? (s + 15) / 16 : 1; }

// Probe columns of every block but the last: as few blocks as there can be, of about one size in whole k-steps.  A block works out
// distances and kernel values again, so a last one of a few probes is dear: with blocks of 64, t = 80 took n = 16384, d = 26 385 us, now
// 261; n = 43945, d = 96 11.5 ms, now 7.4; n = 2048, d = 60 137 us, now 93.
int grad_probe_block(int s, int most) {
  const int blocks = s > 0 ? (s + most - 1) / most : 1;
  return 16 * ((grad_probe_steps(s) + blocks - 1) / blocks);
}

// The work of one block of probes: workgroups of W waves, most chunks one of them takes, pieces of the longest rows (the first
// ones), all workgroups.  `slots` workgroups are taken to run side by side, one of eight waves or two of four to a compute unit.
// Not all kernels of four waves do: those with KH = 1, KT = 2 hold three (planned so, n = 16384, d = 3, t = 17 would take 125 us instead
// of 138), those with three pieces of many dimensions one (n = 4000, d = 96, t = 33 172 instead of 211; from n = 16384 on nothing changes).
struct GradPlan {
  int W, cps, pieces, workgroups;
  int64_t image_rows() const { return (int64_t)workgroups * 32 * W; }
};
GradPlan grad_plan(int KT, int chunks, int cus, int64_t max_rows) {
  GradPlan pl;
  pl.W = grad_waves(KT, chunks, cus);
  const int slots = cus * 8 / pl.W, row_blocks = (chunks + pl.W - 1) / pl.W;
  const int64_t work = (int64_t)row_blocks * chunks - (int64_t)pl.W * row_blocks * (row_blocks - 1) / 2;   // chunks of all rows
  // Rows from long to short fill two generations and more by themselves; fewer are cut into pieces, each an image to write
  // and sum.  Pieces are of about one length, so beyond one generation the time lies between what a slot has to do on the
  // average and whole generations.  The chip waits while this runs: workgroups are counted by piece, at most 64 terms, each a shift
  // (gp_grad_rows_with_piece); counting them by row block, a division
  // each, took 10 us at n = 16384, t = 65 and 48 us at n = 43945, t = 17, and twice that with a second plan for the same block; now 3 us.
  constexpr double FIXED = 6.0;       // prologue and flush of a workgroup, in chunks
  double best = 1e300;
  for (int pieces = 1; pieces <= (row_blocks >= 2 * slots ? 1 : 64); ++pieces) {
    const int cps = (chunks + pieces - 1) / pieces;
    if (pieces > 1 && cps < 4) break;
    int64_t all = 0;
    for (int js = 0; (int64_t)js * cps < chunks; ++js) all += gp_grad_rows_with_piece(js, chunks, cps, pl.W);
    if (pieces > 1 && all * 32 * pl.W > max_rows) break;
    double cost = cps + FIXED;
    if (all > slots) {
      const double mean = ((double)work + FIXED * all) / slots, gens = (double)((all + slots - 1) / slots);
      const double c = 0.5 * (mean + 0.5 * cps) + 0.5 * gens * ((double)work / all + FIXED);
      if (c > cost) cost = c;
    }
    cost += 0.25 * pieces;
    if (cost < best) {
      best = cost;
      pl.cps = cps;
    }
  }
  pl.pieces = (chunks + pl.cps - 1) / pl.cps;
  pl.workgroups = 0;
  for (int js = 0; js < pl.pieces; ++js) pl.workgroups += gp_grad_rows_with_piece(js, chunks, pl.cps, pl.W);
  return pl;
}

}  // namespace

int gp_grad_run_f16(gp_ctx* ctx, const float* dV, int64_t ldv, const float* dB, int64_t ldb, int t,
                    double* h_grad) {
  const int d = ctx->d;
  const int64_t n = ctx->n;
  const int nq = 2 * d + 2;         // Q columns (2d+1) + the vector-ALU column
  const int ldq = 2 * d + 1;
  const int s = t - 1;
  const float half_w = 0.5f;
  const float probe_w = s > 0 ? (float)(-0.5 / (double)s) : 0.0f;

  const int64_t chunks = (n + 31) / 32;
  const int64_t chunks_pad = ctx->n_pad / 32;
  // workgroups of the fp64 reduction: one step of 256 / (d + 2) rows each when n allows, so that
  // enough loads are in flight (the kernel is latency-bound at small n)
  int G;
  {
    const int per_step = 256 / (d + 2 < 256 ? d + 2 : 256);
    const int64_t want = (n + per_step - 1) / per_step;
    G = (int)(want < 8 * ctx->num_cu ? want : 8 * ctx->num_cu);
    if (G < 1) G = 1;
  }
  const size_t q_bytes = align_up((size_t)chunks * 2 * 2 * 2 * 64 * 16, 256);
  const size_t part_bytes = align_up((size_t)G * (d + 2) * sizeof(double), 256);
  const size_t acc_bytes = align_up((size_t)(d + 2) * sizeof(double), 256);
  const size_t cm_bytes = align_up((size_t)t * sizeof(unsigned), 256);
  const size_t sc_bytes = align_up((size_t)(1 + 2 * PROBE_BLOCK) * sizeof(int), 256);
  const size_t vy_bytes = align_up((size_t)chunks_pad * 32 * sizeof(float), 256);
  // Where the device does not have the memory, operands of fewer probes and fewer images do, from then on: a call's result does
  // not depend on what else is allocated while it runs.
  int block, first_block, rc;
  GradPlan first_plan, last_plan;
  size_t op_bytes, out_bytes;
  for (;;) {
    block = grad_probe_block(s, ctx->grad_tight ? PROBE_BLOCK_TIGHT : PROBE_BLOCK);
    first_block = s < block ? s : block;
    const int last_block = s > block ? (s - 1) % block + 1 : first_block;
    const int KTmax = 2 * grad_probe_steps(first_block);
    const int64_t max_rows = ctx->grad_tight ? IMAGE_ROWS_TIGHT : IMAGE_ROWS;
    first_plan = grad_plan(KTmax, (int)chunks, ctx->num_cu, max_rows);
    last_plan = last_block == first_block ? first_plan : grad_plan(2 * grad_probe_steps(last_block), (int)chunks, ctx->num_cu, max_rows);
    const int64_t rows = first_plan.image_rows() > last_plan.image_rows() ? first_plan.image_rows() : last_plan.image_rows();
    op_bytes = align_up((size_t)chunks_pad * 2 * KTmax * 64 * 16, 256);
    out_bytes = align_up((size_t)rows * nq * sizeof(float), 256);
    rc = gp_ensure_scratch(ctx, 2 * op_bytes + q_bytes + out_bytes + part_bytes + acc_bytes + 2 * cm_bytes + sc_bytes + vy_bytes);
    if (rc >= 0) break;
    if (ctx->grad_tight) return rc;
    (void)hipGetLastError();      // of the failed allocation
    ctx->grad_tight = true;
  }
  char* w = (char*)ctx->dScratch;
  u32x4* CA = (u32x4*)w; w += op_bytes;
  u32x4* AB = (u32x4*)w; w += op_bytes;
  u32x4* QP = (u32x4*)w; w += q_bytes;
  float* OUT = (float*)w; w += out_bytes;
  double* part = (double*)w; w += part_bytes;
  double* acc = (double*)w; w += acc_bytes;
  unsigned* cmV = (unsigned*)w; w += cm_bytes;
  unsigned* cmB = (unsigned*)w; w += cm_bytes;
  int* scales = (int*)w; w += sc_bytes;
  float* VY = (float*)w;
  hipStream_t st = ctx->stream;

  GP_HIP(ctx, hipMemsetAsync(acc, 0, acc_bytes + 2 * cm_bytes, st));   // acc, cmV, cmB lie back to back
  rc = gp_launch_colmax(ctx, dV, ldv, t, cmV, dB, ldb, cmB, true);
  if (rc < 0) return rc;

  // Q' = 2^qshift Q with max |Q| = max(1, max_i |xs_i|^2) kept below 2^15
  int qshift = 8;
  {
    int e = 0;
    (void)frexpf(ctx->max_norm > 1.0f ? ctx->max_norm : 1.0f, &e);   // max <= 2^e
    if (14 - e < qshift) qshift = 14 - e;
    if (qshift < 0) qshift = 0;
  }

  GradArgsH a;
  for (int pc = 0; pc < 3; ++pc) {
    a.XA[pc] = (const u32x4*)ctx->dXAh[pc];
    a.XB[pc] = (const u32x4*)ctx->dXBh[pc];
  }
  a.CA = CA;
  a.AB = AB;
  a.QP = QP;
  a.VY = VY;
  a.scales = scales;
  a.OUT = OUT;
  a.ldo = nq;
  a.n = n;
  a.nchunks = (int)chunks;
  a.qshift = qshift;
  a.slot_kh = a.slot_h = a.slot_e = -1;
  if (ctx->kernel == GP_SE_ARD) {
    const int k = d + 2;
    a.slot_kh = k / 16;
    a.slot_h = (k % 16) / 8;
    a.slot_e = k % 8;
  }
  for (int c0 = 1; c0 == 1 || c0 < t; c0 += block) {
    const int sb = t - c0 < block ? t - c0 : block;       // 0 when y is the only column
    const int KTH = grad_probe_steps(sb), KT = 2 * KTH, with_y = c0 == 1;
    const GradPlan& pl = sb == first_block ? first_plan : last_plan;
    a.cps = pl.cps;
    hipLaunchKernelGGL(grad_scales_kernel, dim3(1), dim3(SCALE_THREADS), 0, st, (const unsigned*)cmV, (const unsigned*)cmB, c0, sb, with_y,
                       half_w, probe_w, scales);
    GP_HIP(ctx, hipGetLastError());
    {
      const int64_t units = chunks_pad * KTH * 64;
      hipLaunchKernelGGL(grad_pack_ac_f16_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st, dV, ldv, dB, ldb,
                         n, chunks_pad, c0, sb, KTH, with_y, probe_w, (const int*)scales, CA, AB, VY);
      GP_HIP(ctx, hipGetLastError());
    }
    int vcol = nq - 1;
    for (int c = 0; c < ldq;) {
      const int rem = ldq - c;
      const int NT = rem > 32 ? 2 : 1;
      a.col0 = c;
      a.ncols = rem < 32 * NT ? rem : 32 * NT;
      a.vcol = vcol;
      vcol = -1;
      {
        const int64_t units = chunks * 2 * NT * 64;
        hipLaunchKernelGGL(grad_pack_q_f16_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st,
                           (const float*)ctx->dXs, n, d, (int)chunks, NT, a.col0, a.ncols, qshift, QP);
        GP_HIP(ctx, hipGetLastError());
      }
      gradh_fn fn = pick_gradh(ctx->kernel, ctx->KH, ctx->XP, KT, NT, pl.W);
      if (!fn) return gp_fail(ctx, GP_ERR_ARG, "gp_mll_grad: no fp16 kernel for KH=%d", ctx->KH);
      const bool pr = gp_prof_begin(ctx, GP_PROF_GRAD_TILE);
      hipLaunchKernelGGL(fn, dim3(pl.workgroups), dim3(64 * pl.W), 0, st, a);
      gp_prof_end(ctx, pr);
      GP_HIP(ctx, hipGetLastError());
      c += a.ncols;
    }
    rc = gp_grad_reduce_launch(ctx, OUT, pl.pieces, nq, dV, ldv, dB, ldb, t, half_w, probe_w, with_y, part, G, acc,
                               pl.W, pl.cps);
    if (rc < 0) return rc;
  }

  double* hacc = (double*)ctx->hPinned;
  GP_HIP(ctx, hipMemcpyAsync(hacc, acc, sizeof(double) * (d + 2), hipMemcpyDeviceToHost, st));
  GP_HIP(ctx, hipStreamSynchronize(st));
  const double a2 = ctx->a * ctx->a;
  for (int k = 0; k < d; ++k) h_grad[k] = a2 / ctx->ell[k] * hacc[k];
  h_grad[d] = 2.0 * ctx->a * hacc[d];
  h_grad[d + 1] = 2.0 * ctx->sigma * hacc[d + 1];
  return GP_OK;
}
