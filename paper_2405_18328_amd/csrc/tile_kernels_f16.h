// Matrix-free product OUT = K V (+ sigma^2 V), split-fp16 matrix-core path.
//
// On gfx950 the fp32 MFMA shares the SIMD's FMA lanes with the VALU (measured: VALU work adds to
// fp32-MFMA time instead of hiding under it), while the fp16 MFMA runs on the matrix cores at 16x the
// rate and overlaps with VALU work.  This path therefore evaluates both contractions of the tile pass
// with v_mfma_f32_16x16x32_f16 on operands split into fp16 pieces, fp32 accumulation:
//   x = hi + mid (+ lo), each piece an 11-bit fp16 mantissa, so
//   a.b ~ ah.bh + ah.bm + am.bh (+ ah.bl + al.bh + am.bm): relative error 2^-22 (2^-33), i.e. fp32-class.
// The VALU keeps what needs fp32: the kernel function (exp2 / sqrt) and the split of phi.
//
// Why 16x16x32 and not 32x32x16, which does the same work in half the instructions: under the matrix cores' load the chip
// runs at the clock its power allows, and longer sums in smaller tiles need less of it.  Loops of either, on random operands in
// registers: 20.2 ns per 32x32x16 at 1.60 GHz, 16.7 ns for two 16x16x32 at 1.98 GHz (on zeros 13.7 and 14.0 ns, 2.39 GHz).
// The pass itself ran at 1.74 GHz (d = 11) to 1.98 GHz (d = 26) on the former and runs at 2.16 to 2.23 GHz of 2.4 on the latter.  Matrix cores are busy 63 %
// and 43 % of the cycles there, the vector port beside them in 27 to 30 % of that time: what bounds it is that the two hardly overlap.
//
// Per 16x16 tile of pairs (j, i), one wavefront:
//   1. S[j][i] = XA_j . XB_i     the products of dist_f16.h, 32 slots each (= g r^2_ij [+ 15 for SE])
//   2. phi' = 2^15 phi(S)        VALU; hi = phi' cut to fp16, lo = phi' - hi rounded; packed to fp16 pairs
//   3. OUT_i += phi'[i][j] V'_j  3 MFMAs per 16 columns, over the two tiles of a chunk of 32 columns j; V' = V scaled per
//                                column by a power of two so that max |V'_c| is in [2^13, 2^14), pre-split and pre-packed
// The accumulator layout of step 1 (lane = i, register r <-> j = 4(lane/16) + r) gives each lane the eight values of its
// A operand in step 3: four of the chunk's first tile and four of its second, provided the V' rows are packed in that
// order (j = 16(e/4) + 4(lane/16) + e%4 for element e); phi never leaves registers, K is never stored.
#ifndef GPWS_TILE_KERNELS_F16_H
#define GPWS_TILE_KERNELS_F16_H

#include "tile_f16.h"

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

namespace {

// first chunk of the column side (0 unless the launch works on a block chosen on the device)
__device__ __forceinline__ int window_chunk(const TileArgsH& p) {
  return p.win_sel ? __builtin_amdgcn_readfirstlane((int)(((int64_t)*p.win_sel * p.win_block) >> 5)) : 0;
}

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// The tile pass of one workgroup: W waves, RT row tiles each, stages of SC chunks.  CG waves share their rows and split the chunks of
// a stage, which makes the workgroup's rows fewer instead of the output's partial images more; their sums are
// added up in LDS at the end, in a fixed order.
//
// Staging goes global -> LDS directly (global_load_lds_dwordx4: lane L of a wave lands at the wave's LDS base + 16 L), one stage
// ahead, so no registers are held.  The loads are issued through inline assembly on purpose: the compiler's wait-count pass
// treats an LDS-DMA load as aliasing every later LDS read and would drain it at once.  Here the ordering is explicit: s_waitcnt
// vmcnt(0) at the top of a stage, then the barrier, then the next stage's loads.
//
// Vector and matrix instructions are left to the compiler's order, and the other waves of the SIMD fill the gaps.  Software pipelines
// (distances and phi a chunk ahead of the contraction, one matrix instruction per bundle of vector work) measured 5 to 8 %
// slower at n = 131072, raised wave priority around the matrix instructions 8 %, other orders of the three products level.
template <int KIND, int DS, int XP, int NT, int RT, bool Y, int FORM, int SC>
__device__ __forceinline__ void tile_pass(const TileArgsH& p, u32x4* lds) {
  constexpr DistShape D = dist_shape(XP, DS);
  constexpr bool DIAGONAL = dist_diagonal(XP, DS);
  constexpr int G = dist_groups(XP, DS);
  constexpr int W = TILE_WAVES;
  constexpr int XA_G = 2 * G;                       // groups of 64 16-byte units per chunk: points, then V' images
  constexpr int V_G = 2 * NT;
  constexpr int CH_G = XA_G + V_G;
  constexpr int VY_OFF = SC * CH_G * 64;                 // the chunks' 32 y values each: 8 units (64 are fetched)
  constexpr int STAGE = VY_OFF + (Y ? 64 : 0);
  constexpr int LPW = (SC * CH_G + W - 1) / W;      // group loads per wave and stage; surplus slots repeat the last group
  static_assert(NT > 0 || Y, "nothing to multiply");

  const int over = FORM != FORM_PLAIN && p.done ? *p.done : 0;   // looked at only once the first loads are on their way
  if (p.clear && blockIdx.x == 0)
    for (int c = threadIdx.x; c < p.clear_n; c += blockDim.x) p.clear[c] = 0u;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction: lets the compiler branch on it
  const int q = lane >> 4;
  const int li = lane & 15;
  // Workgroup b runs on XCD b % 8: every XCD gets a run of consecutive row blocks of one column range, whose chunks its L2 then fetches once
  const int order = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  const int js = __builtin_amdgcn_readfirstlane(order / p.row_blocks);
  const int rb = order - js * p.row_blocks;
  if (js >= p.JS) return;
  const int cg = wave & (p.CG - 1);
  const int tile0 = (rb * W + wave) / p.CG * RT;               // the wave's first row tile
  const int chunk0 = has_window(FORM) ? window_chunk(p) : 0;
  // The workgroup's column range [r_begin, r_end) is walked in segments [c_begin, c_end) of at most
  // GP_FLUSH_CHUNKS chunks; the accumulators are added into OUT after each segment (see flush below).
  const int r_begin = js * p.cps;
  int r_end = min(p.nchunks, r_begin + p.cps);
  if (has_window(FORM)) r_end = min(r_end, (int)((p.npoints + 31) >> 5) - chunk0);
  int c_begin = r_begin;
  int c_end = min(r_end, c_begin + GP_FLUSH_CHUNKS);

  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
  const unsigned lane16 = lane * 16u;
  auto dma16 = [](uint64_t base, unsigned off, unsigned lds_addr) {
    // m0 carries the LDS address of the load; it is declared clobbered, so the compiler keeps nothing in it
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds_addr) : "memory", "m0");
  };
  // Chunks ch0 .. ch0 + SC - 1, as they lie in memory: the points of all of them, then the images of V'.  Groups past the end are the
  // last one again, which nobody reads.
  const char* XA = reinterpret_cast<const char*>(p.XA) + (int64_t)chunk0 * XA_G * 1024;
  auto issue_stage = [&](int ch0, int st) {
#pragma unroll
    for (int x = 0; x < LPW; ++x) {
      const int g = min(wave + W * x, SC * CH_G - 1);
      const bool points = g < SC * XA_G;
      const int64_t at = points ? min((int64_t)ch0 * XA_G + g, (int64_t)c_end * XA_G - 1) : min((int64_t)ch0 * V_G + (g - SC * XA_G), (int64_t)c_end * V_G - 1);
      dma16((uint64_t)((points ? XA : reinterpret_cast<const char*>(p.VP)) + at * 1024), lane16, lds_base + 16u * (unsigned)(st * STAGE + g * 64));
    }
    if (Y && wave == W - 1) {   // 8 chunks' y values, the last quad again past the end
      const int at = min(ch0 * 8 + lane, c_end * 8 - 1);
      dma16((uint64_t)p.VY, (unsigned)at * 16u, lds_base + 16u * (unsigned)(st * STAGE + VY_OFF));
    }
  };
  const bool empty = has_window(FORM) && r_begin >= r_end;     // a block at the end of the points is shorter than the launch
  if (!empty) issue_stage(c_begin, 0);

  // row-side operands: registers for the whole pass
  f16x8 xb[RT][G];
  f32x4 start[RT];
#pragma unroll
  for (int it = 0; it < RT; ++it) {
    const int64_t slot = (int64_t)(tile0 + it) * 16 + li;
    int64_t i = slot;
    if (has_gather(FORM) && p.gather) {
      const int64_t v = p.gather[slot < p.n ? slot : 0];
      i = v >= 0 && v < p.npoints ? v : 0;
    }
    const int64_t at = (i >> 4) * G * 64 + (lane & 48) + (i & 15);
#pragma unroll
    for (int g = 0; g < G; ++g) xb[it][g] = as_f16x8(p.XB[at + g * 64]);
    const float c = dist_both_norms(XP, D.Q) ? 0.0f : p.CI[i];
    start[it] = f32x4{c, c, c, c};
  }

  // What the output is scaled with goes out with the first loads and waits in registers, where there are some: fetched behind the loop, a
  // short product waits for it again (t <= 48: n = 1000 1 to 2 %, n = 2200 0.5 %; level from n = 16384 on).
  constexpr bool SCALES = RT == 2;
  unsigned top[SCALES && NT > 0 ? NT : 1];
  float scales[SCALES && NT > 0 ? NT : 1];
  auto column_top = [&](int nt, int of) { return p.colmax[p.col0 + min(16 * nt + of, p.ncols - 1)]; };
  auto out_scale = [&](unsigned max_bits) { return p.a2 * ldexpf(1.0f, column_exponent(max_bits) - V_TOP - PHI_SHIFT); };
  if constexpr (SCALES) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) top[nt] = column_top(nt, li);
  }

  f32x4 acc[RT][NT > 0 ? NT : 1];
  float accv[RT];
#pragma unroll
  for (int it = 0; it < RT; ++it) {
    accv[it] = 0.0f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[it][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // S of a tile of points against row tile `it`, smallest terms first
  auto distance = [&](const f16x8 (&xa)[G], int it) {
    f32x4 r = start[it];
    auto mul = [&](int a, int b) { r = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[a], xb[it][b], r, 0, 0, 0); };
    constexpr int B0 = XP * D.Q, WHOLE = D.Q + (DIAGONAL ? 0 : 1);
    if constexpr (DIAGONAL) {
#pragma unroll
      for (int k = 0; k + 1 < D.R; ++k) mul(B0 + k, B0 + k);
    }
#pragma unroll
    for (int f = 0; f < WHOLE; ++f) {
      if constexpr (XP == 3) {
        mul(XP * f + 1, XP * f + 1);
        mul(XP * f + 2, XP * f);
        mul(XP * f, XP * f + 2);
      }
      mul(XP * f + 1, XP * f);
      mul(XP * f, XP * f + 1);
    }
#pragma unroll
    for (int f = 0; f < WHOLE; ++f) mul(XP * f, XP * f);
    if constexpr (DIAGONAL) mul(B0 + D.R - 1, B0 + D.R - 1);
    return r;
  };
  auto phi = [](float s) {
    if (KIND == GP_SE_ARD) return __builtin_amdgcn_exp2f(s);      // s = -log2(e)/2 r^2 + 15
    // s = 3 r^2; a rounding-level negative value is mirrored instead of clamped (|.| is a free source modifier)
    const float u = __builtin_amdgcn_sqrtf(__builtin_fabsf(s));
    const float ex = __builtin_amdgcn_exp2f(fmaf(u, -LOG2E, (float)PHI_SHIFT));
    return fmaf(u, ex, ex);
  };

  // The pair (i, i) of a square product counts with r^2 = 0 exactly: with 2^15 V'_i.  The loop takes it as it comes, with the rounding of its
  // distance, as hi V'_i + lo Vh_i (phi(S_ii) in two pieces, V' = Vh + Vl), and the accumulators start with what that is short of:
  // (2^15 - hi - lo) Vh_i + (2^15 - hi) Vl_i, S_ii worked out here by the same instructions.  (Short of phi(S_ii) itself the split's own rounding and the
  // dropped product would stay in: K = a^2 I came out 1.1e-7 off instead of 4.4e-8, which is what V' has.)  A
  // special case inside the loop would put a branch between distances and phi, across which nothing is scheduled.
  const int own = tile0 / 2 + p.diag_shift;      // the chunk that holds the first row tile's own points
  if (p.diag && cg == 0 && own + RT / 2 > r_begin && own < r_end) {
    // all loads first, from the nearest chunk of the range where a tile's own is not in it
    auto own_chunk = [&](int it) { return max(r_begin, min(own + it / 2, r_end - 1)); };
    f16x8 xa[RT][G], vh[RT / 2][NT > 0 ? NT : 1], vl[RT / 2][NT > 0 ? NT : 1];
    float vy[RT];
#pragma unroll
    for (int it = 0; it < RT; ++it) {
#pragma unroll
      for (int g = 0; g < G; ++g) xa[it][g] = as_f16x8(p.XA[((int64_t)(2 * own_chunk(it) + (it & 1)) * G + g) * 64 + lane]);
      if (Y) vy[it] = p.VY[(int64_t)own_chunk(it) * 32 + 16 * (it & 1) + li];
    }
#pragma unroll
    for (int m = 0; m < RT / 2; ++m)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {      // V' is packed in the order the accumulators have
        const u32x4* v = p.VP + ((int64_t)own_chunk(2 * m) * NT + nt) * 128 + lane;
        vh[m][nt] = as_f16x8(v[0]);
        vl[m][nt] = as_f16x8(v[64]);
      }
#pragma unroll
    for (int it = 0; it < RT; ++it) {
      const int jt = it & 1;
      const bool here = own + it / 2 >= r_begin && own + it / 2 < r_end;
      const f32x4 S = distance(xa[it], it);
      const float s = li & 2 ? (li & 1 ? S[3] : S[2]) : li & 1 ? S[1] : S[0];
      const bool mine = here && q == li >> 2;      // lane 20 (li/4) + li%4 holds row li's
      const float f = mine ? phi(s) : (float)(1 << PHI_SHIFT);
      // An infinite V_i is infinite in the loop; what is missing of it would make a NaN of that.  (With `mine` in this condition the load of
      // V_i would move behind it, to be waited for on its own.)
      if (Y) accv[it] = __builtin_isfinite(vy[it]) ? ((float)(1 << PHI_SHIFT) - f) * vy[it] : 0.0f;
      if constexpr (NT > 0) {
        unsigned hi, lo;
        split_pair_positive(f, 0.0f, hi, lo);
        const int both = (int)(hi | lo << 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const unsigned of_row = (unsigned)__shfl(both, 20 * q + r);
          const float less_hi = minus_half<0>(of_row, (float)(1 << PHI_SHIFT)), less_both = minus_half<1>(of_row, less_hi);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[it][nt][r] = fmaf((float)vh[it / 2][nt][4 * jt + r], less_both, (float)vl[it / 2][nt][4 * jt + r] * less_hi);
        }
      }
    }
  }

  auto chunk = [&](const u32x4* s, const u32x4* sv, const u32x4* sy) {
    f32x4 S[RT][2];
#pragma unroll
    for (int jt = 0; jt < 2; ++jt) {
      f16x8 xa[G];
#pragma unroll
      for (int g = 0; g < G; ++g) xa[g] = as_f16x8(s[(jt * G + g) * 64 + lane]);
#pragma unroll
      for (int it = 0; it < RT; ++it) S[it][jt] = distance(xa, it);
    }
    f32x4 vy[2];
    if (Y) {
#pragma unroll
      for (int jt = 0; jt < 2; ++jt) vy[jt] = __builtin_bit_cast(f32x4, sy[4 * jt + q]);
    }
#pragma unroll
    for (int it = 0; it < RT; ++it) {
      u32x4 ph{}, pl{};
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        float f[2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          const int r = 2 * (e2 & 1) + z;
          f[z] = phi(S[it][e2 >> 1][r]);
          if (Y) accv[it] = fmaf(f[z], vy[e2 >> 1][r], accv[it]);
        }
        if constexpr (NT > 0) {
          unsigned oh, ol;
          split_pair_positive(f[0], f[1], oh, ol);
          ph[e2] = oh;
          pl[e2] = ol;
        }
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {      // smallest terms first: lo*hi, hi*lo, hi*hi
        const f16x8 bh = as_f16x8(sv[2 * nt * 64 + lane]), bl = as_f16x8(sv[(2 * nt + 1) * 64 + lane]);
        acc[it][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(pl), bh, acc[it][nt], 0, 0, 0);
        acc[it][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(ph), bl, acc[it][nt], 0, 0, 0);
        acc[it][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(ph), bh, acc[it][nt], 0, 0, 0);
      }
    }
  };

  // The waves that share rows add up what they hold: in step s every second one of those left hands its accumulators to its
  // neighbour through LDS.  Nobody reads or writes the stages any more.
  constexpr int AU = RT * NT + (Y ? (RT + 3) / 4 : 0);           // 16-byte units per lane
  static_assert(TILE_WAVES / 2 * AU * 64 <= 2 * STAGE, "the accumulators of half the waves do not fit the stages");
  auto add_up = [&]() {
    for (int s = 1; s < p.CG; s *= 2) {
      f32x4* box = reinterpret_cast<f32x4*>(lds) + wave / (2 * s) * AU * 64 + lane;
      const int turn = cg & (2 * s - 1);
      if (turn == s) {
#pragma unroll
        for (int it = 0; it < RT; ++it)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) box[(it * NT + nt) * 64] = acc[it][nt];
        if (Y) {
#pragma unroll
          for (int it = 0; it < RT; ++it) reinterpret_cast<float*>(&box[(RT * NT + it / 4) * 64])[it & 3] = accv[it];
        }
      }
      __syncthreads();
      if (turn == 0) {
#pragma unroll
        for (int it = 0; it < RT; ++it)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[it][nt] += box[(it * NT + nt) * 64];
        if (Y) {
#pragma unroll
          for (int it = 0; it < RT; ++it) accv[it] += reinterpret_cast<const float*>(&box[(RT * NT + it / 4) * 64])[it & 3];
        }
      }
      __syncthreads();
    }
  };

  // Writes what the accumulators hold to OUT (first: stores, adds the noise term once; later: adds to
  // what is there) and clears them.  Undoes the power-of-two scalings and multiplies by a^2.  All loads go out before the first
  // value is used, with clamped indices instead of a branch around each, behind which they would be waited for one by one.
  float* out = p.OUT + (int64_t)js * p.split_stride;
  auto flush = [&](bool first) {
    const bool noise = first && p.add_noise && js == 0;
    // an opaque zero keeps the address arithmetic of the flush inside it, that of rows and that of columns: hoisted out of the segment
    // loop it would hold dozens of registers across the main loop, or be stored to scratch memory in front of it
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    const bool mine = cg == 0;
    const int li0 = li + zero, q0 = q + zero;
    const int64_t ibase = (int64_t)tile0 * 16 + zero;
    const bool columns = FORM == FORM_ANY ? p.cm_ld != 0 : FORM != FORM_PLAIN;
    float oscale[NT > 0 ? NT : 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) oscale[nt] = SCALES ? scales[SCALES ? nt : 0] : out_scale(column_top(nt, li0));
    const float yscale = p.a2 * ldexpf(1.0f, -PHI_SHIFT);
#pragma unroll
    for (int it = 0; it < RT; ++it) {
      const int64_t i0 = ibase + 16 * it;
      if (Y) {
        accv[it] += __shfl_xor(accv[it], 16);
        accv[it] += __shfl_xor(accv[it], 32);
      }
      if (columns) {
        if (mine && i0 < p.cm_ld) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const int c = 16 * nt + li0;
            f32x4 v = oscale[nt] * acc[it][nt];
            if (c < p.ncols) {
              f32x4* d = reinterpret_cast<f32x4*>(out + (int64_t)(p.col0 + c) * p.cm_ld + i0 + 4 * q0);
              if (!first) v += *d;
              *d = v;
            }
          }
          if (Y && q0 == 0) {
            float* o = out + (int64_t)p.vcol * p.cm_ld + i0 + li0;
            const float v = yscale * accv[it];
            *o = first ? v : *o + v;
          }
        }
      } else if (mine) {
        auto row = [&](int r) { return i0 + 4 * q0 + r; };
        float v[NT > 0 ? NT : 1][4];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int r = 0; r < 4; ++r) v[nt][r] = oscale[nt] * acc[it][nt][r];
        auto add = [&](const float* from, int64_t ld, float times) {
          float w[NT > 0 ? NT : 1][4];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) w[nt][r] = from[min(row(r), p.n - 1) * ld + p.col0 + min(16 * nt + li0, p.ncols - 1)];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[nt][r] = fmaf(times, w[nt][r], v[nt][r]);
        };
        if (noise) add(p.V, p.ldv, p.sigma2);
        if (!first) add(out, p.ldo, 1.0f);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * nt + li0 < p.ncols && row(r) < p.n) out[row(r) * p.ldo + p.col0 + 16 * nt + li0] = v[nt][r];
        if (Y && q0 == 0 && i0 + li0 < p.n) {
          const int64_t i = i0 + li0;
          float v1 = yscale * accv[it];
          if (noise) v1 = fmaf(p.sigma2, p.V[i * p.ldv + p.vcol], v1);
          if (!first) v1 += out[i * p.ldo + p.vcol];
          out[i * p.ldo + p.vcol] = v1;
        }
      }
      accv[it] = 0.0f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[it][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };

  // Rounding error of an fp32 accumulator grows with the length of its chain of partial sums, so the
  // accumulators are added into OUT after every segment (the running sum then sees one addition per
  // segment).  The same threads read and write the same elements: no race, fixed order.
  // The row operands are waited for here, where the compiler sees it: it would otherwise wait for them at their first use,
  // inside the loop, and there drain the stage in flight too.
  __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
  if constexpr (SCALES) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) scales[nt] = out_scale(top[nt]);
  }
  if (over) return;                       // nothing is in flight any more
  bool first = true;
  if (empty) {
    flush(true);
    return;
  }
  for (;;) {
    int st = 0;
    for (int ch0 = c_begin; ch0 < c_end; ch0 += SC) {
      asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
      __syncthreads();              // this stage is complete in LDS, every wave is done with the other one
      if (ch0 + SC < c_end) issue_stage(ch0 + SC, st ^ 1);
      const u32x4* s = lds + st * STAGE;
      for (int k = cg; k < SC && ch0 + k < c_end; k += p.CG)
        chunk(s + k * XA_G * 64, s + (SC * XA_G + k * V_G) * 64, s + VY_OFF + 8 * k);
      st ^= 1;
    }
    __syncthreads();                // no wave is still reading when the stages are refilled or reused
    add_up();
    flush(first);
    first = false;
    if (c_end >= r_end) break;
    c_begin = c_end;
    c_end = min(r_end, c_begin + GP_FLUSH_CHUNKS);
    issue_stage(c_begin, 0);
  }
}

// Two row tiles per wave, for what holds few accumulators, and where the points' operands fill the registers.  NT = 0 is the product with
// a single vector (the mean of a prediction): no contraction at all, phi goes straight into one FMA per pair.
template <int KIND, int DS, int XP, int NT, bool Y, int FORM>
__global__ __launch_bounds__(64 * TILE_WAVES) __attribute__((amdgpu_waves_per_eu(tile_waves(DS, XP, NT), tile_waves(DS, XP, NT)))) void kmv_tile_f16_kernel(TileArgsH p) {
  constexpr int SC = stage_chunks(DS, XP, NT, Y, tile_waves(DS, XP, NT) / 2);
  __shared__ u32x4 lds[2 * (SC * chunk_units(DS, XP, NT) + (Y ? 64 : 0))];
  tile_pass<KIND, DS, XP, NT, 2, Y, FORM, SC>(p, lds);
}

// Four row tiles per wave and 48 or 64 columns: every operand read from LDS serves 64 rows, two waves per SIMD, one
// workgroup per compute unit.  Against four waves per SIMD with two row tiles, n = 131072, loops of the main part: d = 26, t = 65 (Matern) 478 and
// 498 ns per 32x32 tile and SIMD, d = 11 (SE) 375 and 392, d = 3 (SE) 347 and 364.
template <int KIND, int DS, int XP, int NT, bool Y, int FORM>
__global__ __launch_bounds__(64 * TILE_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void kmv_tile_f16_wide_kernel(TileArgsH p) {
  constexpr int SC = stage_chunks(DS, XP, NT, Y, 1);
  __shared__ u32x4 lds[2 * (SC * chunk_units(DS, XP, NT) + (Y ? 64 : 0))];
  tile_pass<KIND, DS, XP, NT, 4, Y, FORM, SC>(p, lds);
}

// Two row tiles: built once per form where a short product or step may take them, whose time is to a good part that of the code in front of the
// loop and behind it (one kernel with everything in it: n = 1000, d = 3, t = 17 6 % longer, n = 5000 1 %, level from 16384 on).
template <int KIND, int DS, int XP, int NT, bool Y>
tileh_fn pick_rows(int form, bool wide) {
  if constexpr (wide_tiles(DS, XP, NT)) {
    if (wide) return kmv_tile_f16_wide_kernel<KIND, DS, XP, NT, Y, FORM_ANY>;
  }
  if (form == FORM_PLAIN) return kmv_tile_f16_kernel<KIND, DS, XP, NT, Y, FORM_PLAIN>;
  if (form == FORM_COLUMNS) return kmv_tile_f16_kernel<KIND, DS, XP, NT, Y, FORM_COLUMNS>;
  if constexpr (NT > 0 && NT <= 2 && DS <= 2) {
    if (form == FORM_GATHER) return kmv_tile_f16_kernel<KIND, DS, XP, NT, Y, FORM_GATHER>;
    if (form == FORM_WINDOW) return kmv_tile_f16_kernel<KIND, DS, XP, NT, Y, FORM_WINDOW>;
  }
  return kmv_tile_f16_kernel<KIND, DS, XP, NT, Y, FORM_ANY>;
}

template <int KIND, int DS, int XP, bool Y>
tileh_fn pick_nt(int NT, int form, bool wide) {
  switch (NT) {
    case 1: return pick_rows<KIND, DS, XP, 1, Y>(form, wide);
    case 2: return pick_rows<KIND, DS, XP, 2, Y>(form, wide);
    case 3: return pick_rows<KIND, DS, XP, 3, Y>(form, wide);
  }
  return pick_rows<KIND, DS, XP, 4, Y>(form, wide);
}

template <int KIND, int XP, int DS = 1>
tileh_fn pick_shape(int ds, int NT, bool y, int form, bool wide) {
  if (ds == DS) {
    if (NT == 0) return pick_rows<KIND, DS, XP, 0, true>(form, wide);
    return y ? pick_nt<KIND, DS, XP, true>(NT, form, wide) : pick_nt<KIND, DS, XP, false>(NT, form, wide);
  }
  if constexpr (DS < (XP == 2 ? DIST_SHAPES_X2 : DIST_SHAPES_X3)) return pick_shape<KIND, XP, DS + 1>(ds, NT, y, form, wide);
  else return nullptr;
}

}  // namespace

#endif
