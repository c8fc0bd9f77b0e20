// What the split-fp16 tile pass (tile_kernels_f16.h) and the code that launches it agree on.
#ifndef GPWS_TILE_F16_H
#define GPWS_TILE_F16_H

#include "dist_f16.h"
#include "gpws_internal.h"
#include "split_f16.h"

struct TileArgsH {
  const u32x4* XA;        // column-side operands, 16-byte units [(16 points)*G + group]*64 + lane
  const u32x4* XB;        // row-side operands
  const float* CI;        // gamma |x_i|^2 of the rows, where the accumulators start on two pieces
  const u32x4* VP;        // packed V' images of this pass, [chunk][nt][part][lane]
  const float* VY;        // [n_pad] the VALU column, unscaled (zeros when unused)
  const float* V;         // the caller's V (noise term in the epilogue)
  int64_t ldv;
  const unsigned* colmax; // [t] bit patterns of max_i |V_ic|
  float* OUT;
  int64_t ldo;
  int64_t split_stride;
  int64_t n;               // rows of the output (the context's n, or m for a rectangular product)
  int diag;                // square product: the pair (i, i) counts with r^2 = 0, as 2^15 V'_i (all pieces of V')
  int diag_shift;          // chunk of the first row minus the first chunk of the contraction
  int nchunks;             // column chunks (always the context's points)
  int col0, ncols, vcol;
  int JS, cps;             // column-range splits inside this launch, chunks per split
  int row_blocks;          // workgroups per column range
  int CG;                  // waves of a workgroup that share its rows and take every CG-th chunk: 1, 2, 4 or 8
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

// What a tile kernel is compiled for, besides the row-major product of gp_kmv and gp_predict (FORM_PLAIN).
enum {
  FORM_PLAIN,
  FORM_COLUMNS,   // the solvers' products: column-major images, early return
  FORM_GATHER,    // and rows gathered from the context's points
  FORM_WINDOW,    // and a column window chosen on the device
  FORM_ANY        // all of it, row-major or in columns, chosen by the arguments
};
constexpr bool has_gather(int form) { return form == FORM_GATHER || form == FORM_ANY; }
constexpr bool has_window(int form) { return form == FORM_WINDOW || form == FORM_ANY; }

constexpr int TILE_WAVES = 8;                   // per workgroup: with four, twice the L2-to-LDS traffic, n = 131072 3 to 8 % slower
constexpr int LDS_BYTES = 160 * 1024;

// 16-byte units of a chunk in LDS: operands of its two tiles of points, then V' images
constexpr int chunk_units(int DS, int XP, int NT) { return (2 * dist_groups(XP, DS) + 2 * NT) * 64; }
// Chunks per stage; two stages in LDS, workgroups of a compute unit side by side.  Few: the first stage is waited for.  Many: one
// barrier for them all, and up to as many waves can share the rows of a workgroup.
constexpr int stage_chunks(int DS, int XP, int NT, bool y, int per_cu) {
  for (int c = 8; c > 1; c /= 2)
    if (2 * per_cu * (c * chunk_units(DS, XP, NT) + (y ? 64 : 0)) * 16 <= LDS_BYTES) return c;
  return 1;
}
// Which kernel: four row tiles per wave, or two with this many waves per SIMD.  Four pay with 48 and 64 columns in long products (plan_h), where
// they halve the operands read from LDS, and fit up to four groups of operands per tile.  With fewer columns two row tiles are as fast and
// cut rows finer: n = 43945, d = 20, t = 17 (Matern) 625 us a product against 729, n = 65536, d = 11, t = 33 1517 against 1539.
constexpr bool wide_tiles(int DS, int XP, int NT) { return NT >= 3 && dist_groups(XP, DS) <= 4; }
// Three column tiles leave four waves 28 registers short, two have them all: n = 5000, d = 26, t = 49 1.2 times faster, level from n = 14000 on.
constexpr int tile_waves(int DS, int XP, int NT) {
  return NT == 0 && dist_groups(XP, DS) <= 2 ? 8 : dist_groups(XP, DS) <= (NT == 0 ? 6 : 4) && NT < 3 ? 4 : 2;
}

typedef void (*tileh_fn)(TileArgsH);

// The kernel for operands of shape ds (dist_f16.h) and NT column tiles; y: with the vector-ALU column.  One translation unit for each
// kind of kernel function and number of pieces, which compile side by side.  wide: with four row tiles where wide_tiles says there are.
tileh_fn gp_tile_se_x2(int ds, int NT, bool y, int form, bool wide);
tileh_fn gp_tile_se_x3(int ds, int NT, bool y, int form, bool wide);
tileh_fn gp_tile_matern32_x2(int ds, int NT, bool y, int form, bool wide);
tileh_fn gp_tile_matern32_x3(int ds, int NT, bool y, int form, bool wide);

#endif
