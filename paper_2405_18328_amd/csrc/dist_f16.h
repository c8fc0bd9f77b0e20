// How the fp16 pieces of a point are laid out for the distance contraction of the tile pass: which products of pieces
// make up gamma r^2, and in which slots of the 32-wide matrix instruction each of them stands.
//
// Points are x = hi + mid (+ lo), each piece rounded to nearest.  gamma r^2_ij = gamma |x_i|^2 + gamma |x_j|^2 - 2 gamma x_i.x_j with
//   two pieces    hi.hi + hi.mid + mid.hi                             relative error 2^-22 per product
//   three pieces  the same and mid.mid + hi.lo + lo.hi                2^-33
// The column side (A) holds pieces of x_j and of gamma |x_j|^2, the row side (B) pieces of -2 gamma x_i and ones; for SE a
// slot 1 . 15 carries phi as 2^15 phi.  On two pieces and up to 31 dimensions gamma |x_i|^2 is the accumulator's start, in fp32; else it
// takes slots of its own.
//
// The first 32 Q dimensions fill whole groups of 32 slots, a group per piece, so that one operand serves several products.
// The rest and the norms: where all their products fit fewer instructions side by side, one slot per product, they are laid
// out like that ("diagonal": group k of A meets group k of B), smallest products first; else a group per piece again.  In units of
// 32x32 pairs and 16 slots, on two pieces: d = 3, 8 and 9 take 2 (3 with whole pieces in instructions of 16 slots), d = 20 4 (6),
// d = 26 6 (6), d = 64 16 (18), d = 90 18 (18), d = 96 24 (24); only 11 <= d <= 14 take 4 instead of 3.
// They cost those dimensions more than the instruction saves where little else is issued (a product, instructions of 16 slots and 32x32x16 -> now,
// d = 11, n = 131072: t = 1 SE 2.01 -> 2.17 ms, Matern 3.52 -> 3.63; d = 12, t = 17 and more columns gain).  v_mfma_f32_16x16x16_f16 for half a group takes
// 0.86 of a whole one's time.
// What is rounded where: v_mfma_f32_16x16x32_f16 adds eight slots at a time to its accumulator, slots 0-7 first; all nine terms are
// cut off 24 bits below the largest of them, and the sum is an fp32 number before the next eight (probed with single products).
// So the largest terms come last, and the shift, larger than all of them, stands in the last slot of the last group, where there
// is room with no products beside it.  Error of gp_kmv against 64 bits, SE, t = 17, n = 1536 - 2048, d = 8 / 90: shift at the accumulator's start
// 4.8e-7 / 11.2e-7, among the hi.hi products 5.0e-7 / 4.2e-7, in the last slot 3.5e-7 / 3.9e-7; instructions of 16 slots had 3.7e-7 / 4.5e-7.
//
#ifndef GPWS_DIST_F16_H
#define GPWS_DIST_F16_H

struct DistShape {
  int Q;       // groups of 32 dimensions with a group per piece
  int R;       // instructions for the rest: 3 (two pieces) or 6 (three) mean a group per piece, fewer are diagonal
  int most;    // most dimensions
  int most_shift;      // with the shift among the slots
};
constexpr DistShape DIST_X2[] = {{0, 1, 10, 8}, {0, 2, 20, 20}, {0, 3, 31, 30}, {1, 1, 41, 41}, {1, 2, 52, 51}, {1, 3, 62, 61},
                                 {2, 2, 84, 83}, {2, 3, 94, 93}, {3, 3, 126, 125}};
constexpr DistShape DIST_X3[] = {{0, 2, 5, 5}, {0, 3, 12, 12}, {0, 4, 18, 18}, {0, 6, 30, 29}, {1, 3, 44, 44}, {1, 4, 50, 50}, {1, 6, 62, 61},
                                 {2, 6, 94, 93}, {3, 6, 126, 125}};
constexpr int DIST_SHAPES_X2 = sizeof(DIST_X2) / sizeof(DIST_X2[0]), DIST_SHAPES_X3 = sizeof(DIST_X3) / sizeof(DIST_X3[0]);

// whether the norms of the row side take slots, too: past 32 dimensions an accumulator that starts with them would be rounded too
// often at their size (SE and Matern-3/2, d = 78: error 2 % larger)
constexpr bool dist_both_norms(int XP, int Q) { return XP == 3 || Q > 0; }
// shapes are counted from 1
constexpr DistShape dist_shape(int XP, int id) { return XP == 2 ? DIST_X2[id - 1] : DIST_X3[id - 1]; }
constexpr bool dist_diagonal(int XP, int id) { return dist_shape(XP, id).R < (XP == 2 ? 3 : 6); }
constexpr int dist_groups(int XP, int id) { return XP * dist_shape(XP, id).Q + (dist_diagonal(XP, id) ? dist_shape(XP, id).R : XP); }
constexpr int dist_products(int XP, int id) { return (XP == 2 ? 3 : 6) * dist_shape(XP, id).Q + dist_shape(XP, id).R; }
constexpr int DIST_MOST_GROUPS_X2 = dist_groups(2, DIST_SHAPES_X2), DIST_MOST_GROUPS_X3 = dist_groups(3, DIST_SHAPES_X3);
constexpr int dist_shape_of(int XP, int d, bool shift) {
  for (int id = 1; id < (XP == 2 ? DIST_SHAPES_X2 : DIST_SHAPES_X3); ++id)
    if (d <= (shift ? dist_shape(XP, id).most_shift : dist_shape(XP, id).most)) return id;
  return XP == 2 ? DIST_SHAPES_X2 : DIST_SHAPES_X3;      // more dimensions than fit do not get here
}

// What stands in slot k (0 .. 31) of group g on one side: a piece (0 hi, 1 mid, 2 lo) of a value, or a constant.
// DIST_X: the coordinate (A) or -2 gamma times it (B); DIST_NORM: gamma |x|^2; DIST_SHIFT: 15
enum { DIST_ZERO, DIST_ONE, DIST_X, DIST_NORM, DIST_SHIFT };
struct DistSlot {
  int what, comp, piece;
};
inline DistSlot dist_slot(int XP, int Q, int R, int d, bool shift, bool side_a, int g, int k) {
  const bool diagonal = R < (XP == 2 ? 3 : 6), last = diagonal && g == XP * Q + R - 1;
  const DistSlot zero = {DIST_ZERO, 0, 0}, one = {DIST_ONE, 0, 0};
  const int r = d > 32 * Q ? d - 32 * Q : 0, own = dist_both_norms(XP, Q) ? 2 : 1;      // norms of one piece
  auto norm = [&](int s, int p) { return (s == 0) == side_a ? DistSlot{DIST_NORM, 0, p} : one; };
  if (shift && k == 31 && (last || (!diagonal && g >= XP * Q)))
    return !last && g != XP * Q ? zero : side_a ? one : DistSlot{DIST_SHIFT, 0, 0};
  if (g < XP * Q || !diagonal) {
    const int c = 32 * (g / XP) + k, piece = g % XP;
    if (g < XP * Q) return c < d ? DistSlot{DIST_X, c, piece} : zero;
    if (k < r) return DistSlot{DIST_X, c, piece};
    if (k >= r + own) return zero;
    const DistSlot s = norm(k - r, piece);
    return s.what == DIST_ONE && piece != 0 ? zero : s;      // the norm's pieces meet the one of the other side's hi group
  }
  // pieces of A and B, smallest products first; behind them the piece of the norms that is about as large
  struct { int a, b, norm; } const terms[6] = {{1, 1, -1}, {0, 2, -1}, {2, 0, 2}, {0, 1, -1}, {1, 0, 1}, {0, 0, 0}};
  // Products fill their groups to the end, or to the eight slots of the shift.  On three pieces the hi.hi products have the last
  // group for themselves.
  const int largest = r + own, others = XP == 3 ? 5 * r + 2 * own : 2 * r + own;
  const int end = 32 * R - (shift ? 8 : 0);
  int s = 32 * (g - XP * Q) + k;
  if (XP == 2) {
    if (end >= largest + others) s -= end - largest - others;
  } else if (last) {
    s -= end - largest - others;
    if (s < others) return zero;
  } else {
    s -= 32 * (R - 1) - others;
  }
  if (s < 0) return zero;
  for (int t = XP == 2 ? 3 : 0; t < 6; ++t) {
    if (s < r) return DistSlot{DIST_X, 32 * Q + s, side_a ? terms[t].a : terms[t].b};
    s -= r;
    if (terms[t].norm < 0) continue;
    if (s < own) return norm(s, terms[t].norm);
    s -= own;
  }
  return zero;
}

#endif
