"""Layout of the distance operands: the slots of both sides, multiplied instruction by instruction, give every product of pieces that
gamma r^2 is made of exactly once, for every number of dimensions, both kernels and both numbers of pieces."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2405_18328_amd", "csrc")

CODE = r"""
#include "dist_f16.h"
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>
static double unit() { return rand() / (double)RAND_MAX; }
int main() {
  srand(1);
  for (int shift = 0; shift < 2; ++shift)
    for (int XP = 2; XP <= 3; ++XP)
      for (int d = 1; d <= 126 - shift; ++d) {
        const int id = dist_shape_of(XP, d, shift);
        const DistShape s = dist_shape(XP, id);
        const bool both = dist_both_norms(XP, s.Q);
        std::vector<double> x(3 * d), y(3 * d), nj(3), ni(3);
        for (auto* v : {&x, &y, &nj, &ni})
          for (double& e : *v) e = unit();
        auto value = [&](bool a, int g, int k) {
          const DistSlot t = dist_slot(XP, s.Q, s.R, d, shift, a, g, k);
          if (t.what == DIST_ONE) return 1.0;
          if (t.what == DIST_SHIFT) return 15.0;
          if ((t.what == DIST_X && t.comp >= d) || t.piece >= XP) abort();
          return t.what == DIST_X ? (a ? x : y)[3 * t.comp + t.piece] : t.what == DIST_NORM ? (a ? nj : ni)[t.piece] : 0.0;
        };
        int products = 0;
        auto mul = [&](int a, int b) {
          double q = 0;
          for (int k = 0; k < 32; ++k) q += value(true, a, k) * value(false, b, k);
          ++products;
          return q;
        };
        auto whole = [&](int base) {
          double q = mul(base + 1, base) + mul(base, base + 1) + mul(base, base);
          if (XP == 3) q += mul(base + 1, base + 1) + mul(base + 2, base) + mul(base, base + 2);
          return q;
        };
        double got = 0;
        for (int f = 0; f < s.Q; ++f) got += whole(XP * f);
        if (dist_diagonal(XP, id)) for (int k = 0; k < s.R; ++k) got += mul(XP * s.Q + k, XP * s.Q + k);
        else got += whole(XP * s.Q);
        double want = shift ? 15.0 : 0.0;
        for (int c = 0; c < d; ++c)
          for (int p = 0; p < XP; ++p)
            for (int q = 0; p + q < XP; ++q) want += x[3 * c + p] * y[3 * c + q];
        for (int p = 0; p < XP; ++p) want += nj[p] + (both ? ni[p] : 0.0);
        if (std::fabs(got - want) > 1e-9 || products != dist_products(XP, id)) {
          printf("XP %d d %d shift %d: %.12g, not %.12g\n", XP, d, shift, got, want);
          return 1;
        }
      }
  return 0;
}
"""


def test_every_product_of_pieces_has_one_slot(tmp_path):
    (tmp_path / "layout.cpp").write_text(CODE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "layout.cpp"), "-o", str(tmp_path / "layout")], check=True)
    r = subprocess.run([str(tmp_path / "layout")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
