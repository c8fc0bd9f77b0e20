"""Products at the edges of the distance layouts, of the column tiles and of the rows and waves of a workgroup, against exact fp64 sums.

Bar: 1e-5 normwise as everywhere; the sums are of at most 1100 terms, whose products carry 2^-22 (3e-7 observed)."""
import numpy as np
import pytest

from oracle import gp_oracle as orc
from tests.gpu_util import Dev, relerr

pytestmark = pytest.mark.gpu

KMV_TOL = 1e-5


def _case(n, d, t, seed):
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    X[: n // 10] = X[n // 2: n // 2 + n // 10]          # coincident points
    return X, rng.standard_normal((n, t)).astype(np.float32), np.full(d, 0.6 * np.sqrt(d)) * rng.uniform(0.8, 1.2, size=d)


@pytest.mark.parametrize("path", ["f16x2", "f16x3"])
@pytest.mark.parametrize("kind", ["se", "matern32"])
def test_every_distance_layout(monkeypatch, path, kind):
    monkeypatch.setenv("GPWS_PATH", path)
    for d in (1, 5, 6, 8, 9, 10, 11, 12, 13, 18, 19, 20, 21, 29, 30, 31, 32, 33, 41, 42, 44, 45, 50, 51, 52, 53, 61, 62, 63, 64, 83, 84, 85, 93,
              94, 95, 96, 124, 125):
        n, t = 257 + d % 3, 65 if d % 2 else 17
        X, V, ell = _case(n, d, t, d)
        print(f"[dist] {path} {kind} d={d} t={t}", flush=True)
        dv = Dev(X, kind, ell, 1.2, 0.4)
        try:
            assert relerr(dv.kmv(V, 1), orc.kmv_dense(X, ell, 1.2, kind, V, sigma=0.4)) <= KMV_TOL, d
        finally:
            dv.close()


@pytest.mark.parametrize("t", [1, 2, 15, 16, 17, 18, 32, 33, 34, 48, 49, 50, 63, 64, 65, 66, 80, 81, 97, 98, 113, 129])
def test_every_number_of_column_tiles(t):
    X, V, ell = _case(700, 6, 129, 3)
    V *= np.exp2(np.random.default_rng(2).integers(-9, 10, size=129)).astype(np.float32)
    rng = np.random.default_rng(4)
    Xs = rng.uniform(-1.0, 1.0, size=(33, 6)).astype(np.float32)
    dv = Dev(X, "matern32", ell, 1.1, 0.3)
    try:
        ref, pred = orc.kmv_dense(X, ell, 1.1, "matern32", V[:, :t], sigma=0.3), orc.cross_kmv(Xs, X, ell, 1.1, "matern32", V[:, :t])
        got, gp = dv.kmv(np.ascontiguousarray(V[:, :t]), 1, ldv=t + 1, ldo=t + 2), dv.predict(Xs, np.ascontiguousarray(V[:, :t]))
        for c in range(t):
            assert relerr(got[:, c], ref[:, c]) <= KMV_TOL and relerr(gp[:, c], pred[:, c]) <= KMV_TOL, c
    finally:
        dv.close()


@pytest.mark.parametrize("d", [3, 18, 26, 40, 50, 61])
def test_four_row_tiles_in_long_products(d):
    """The layouts that have a kernel with four row tiles per wave, at a size where it is chosen; 64 rows are checked.  Rows add up 30011
    terms in ranges of at most 1024 chunks: an fp32 chain of partial sums adds below 1e-6 normwise."""
    n, t, kind = 30011, 65, "se" if d % 4 else "matern32"
    X, V, ell = _case(n, d, t, d)
    rows = np.r_[0:8, n // 2: n // 2 + 24, n - 32: n]
    dv = Dev(X, kind, ell, 1.2, 0.4)
    try:
        ref = orc.cross_kmv(X[rows], X, ell, 1.2, kind, V) + 0.4 ** 2 * V[rows].astype(np.float64)
        assert relerr(dv.kmv(V, 1)[rows], ref) <= KMV_TOL
    finally:
        dv.close()


@pytest.mark.parametrize("d,t", [(4, 17), (26, 65), (90, 40)])
def test_rows_and_chunks_around_the_cuts(d, t):
    """129 to 1100 points: from 5 chunks of columns on, waves share rows and columns are cut into ranges."""
    for n in (31, 128, 129, 160, 161, 255, 256, 257, 511, 513, 769, 1023, 1025, 1100):
        X, V, ell = _case(n, d, t, n)
        dv = Dev(X, "se", ell, 0.9, 0.5)
        try:
            assert relerr(dv.kmv(V, 1), orc.kmv_dense(X, ell, 0.9, "se", V, sigma=0.5)) <= KMV_TOL, n
        finally:
            dv.close()


def test_far_test_inputs_take_three_pieces_of_both_sides():
    """Training inputs on two pieces, test inputs so far out that three are needed: operands the theta did not ask for are packed
    by the prediction, once for the training inputs, and a product afterwards is the one before."""
    X, V, ell = _case(300, 7, 9, 5)
    rng = np.random.default_rng(6)
    near, far = (rng.uniform(-1.0, 1.0, size=(70, 7)).astype(np.float32) for _ in range(2))
    far[::2] *= 12.0
    dv = Dev(X, "matern32", ell, 1.0, 0.3)
    try:
        first = dv.kmv(V, 1)
        for Xs in (far, near, far):
            assert relerr(dv.predict(Xs, V), orc.cross_kmv(Xs, X, ell, 1.0, "matern32", V)) <= KMV_TOL
        assert np.array_equal(first, dv.kmv(V, 1))
    finally:
        dv.close()
