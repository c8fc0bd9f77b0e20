"""The tile-pass kernels chosen by size and column count, at the edges of their ranges, against exact fp64 rows.

  - one vector (t = 1): the kernel without contraction tiles, every bucket of distance steps, both
    fp16 paths, single rows, tile edges, an odd chunk count, and the rectangular product with few rows;
  - d <= 29, t > 32 and n at and past 32768: the kernel with four waves per SIMD, with and without the
    vector-ALU column, and a second column pass on the other kernel;
  - t <= 32 at n past 8192: two sub-tiles per wave for both short distance chains;
  - n <= 8192, one column pass: operands packed in one launch, at the edges of its rows per thread and
    of its groups of eight columns; and repeated calls of different widths around it, since the column
    maxima of longer products are accumulated in words that every call has to leave clear.
"""
import numpy as np
import pytest

from oracle import gp_oracle as orc
from tests.gpu_util import Dev, relerr

pytestmark = pytest.mark.gpu

KMV_TOL = 1e-5


def _case(n, d, kind, t, seed=5):
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    V = rng.standard_normal((n, t)).astype(np.float32)
    ell = np.full(d, 0.6 * np.sqrt(d)) * rng.uniform(0.8, 1.2, size=d)
    return X, V, ell


def _rows(n, k=96, seed=1):
    """A sample of rows with the first, the last and both sides of the tile edges among them."""
    edges = [i for i in (0, 31, 32, 127, 128, 255, 256, n - 257, n - 33, n - 1) if 0 <= i < n]
    return np.unique(np.concatenate([edges, np.random.default_rng(seed).integers(0, n, size=k)]))


@pytest.mark.parametrize("path", ["f16x2", "f16x3"])
@pytest.mark.parametrize("kind", ["se", "matern32"])
@pytest.mark.parametrize("n,d", [(1, 3), (31, 3), (33, 13), (97, 14), (257, 29), (1000, 30), (3001, 61), (515, 62), (770, 93), (901, 125)])
def test_one_vector(monkeypatch, path, kind, n, d):
    monkeypatch.setenv("GPWS_PATH", path)
    X, V, ell = _case(n, d, kind, 1)
    dv = Dev(X, kind, ell, 1.3, 0.4)
    try:
        assert relerr(dv.kmv(V, 1), orc.kmv_dense(X, ell, 1.3, kind, V, sigma=0.4)) <= KMV_TOL
        rng = np.random.default_rng(9)
        for m in (1, 300):
            Xs = rng.uniform(-1.0, 1.0, size=(m, d)).astype(np.float32)
            assert relerr(dv.predict(Xs, V), orc.cross_kmv(Xs, X, ell, 1.3, kind, V)) <= KMV_TOL
    finally:
        dv.close()


@pytest.mark.parametrize("n,d,kind,t", [
    (32767, 20, "matern32", 65), (32768, 26, "se", 65), (32801, 14, "matern32", 64), (33000, 29, "se", 97), (70001, 26, "matern32", 34),
    (9001, 26, "matern32", 17), (9001, 12, "se", 33), (8191, 20, "se", 9), (40000, 8, "matern32", 1), (66001, 9, "se", 17)])
@pytest.mark.parametrize("path", ["f16x2", "f16x3"])
def test_kernel_choice_by_size(monkeypatch, path, n, d, kind, t):
    monkeypatch.setenv("GPWS_PATH", path)
    X, V, ell = _case(n, d, kind, t)
    rows = _rows(n)
    ref = orc.kmv_rows(X, ell, 0.9, kind, V, rows, sigma=0.5)
    dv = Dev(X, kind, ell, 0.9, 0.5)
    try:
        assert relerr(dv.kmv(V, 1, ldv=t + 3, ldo=t + 1)[rows], ref) <= KMV_TOL
    finally:
        dv.close()


@pytest.mark.parametrize("n", [1, 33, 1024, 1025, 2049, 4096, 4097, 8192, 8193])
def test_short_pack_and_column_maxima(n):
    X, V, ell = _case(n, 7, "matern32", 97)
    V *= np.exp2(np.random.default_rng(2).integers(-9, 10, size=97)).astype(np.float32)    # columns of very different size
    rows = _rows(n, 32)
    ref = orc.kmv_rows(X, ell, 1.1, "matern32", V, rows, sigma=0.3)
    dv = Dev(X, "matern32", ell, 1.1, 0.3)
    try:
        for c0, t in [(0, 97), (40, 2), (0, 64), (8, 65), (31, 66), (60, 9), (0, 33), (5, 8), (64, 31)]:
            got = dv.kmv(np.ascontiguousarray(V[:, c0:c0 + t]), 1)[rows]
            for c in range(t):
                assert relerr(got[:, c], ref[:, c0 + c]) <= KMV_TOL, (t, c)
    finally:
        dv.close()


@pytest.mark.parametrize("n,d,t", [(400000, 3, 65), (400000, 26, 129), (510000, 3, 257), (200000, 26, 1024), (2000000, 3, 65)])
def test_partial_images_are_bounded(n, d, t):
    """Column splits leave at most 2 GB of partial images, whatever the sizes: the CG workspace is eight arrays of n x t at
    most, the packed operands and those images."""
    import torch
    from paper_2405_18328_amd import binding as gp
    X = torch.rand(n, d, device="cuda:0")
    ctx = gp.gp_create(gp.GP_MATERN32_ARD, n, d, X, torch.cuda.current_stream().cuda_stream)
    try:
        size = gp.gp_workspace_bytes(ctx, t)
        print(f"[scratch] n={n} t={t}: {size / 1e9:.2f} GB", flush=True)
        assert 0 < size <= 8 * 4 * n * t + 264 * n + 2.0e9 + 1e8
    finally:
        gp.gp_destroy(ctx)
