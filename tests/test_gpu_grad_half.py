"""The gradient's tile pass over one half of the pairs, at the sizes where its rows, pieces and blocks of probes end.

Rows: tiles of 32, workgroups of 4 or 8 of them (8 with more than 32 probes and from n = 3169 on).  Columns: pieces of at least 4 tiles, several per row
from n = 300 on.  Probes: 16 per step, at most 80 per pass, passes of about one size, one step at least.  Bound, per component: the sum over all pairs of the
terms' sizes times

    2^-22 (3 + 2 max |x|^2 + 2)   products of two split factors and G Q (three times 2^-22 at most, each piece being rounded to
                                  nearest), r^2 (2^-22 of the two squared norms), exp and sqrt (1 ulp each)

and the result's own rounding, which that covers."""
import numpy as np
import pytest

from oracle import gp_oracle as orc
from tests.gpu_util import Dev

pytestmark = pytest.mark.gpu


def _check(n, d, t, kind, seed, change=None):
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    V = rng.standard_normal((n, t)).astype(np.float32) * np.exp(rng.uniform(-3, 3, t)).astype(np.float32)
    B = rng.standard_normal((n, t)).astype(np.float32) * np.exp(rng.uniform(-3, 3, t)).astype(np.float32)
    if change:
        change(V, B)
    ell, a, sigma = rng.uniform(0.7, 1.3, d) * np.sqrt(d / 3.0), 1.2, 0.4
    V64, B64 = V.astype(np.float64), B.astype(np.float64)
    s = t - 1
    A, C = V64.copy(), B64.copy()
    A[:, 0] *= 0.5
    C[:, 0] = V64[:, 0]
    if s:
        A[:, 1:] *= -0.5 / s
    W = np.abs(A) @ np.abs(C).T        # sizes of the terms of w_ij
    xs = (X.astype(np.float64) - X.astype(np.float64).mean(0)) / ell
    unit = 2.0 ** -22 * (5.0 + 2.0 * (xs ** 2).sum(1).max())
    dv = Dev(X, kind, ell, a, sigma)
    try:
        got = np.array(dv.grad(dv.to(V), dv.to(B)))
        again = np.array(dv.grad(dv.to(V), dv.to(B)))
    finally:
        dv.close()
    assert (got == again).all()
    ref = orc.mll_grad_hutchinson(X, ell, a, sigma, kind, B64, V=V64)
    for k, dH in enumerate(orc.dH_list(X.astype(np.float64), ell, a, sigma, kind)):
        # an expanded square has terms the size of both squared coordinates, where dH has their difference
        size = (W * np.abs(dH)).sum()
        if k < d:
            psi = np.exp(-0.5 * orc.scaled_sqdist(X, X, ell)) if kind == "se" else 3.0 * np.exp(-np.sqrt(3.0 * orc.scaled_sqdist(X, X, ell)))
            size = a * a / ell[k] * (W * psi * 2.0 * (xs[:, k][:, None] ** 2 + xs[:, k][None, :] ** 2)).sum()
        assert abs(got[k] - ref[k]) <= unit * size, (k, got[k], ref[k], unit * size)


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 127, 128, 129, 255, 256, 257, 300, 511, 513, 1031])
@pytest.mark.parametrize("t", [3, 66])
def test_rows(n, t):
    print(f"[grad half] n={n} t={t}", flush=True)
    _check(n, 4, t, "matern32" if n % 2 else "se", n + t)


@pytest.mark.parametrize("t", [1, 2, 16, 17, 18, 33, 34, 49, 50, 65, 66, 80, 81, 82, 97, 98, 129, 130, 161, 162])
def test_probes(t):
    print(f"[grad half] t={t}", flush=True)
    _check(413, 5, t, "se" if t % 2 else "matern32", t)


@pytest.mark.parametrize("d,t", [(13, 20), (14, 70), (15, 40), (31, 20), (32, 70), (46, 33), (63, 65), (96, 66), (125, 65), (13, 81), (46, 66), (96, 81), (125, 82)])
def test_dimensions(d, t):
    print(f"[grad half] d={d} t={t}", flush=True)
    _check(290, d, t, "matern32", d)


def _zero_columns(which, size):
    def change(V, B):
        V *= np.float32(size)
        for k, M in (("V", V), ("B", B)):
            if which == k:
                M[:, 1] = 0.0
            elif which == k + "*":
                M[:, 1:] = 0.0
        if which == "y":
            V[:, 0] = 0.0
    return change


@pytest.mark.parametrize("which", ["V", "V*", "B", "B*", "y"])
@pytest.mark.parametrize("size", [1e-3, 1e-12])
@pytest.mark.parametrize("t", [3, 40, 66])
def test_zero_columns(which, size, t):
    """A column of zeros on one side takes no part in the bound the weights are scaled by; the other side's values, however
    large next to the small solutions, must not overflow against it."""
    print(f"[grad half] zero {which} size={size} t={t}", flush=True)
    _check(256, 4, t, "matern32", t, _zero_columns(which, size))


def _check_rows(n, d, t, kind, seed):
    """As _check, at sizes where a dense n x n oracle takes too long: V is zero outside 96 rows, which leaves their terms only."""
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    R = np.unique(np.concatenate([rng.choice(n, 88, replace=False), [0, 31, 32, 127, 128, 255, 256, n - 2, n - 1]]))
    V = np.zeros((n, t), dtype=np.float32)
    V[R] = rng.standard_normal((R.size, t))
    B = rng.standard_normal((n, t)).astype(np.float32) * np.exp(rng.uniform(-3, 3, t)).astype(np.float32)
    ell, a, sigma = rng.uniform(0.7, 1.3, d) * np.sqrt(d / 3.0), 1.2, 0.4
    dv = Dev(X, kind, ell, a, sigma)
    try:
        got = np.array(dv.grad(dv.to(V), dv.to(B)))
        assert (got == np.array(dv.grad(dv.to(V), dv.to(B)))).all()
    finally:
        dv.close()
    ref = orc.mll_grad_hutchinson_rows(X, ell, a, sigma, kind, B, V, rows=R, row_block=32, workers=8)
    A, C = V[R].astype(np.float64), B.astype(np.float64)
    A[:, 0] *= 0.5
    C[:, 0] = V[:, 0]
    A[:, 1:] *= -0.5 / (t - 1)
    W = np.abs(A) @ np.abs(C).T
    xs = (X.astype(np.float64) - X.astype(np.float64).mean(0)) / ell
    unit = 2.0 ** -22 * (5.0 + 2.0 * (xs ** 2).sum(1).max())
    r2 = orc.scaled_sqdist(X[R], X, ell)
    psi = np.exp(-0.5 * r2) if kind == "se" else 3.0 * np.exp(-np.sqrt(3.0 * r2))
    size = a * a / ell * 2.0 * (((W * psi).sum(1)[:, None] * xs[R] ** 2).sum(0) + ((W * psi).sum(0)[:, None] * xs ** 2).sum(0))
    size = np.append(size, [(W * 2.0 * orc.kernel_from_sqdist(r2, a, kind) / a).sum(), 2.0 * sigma * W[np.arange(R.size), R].sum()])
    bad = np.abs(got - ref) > unit * size
    assert not bad.any(), (got[bad], ref[bad], (unit * size)[bad])


@pytest.mark.parametrize("n,d,t", [(3168, 5, 66), (3169, 5, 66), (3169, 26, 34), (3329, 13, 65), (3361, 14, 81), (3457, 31, 66), (3500, 46, 65),
                                   (3200, 62, 81), (3169, 96, 65), (3329, 96, 66), (3329, 125, 81), (3329, 60, 98)])
def test_eight_waves(n, d, t):
    print(f"[grad half] n={n} d={d} t={t}", flush=True)
    _check_rows(n, d, t, "matern32" if n % 2 else "se", n + d)


@pytest.mark.parametrize("n,d,t", [(290, 5, 18), (290, 31, 50), (300, 46, 65), (290, 62, 66), (290, 96, 34), (310, 96, 81), (290, 125, 65),
                                   (3169, 31, 50), (3329, 46, 66), (3200, 62, 65), (3329, 96, 34), (3169, 96, 66), (3329, 125, 81)])
def test_three_pieces(monkeypatch, n, d, t):
    monkeypatch.setenv("GPWS_PATH", "f16x3")
    print(f"[grad half] three pieces n={n} d={d} t={t}", flush=True)
    _check_rows(n, d, t, "matern32" if n % 2 else "se", n + d)
