"""The pair (i, i) of a square product counts with r^2 = 0 exactly: K about a^2 I gives a^2 V back.

Points so far apart that everything off the diagonal underflows; the distance of a point to itself, which the matrix cores work
out with an error of up to 2^-21 |x|^2 like any other, must not show.  What may: V as the two fp16 pieces it is multiplied as (worked out here as
the packing does), one rounding of a sum whose other terms are at most 2^-11 of it, two of the scales: 2^-23 in all at the
worst element, 2^-25 in the mean (the vector-ALU column is fp32 throughout, and has the same roundings)."""
import numpy as np
import pytest

from tests.gpu_util import Dev

pytestmark = pytest.mark.gpu


def _pieces(V):
    """V as hi + lo, per column scaled so that the largest is in [2^13, 2^14)"""
    e = np.frexp(np.abs(V).max(axis=0))[1]
    S = np.ldexp(V.astype(np.float64), 14 - e)
    hi = S.astype(np.float32).astype(np.float16)
    lo = (S - hi).astype(np.float32).astype(np.float16)
    return np.ldexp(hi.astype(np.float64) + lo.astype(np.float64), e - 14)


@pytest.mark.parametrize("path", ["f16x2", "f16x3"])
@pytest.mark.parametrize("kind", ["se", "matern32"])
@pytest.mark.parametrize("n,d,t", [(700, 26, 17), (700, 26, 33), (700, 20, 65), (700, 62, 40), (700, 90, 65), (700, 50, 1),
                                   (30011, 26, 65), (30011, 40, 64)])       # the last two: four row tiles per wave
def test_k_of_points_far_apart_is_the_identity(monkeypatch, path, kind, n, d, t):
    monkeypatch.setenv("GPWS_PATH", path)
    rng = np.random.default_rng(n + d + t)
    X = rng.standard_normal((n, d)).astype(np.float32)
    V = rng.standard_normal((n, t)).astype(np.float32)
    dv = Dev(X, kind, np.full(d, np.sqrt(d / 3000.0)), 1.0, 0.3)     # |x|^2 about 3000, distances about 77
    try:
        got = dv.kmv(V, 0)
    finally:
        dv.close()
    want = _pieces(V)
    first = t % 64 in (1, 17, 33)
    if first:
        want[:, 0] = V[:, 0]
    err = got - want
    assert np.abs(err / want).max() <= 2.0 ** -23
    assert np.linalg.norm(err) <= 2.0 ** -25 * np.linalg.norm(want)


@pytest.mark.parametrize("kind", ["se", "matern32"])
@pytest.mark.parametrize("n,d,t", [(300, 5, 1), (300, 26, 17), (300, 90, 65), (300, 5, 33)])
def test_an_infinity_stays_one(kind, n, d, t):
    """The vector-ALU column is multiplied in fp32 as it is: where every entry of K is positive, an infinity in it is one in every row."""
    rng = np.random.default_rng(n + t)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    V = rng.standard_normal((n, t)).astype(np.float32)
    V[[7, 100, 299], 0] = np.inf
    dv = Dev(X, kind, np.full(d, 0.6 * np.sqrt(d)), 1.0, 0.3)
    try:
        got = dv.kmv(V, 1)
    finally:
        dv.close()
    assert np.isposinf(got[:, 0]).all()
    assert np.isfinite(got[:, 1:]).all()
