"""Packing of points (32 rows to a workgroup, eight threads to a norm) and the norm that a prediction waits for.

Row counts around a chunk of 32 and the packed arrays' 512 rows, dimensions around a thread's eight components and a k-step's 16,
and up to the largest.  Bound: products of two split factors (3 2^-22) and r^2 from two pieces per coordinate (2^-22 of the two
squared norms, taken four times for the steps of the chain that meet in it), against the sum of the terms' sizes."""
import numpy as np
import pytest
import torch

from oracle import gp_oracle as orc
from tests.gpu_util import Dev

pytestmark = pytest.mark.gpu


def _unit(X, Xs, ell):
    mean = X.astype(np.float64).mean(0)
    top = max((((P - mean) / ell) ** 2).sum(1).max() for P in (X.astype(np.float64), Xs.astype(np.float64)))
    return 2.0 ** -22 * (5.0 + 8.0 * top)


def _check(dv, X, Xs, ell, a, kind, V):
    got = dv.predict(Xs, V)
    ref = orc.cross_kmv(Xs, X, ell, a, kind, V)
    size = a * a * np.abs(V.astype(np.float64)).sum(0)
    assert (np.abs(got - ref) <= _unit(X, Xs, ell) * size).all(), (np.abs(got - ref) / size).max()


@pytest.mark.parametrize("m", [1, 31, 32, 33, 511, 512, 513])
@pytest.mark.parametrize("n,t", [(65, 1), (1025, 34)])
def test_rows(m, n, t):
    print(f"[pack points] m={m} n={n} t={t}", flush=True)
    rng = np.random.default_rng(m + n)
    d, kind = 5, "se" if m % 2 else "matern32"
    X, Xs = rng.uniform(-1, 1, (n, d)).astype(np.float32), rng.uniform(-1, 1, (m, d)).astype(np.float32)
    V = rng.standard_normal((n, t)).astype(np.float32)
    ell = rng.uniform(0.8, 1.2, d)
    dv = Dev(X, kind, ell, 1.1, 0.3)
    try:
        _check(dv, X, Xs, ell, 1.1, kind, V)
    finally:
        dv.close()


@pytest.mark.parametrize("d", [1, 2, 7, 8, 9, 13, 14, 15, 31, 62, 93, 126])
@pytest.mark.parametrize("kind", ["se", "matern32"])
def test_dimensions(d, kind):
    print(f"[pack points] d={d} {kind}", flush=True)
    rng = np.random.default_rng(d)
    X, Xs = rng.uniform(-1, 1, (323, d)).astype(np.float32), rng.uniform(-1, 1, (70, d)).astype(np.float32)
    V = rng.standard_normal((323, 3)).astype(np.float32)
    ell = rng.uniform(0.8, 1.2, d) * np.sqrt(d)
    dv = Dev(X, kind, ell, 0.9, 0.3)
    try:
        _check(dv, X, Xs, ell, 0.9, kind, V)
    finally:
        dv.close()


def test_a_far_prediction_leaves_nothing_for_the_next():
    """Near points, then points whose norm asks for three pieces, then for fp32, then near ones again: the first call's bits."""
    rng = np.random.default_rng(3)
    X, Xs = rng.uniform(-1, 1, (300, 4)).astype(np.float32), rng.uniform(-1, 1, (40, 4)).astype(np.float32)
    V = rng.standard_normal((300, 33)).astype(np.float32)
    ell = np.full(4, 1.0)
    dv = Dev(X, "matern32", ell, 1.0, 0.3)
    try:
        first = dv.predict(Xs, V)
        for far in (30.0, 300.0):
            dv.predict(far * Xs, V)
            assert (dv.predict(Xs, V) == first).all()
            kmv = dv.kmv(V, 1)
            assert (dv.kmv(V, 1) == kmv).all()
        _check(dv, X, Xs, ell, 1.0, "matern32", V)
    finally:
        dv.close()


def test_several_launches():
    """2^20 chunks to a launch at most: 2^25 + 77 points, which repeat a short set, get that set's predictions again."""
    print("[pack points] 2^25 + 77 points", flush=True)
    rng = np.random.default_rng(25)
    n, d, m, period = 100, 2, (1 << 25) + 77, 4099
    X, Xs = rng.uniform(-1, 1, (n, d)).astype(np.float32), rng.uniform(-1, 1, (period, d)).astype(np.float32)
    V = rng.standard_normal((n, 1)).astype(np.float32)
    dv = Dev(X, "se", np.full(d, 1.0), 1.0, 0.3)
    try:
        few = torch.from_numpy(dv.predict(Xs, V).astype(np.float32)).to(dv.dev)
        Xd, Vd, out = dv.to(Xs).repeat(m // period + 1, 1)[:m].contiguous(), dv.to(V), torch.empty(m, 1, device=dv.dev)
        dv.gp.gp_predict(dv.ctx, Xd, m, Vd, 1, 1, out, 1)
        torch.cuda.synchronize()
        assert torch.equal(out, few.repeat(m // period + 1, 1)[:m])
    finally:
        dv.close()


@pytest.mark.parametrize("n,t", [(300, 70), (8300, 33)])
def test_maxima_left_by_a_far_prediction(n, t):
    """Longer V, or more columns than one pass: the maxima are accumulated in words of the context.  A prediction that turns to fp32 has
    taken those of a much larger V and not cleared them; prediction and product of the first V have their bits from before."""
    print(f"[pack points] maxima n={n} t={t}", flush=True)
    rng = np.random.default_rng(n)
    d, kind = 3, "matern32"
    X, Xs = rng.uniform(-1, 1, (n, d)).astype(np.float32), rng.uniform(-1, 1, (40, d)).astype(np.float32)
    V = rng.standard_normal((n, t)).astype(np.float32)
    big = (1e6 * rng.standard_normal((n, t))).astype(np.float32)
    ell, far = np.full(d, 1.0), (300.0 * Xs).astype(np.float32)
    far[::4] = Xs[::4]              # some of them near, so that there is something to predict
    dv = Dev(X, kind, ell, 1.0, 0.3)
    try:
        predicted, product = dv.predict(Xs, V), dv.kmv(V, 1)
        for again in (lambda: (dv.predict(Xs, V) == predicted).all(), lambda: (dv.kmv(V, 1) == product).all()):
            got = dv.predict(far, big)
            ref = orc.cross_kmv(far, X, ell, 1.0, kind, big)
            size = np.abs(big.astype(np.float64)).sum(0)
            # fp32 throughout: r^2 from the expanded square of the near rows' coordinates, sums of n products
            assert (np.abs(got - ref)[::4] <= 2.0 ** -22 * (5.0 + 8.0 * 3 * d) * size).all()
            assert np.isfinite(got).all()
            assert again()
    finally:
        dv.close()
