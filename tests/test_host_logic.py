"""CPU checks of the host-side logic around the library: the Adam / softplus outer loop against the
oracle's own, the seeded workload generators, and the flop accounting of the benchmark."""
import importlib.util
import os

import numpy as np

from oracle import gp_oracle as orc
from paper_2405_18328_amd.inputs import make
from paper_2405_18328_amd.mll import AdamState, softplus, softplus_inverse

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_softplus_pair_is_a_bijection_on_the_positive_reals():
    theta = np.array([1e-6, 0.03, 1.0, 7.5, 40.0, 800.0])
    raw = softplus_inverse(theta)
    assert np.allclose(softplus(raw), theta, rtol=1e-12, atol=0)
    assert np.allclose(raw, orc.softplus_inverse(theta), rtol=1e-12)
    assert np.all(np.diff(raw) > 0)


def test_adam_state_follows_the_oracle_trace():
    """Same update rule as the oracle's adam_ascent (Section 4: Adam, learning rate 0.1, on
    softplus-constrained hyperparameters) for a concave toy objective."""
    target = np.array([0.4, 2.0, 1.3, 0.05])
    grad = lambda th: -2.0 * (th - target) * np.array([1.0, 0.5, 3.0, 10.0])
    theta0 = np.ones(4)
    ref = orc.adam_ascent(orc.softplus_inverse(theta0), grad, steps=60)
    st = AdamState(theta0, lr=0.1)
    for k in range(60):
        th = st.ascend(grad(st.theta))
        assert np.allclose(th, ref[k], rtol=1e-12, atol=1e-14), k
    assert st.k == 60
    # ascent: the objective improved
    f = lambda th: -np.sum(np.array([1.0, 0.5, 3.0, 10.0]) * (th - target) ** 2)
    assert f(st.theta) > f(theta0)


def test_workloads_are_seeded_shaped_and_fp32_representable():
    w1, w1b = make("config1"), make("config1")
    assert (w1.n, w1.d, w1.s) == (2048, 8, 16) and w1.kind == "se" and w1.probe_law == "rademacher"
    assert np.array_equal(w1.X, w1b.X) and np.array_equal(w1.Z, w1b.Z) and np.array_equal(w1.y, w1b.y)
    assert set(np.unique(w1.Z)) == {-1.0, 1.0}
    assert w1.B.shape == (2048, 17) and np.array_equal(w1.B[:, 0], w1.y) and np.array_equal(w1.B[:, 1:], w1.Z)
    for w in (w1, make("config2", n=512), make("config3", n=700), make("config4", n=300), make("config5", n=2000)):
        for arr in (w.X, w.y, w.Z):
            assert np.array_equal(arr, arr.astype(np.float32)), "inputs must be exactly representable in fp32"
        assert abs(float(np.mean(w.y))) < 1e-5 and abs(float(np.std(w.y)) - 1.0) < 1e-3
    w2 = make("config2", n=512)
    assert w2.kind == "matern32" and w2.d == 26 and w2.s == 64 and np.all(w2.ell == 1.0) and w2.tol == 0.01
    assert w2.X.min() >= -1.0 and w2.X.max() <= 1.0 and (w2.ell_truth >= 0.3).all() and (w2.ell_truth <= 3.0).all()
    w5 = make("config5", n=4000)
    rows = {r.tobytes() for r in np.ascontiguousarray(w5.X)}
    assert 4000 - len(rows) >= 150          # about 5 % of the rows are copies of other rows
    assert make("config5", n=4000, seed=7).X[0, 0] != w5.X[0, 0]


def _bench():
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_flop_accounting_of_the_benchmark():
    b = _bench()
    # reporting convention: 2d + 2t + c_phi per pair, c = 4 (SE) / 8 (Matern-3/2)
    assert b.kmv_flops(16384, 26, 65, "matern32") == 16384.0 ** 2 * 190
    assert b.kmv_flops(2_000_000, 11, 65, "se") == 4.0e12 * 156
    # matrix-core flops really issued: on fp16 paths distances in instructions of 32 slots, 3 products per column of the tiles of 16
    assert b.executed_mfma_flops(16384, 26, 65, "matern32", 1) == 16384.0 ** 2 * (3 * 2 * 32 + 3 * 2 * 64)
    assert b.executed_mfma_flops(1000, 11, 65, "se", 2) == 1.0e6 * (6 * 2 * 16 + 3 * 2 * 64)
    assert b.executed_mfma_flops(1000, 11, 65, "se", 1, rows=10) == 1.0e4 * (2 * 2 * 32 + 3 * 2 * 64)
    assert b.executed_mfma_flops(1000, 8, 17, "se", 1) == 1.0e6 * (1 * 2 * 32 + 3 * 2 * 16)
    assert b.executed_mfma_flops(1000, 26, 113, "matern32", 1) == 1.0e6 * (2 * 3 * 2 * 32 + 3 * 2 * 112)
    assert b.executed_mfma_flops(2048, 8, 17, "se", 0) == 2048.0 ** 2 * (2 * 2 * 7 + 2 * 32)
