"""Squared norms of the column solvers: no small term lost behind a large one.

A thread of the solvers' start kernels adds up every 4096th group of four rows.  The right-hand side is 1 in the first
such groups and 4.4e-4 after them: an fp32 sum that has reached 4 drops each later square (2e-7, half an ulp of 4 is 2.4e-7),
an fp64 sum keeps them.  x0 takes the ones away, so that the relative residual a solver reports at its start,

    ||b - H x0|| / ||b||,   H = I up to 1e-16,

has a norm of small terms alone above one of both.  The bound of 2e-7 is three half-ulps of fp32: the rounding of the
result and of the sums of four.  With the squares of a thread's rows in one fp32 chain the error is 4e-7 to 1.6e-6."""
import numpy as np
import pytest

from tests.gpu_util import Dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("solver,n,t", [("cg", 65536, 2), ("cg", 16384, 3), ("sgd", 131072, 1), ("sgd", 65536, 3), ("ap", 65536, 130)])
def test_start_residual(solver, n, t):
    rng = np.random.default_rng(n)
    X = rng.uniform(-1.0, 1.0, size=(n, 2)).astype(np.float32)
    big = np.arange(n) % 65536 < 4096
    if solver == "ap":
        big = np.arange(n) % 32768 < 4096     # two parts of a column
    small = np.float32(4.4e-4)
    B = np.repeat(np.where(big, np.float32(1.0), small)[:, None], t, axis=1)
    X0 = np.repeat(np.where(big, np.float32(1.0), np.float32(0.0))[:, None], t, axis=1)
    ref = np.sqrt(float(small) ** 2 * (~big).sum() / (big.sum() + float(small) ** 2 * (~big).sum()))
    dv = Dev(X, "se", np.full(2, 0.5), 1e-8, 1.0)
    try:
        print(f"[column sums] {solver} n={n} t={t}", flush=True)
        x0 = dv.to(X0)
        if solver == "cg":
            relres = dv.solve(B, 1e-6, max_iters=0, X0=x0)[3]
        elif solver == "ap":
            relres = dv.ap_solve(B, 1e-6, 2000, max_iters=0, X0=x0)[3]
        else:
            relres = dv.sgd_solve(B, 1e-6, np.zeros((1, 1), np.int32), 1e-3, max_iters=0, X0=x0)[3]
        assert np.abs(np.asarray(relres, dtype=np.float64) / ref - 1.0).max() <= 2e-7
    finally:
        dv.close()
