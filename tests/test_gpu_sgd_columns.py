"""gp_sgd_solve with one workgroup per column (on the fp16 product paths, n <= 81920, or 131072 with one or more than 64
columns) at the edges of the column lengths and batch sizes its kernels are built for, and just past them: the oracle's step run on exact rows of the same problem."""
import numpy as np
import pytest

from oracle import gp_oracle as orc
from tests.gpu_util import Dev

pytestmark = pytest.mark.gpu


def _reference(X, ell, a, sigma, kind, B, batches, X0, lr, momentum):
    """The step of the paper with the mini-batch rows of H evaluated exactly (fp64); for n too large for a dense H."""
    B = B.astype(np.float64)
    U = np.zeros_like(B) if X0 is None else X0.astype(np.float64)
    M = np.zeros_like(B)
    for I in batches:
        G = orc.kmv_rows(X, ell, a, kind, U, I, sigma=sigma) - B[I]
        M *= momentum
        M[I] -= lr / len(I) * G
        U = U + M
    return U


@pytest.mark.parametrize("n,t,batch", [(1, 1, 1), (33, 2, 7), (4096, 17, 257), (4097, 33, 1000), (8193, 66, 31), (16384, 65, 1000),
                                       (16385, 9, 1025), (20003, 1, 64), (40001, 17, 1500), (131072, 2, 100), (131073, 2, 100),
                                       (81920, 2, 100), (81921, 64, 50), (131072, 1, 100), (131072, 65, 40)])
@pytest.mark.parametrize("kind", ["se", "matern32"])
def test_iterates_follow_the_step(n, t, batch, kind):
    rng = np.random.default_rng(n + t)
    d = 4
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    B = rng.standard_normal((n, t)).astype(np.float32)
    X0 = (0.2 * rng.standard_normal((n, t))).astype(np.float32)
    ell = np.full(d, 0.5)
    steps = 3
    batches = np.stack([rng.permutation(n)[:batch] for _ in range(steps)]).astype(np.int32)
    lr = 0.3 * batch / max(1.0, batch * 0.2)
    dv = Dev(X, kind, ell, 0.9, 0.8)
    try:
        for x0 in (None, X0):
            print(f"[sgd columns] n={n} t={t} batch={batch} warm={x0 is not None}", flush=True)
            ref = _reference(X, ell, 0.9, 0.8, kind, B, batches, x0, lr, 0.9)
            rc, iters, kmv, relres, Vd = dv.sgd_solve(B, 1e-7, batches, lr, 0.9, X0=None if x0 is None else dv.to(x0))
            V = Vd.cpu().numpy().astype(np.float64)
            assert iters == steps and kmv == (x0 is not None)
            err = np.linalg.norm(V - ref, axis=0) / np.linalg.norm(ref, axis=0)
            assert err.max() <= 1e-4, err.max()
        V1 = Vd.clone()
        _, _, _, _, V2 = dv.sgd_solve(B, 1e-7, batches, lr, 0.9, X0=dv.to(X0))
        assert bool((V1 == V2).all())
    finally:
        dv.close()


def _stopping_run(X, ell, a, sigma, kind, B, batches, lr, momentum, stop):
    """Column c of the step above stops behind step stop[c] (0: at the start, -1: a zero right-hand side, stops there too;
    past the last batch: never).  Returns the iterates, the final residual estimates and tolerances that the
    estimates first pass at those steps, half-way between the smallest before and the one that passes."""
    B = B.astype(np.float64)
    U, M, R = np.zeros_like(B), np.zeros_like(B), B.copy()
    norm = np.where(stop < 0, 1.0, np.linalg.norm(B, axis=0))
    live = stop > 0
    est = np.where(stop < 0, 0.0, 1.0)
    tol = np.where(stop <= 0, 2.0, 1e-7)
    for k, I in enumerate(batches, 1):
        if not live.any():
            break
        G = orc.kmv_rows(X, ell, a, kind, U, I, sigma=sigma) - B[I]
        M *= momentum
        M[I] -= lr / len(I) * G
        U[:, live] += M[:, live]
        R[np.ix_(I, live)] = -G[:, live]
        now = np.linalg.norm(R, axis=0) / norm
        ends = live & (stop == k)
        assert (now[ends] < 0.999 * est[ends]).all()      # the estimates of the live columns fall
        tol[ends] = 0.5 * (now[ends] + est[ends])
        est = np.where(live, now, est)
        live &= ~ends
    return U, est, tol


@pytest.mark.parametrize("n,t,batch,d", [
    (16384, 9, 2500, 2),        # the register form, for comparison
    (16385, 1, 2500, 3), (17000, 9, 2501, 2), (20003, 34, 3000, 2)])
def test_columns_stop_at_their_own_steps(n, t, batch, d):
    """Columns that stop at every step of the solve, the last one ending it: a stopping column has its whole update, every
    row of it, although its stop (and the end of the solve) is published while the workgroup is still at work."""
    rng = np.random.default_rng(n + t)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    steps = 6
    stop = 3 + rng.permutation(t) % (steps - 2)           # the estimates need two steps to move
    if t > 2:
        stop[1], stop[t - 1] = 0, -1
    B = np.cos(X.astype(np.float64) @ rng.uniform(-2.0, 2.0, size=(d, t)) + rng.uniform(0.0, 3.0, size=t)).astype(np.float32)
    B[:, stop < 0] = 0.0
    batches = np.stack([rng.permutation(n)[:batch] for _ in range(steps)]).astype(np.int32)
    ell, lr = np.full(d, 0.5), 0.5
    ref, est, tol = _stopping_run(X, ell, 0.9, 0.8, "se", B, batches, lr, 0.9, stop)
    dv = Dev(X, "se", ell, 0.9, 0.8)
    try:
        for limit in (steps, int(stop.max()) - 1):        # to the end of the solve, and one step short of it
            print(f"[sgd columns] stops n={n} t={t} batch={batch} limit={limit}", flush=True)
            rc, iters, kmv, relres, Vd = dv.sgd_solve(B, tol, batches, lr, 0.9, max_iters=limit)
            assert (rc, iters, kmv) == ((0, stop.max(), 0) if limit == steps else (1, limit, 0))
            V = Vd.cpu().numpy().astype(np.float64)
            done = (stop > 0) & (stop <= limit)
            err = np.linalg.norm(V - ref, axis=0)[done] / np.linalg.norm(ref, axis=0)[done]
            assert err.max(initial=0.0) <= 1e-4, err.max()           # as above; one wave's rows left out of one step are 1e-2
            assert np.abs(relres[done] / est[done] - 1.0).max(initial=0.0) <= 1e-4
            assert not V[:, stop <= 0].any()
    finally:
        dv.close()
