"""gp_ap_solve with one workgroup per column (n <= 65536 and at most 256 blocks on the fp16 product paths) at the edges of
its block counts, column lengths and column counts, and past them, where the general kernels take over: the same step in
fp64 on exactly evaluated blocks of H, following the library's block choices and checking each of them."""
import numpy as np
import pytest
import scipy.linalg as sla

from oracle import gp_oracle as orc
from tests.gpu_util import Dev

pytestmark = pytest.mark.gpu


def _follow(X, ell, a, sigma, kind, B, X0, block, picks):
    """Solution after the block updates `picks`, and the worst ratio of a chosen block's score to the best one's."""
    Bf = B.astype(np.float64)
    n = B.shape[0]
    V = np.zeros_like(Bf) if X0 is None else X0.astype(np.float64)
    R = Bf.copy()
    if X0 is not None:
        for j in range(0, n, 4096):
            R[j:j + 4096] -= orc.kmv_rows(X, ell, a, kind, V, np.arange(j, min(n, j + 4096)), sigma=sigma)
    starts = np.arange(0, n, block)
    worst = 1.0
    for k in picks:
        score = np.add.reduceat((R * R).sum(axis=1), starts)
        worst = min(worst, score[k] / score.max())
        j0, j1 = k * block, min(n, (k + 1) * block)
        H = orc.kernel_cross(X, X[j0:j1], ell, a, kind)
        H[np.arange(j0, j1), np.arange(j1 - j0)] += sigma ** 2
        delta = sla.cho_solve(sla.cho_factor(H[j0:j1], lower=True), R[j0:j1])
        V[j0:j1] += delta
        R -= H @ delta
    return V, np.linalg.norm(R, axis=0) / np.linalg.norm(Bf, axis=0), worst


@pytest.mark.parametrize("n,block,t,warm", [
    (1, 1, 1, True), (256, 1, 2, True), (257, 1, 2, True), (1024, 4, 17, False), (1025, 4, 17, False), (4096, 1000, 48, True),
    (4097, 33, 49, True), (8193, 2000, 80, False), (8200, 500, 81, True), (16385, 1000, 1, False), (65536, 256, 3, False),
    (65537, 300, 3, False)])
def test_steps_follow_the_projection(n, block, t, warm):
    rng = np.random.default_rng(n + t)
    d, kind = 4, "matern32" if n % 2 else "se"
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    B = rng.standard_normal((n, t)).astype(np.float32)
    X0 = (0.05 * rng.standard_normal((n, t))).astype(np.float32) if warm else None
    ell, a, sigma = np.full(d, 0.5), 0.9, 0.8
    dv = Dev(X, kind, ell, a, sigma)
    try:
        print(f"[ap columns] n={n} block={block} t={t} warm={warm}", flush=True)
        rc, iters, kmv, relres, picks, Vd = dv.ap_solve(B, 1e-12, block, max_iters=3, picks=True, X0=None if X0 is None else dv.to(X0))
        assert iters == len(picks) and 1 <= iters <= 3 and kmv == warm
        assert iters == 3 or n <= block         # a single block is a direct solve: nothing may be left after one step
        V, rr, worst = _follow(X, ell, a, sigma, kind, B, X0, block, picks)
        assert worst >= 1.0 - 1e-3              # a choice that fp32 residuals cannot tell from the best one
        err = np.linalg.norm(Vd.cpu().numpy() - V, axis=0) / np.linalg.norm(V, axis=0)
        assert err.max() <= 1e-4, err.max()
        assert np.abs(relres - rr).max() <= 2e-3 * rr.max() + 2e-5
    finally:
        dv.close()


def _stopping_run(H, B, block, stop):
    """Column c stops behind the first step from stop[c] on whose residual is its smallest so far (stop < 0: a zero right-hand
    side).  Returns V, the residuals, tolerances half-way between that residual and the smallest before it, and the choices."""
    n, t = B.shape
    starts = np.arange(0, n, block)
    V, R = np.zeros((n, t)), B.astype(np.float64)
    norm = np.where(stop < 0, 1.0, np.linalg.norm(R, axis=0))
    live = stop >= 0
    least = np.where(live, 1.0, 0.0)
    rr, tol, picks = least.copy(), np.full(t, 2.0), []
    while live.any():
        score = np.add.reduceat((R[:, live] ** 2).sum(axis=1), starts)
        k = int(np.argmax(score))
        assert np.sort(score)[-2] <= (1.0 - 1e-4) * score[k]       # a choice that fp32 residuals cannot turn
        j0, j1 = k * block, min(n, (k + 1) * block)
        D = np.linalg.solve(H[j0:j1, j0:j1], R[j0:j1][:, live])
        V[j0:j1, live] += D
        R[:, live] -= H[:, j0:j1] @ D
        picks.append(k)
        now = np.linalg.norm(R, axis=0) / norm
        ends = live & (len(picks) >= stop) & (now < (1.0 - 1e-4) * least)
        tol[ends] = 0.5 * (now[ends] + least[ends])
        rr = np.where(live, now, rr)
        least = np.where(live, np.minimum(least, now), least)
        live &= ~ends
    return V, rr, tol, picks


@pytest.mark.parametrize("n,block,t", [(2000, 50, 70), (2010, 48, 70), (2000, 20, 70), (2005, 10, 40), (1200, 9, 300)])
def test_columns_stop_at_their_own_steps(n, block, t):
    """Columns that stop all through a solve, over block counts on both sides of the two ways to end a step (40 blocks), with
    the block norms of all columns staged at once or a few columns at a time."""
    rng = np.random.default_rng(n + t)
    d = 3
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    X = X[np.argsort(X[:, 0])]                            # neighbours share a block: the residuals fall quickly
    B = np.cos(X.astype(np.float64) @ rng.uniform(-2.0, 2.0, size=(d, t)) + rng.uniform(0.0, 3.0, size=t)).astype(np.float32)
    stop = 1 + rng.permutation(t) % 20
    stop[t - 1], B[:, t - 1] = -1, 0.0
    ell = np.full(d, 0.5)
    H = orc.coefficient_matrix(X, ell, 0.9, 0.5, "matern32")
    ref, rr, tol, want = _stopping_run(H, B, block, stop)
    dv = Dev(X, "matern32", ell, 0.9, 0.5)
    try:
        print(f"[ap columns] stops n={n} block={block} t={t} steps={len(want)}", flush=True)
        rc, iters, kmv, relres, picks, Vd = dv.ap_solve(B, tol, block, max_iters=len(want) + 5, picks=True)
        assert (rc, iters, kmv) == (0, len(want), 0) and list(picks) == want
        V = Vd.cpu().numpy().astype(np.float64)
        assert not V[:, t - 1].any()
        err = np.linalg.norm(V - ref, axis=0)[:-1] / np.linalg.norm(ref, axis=0)[:-1]
        assert err.max() <= 1e-4, err.max()
        assert np.abs(relres - rr).max() <= 1e-4
    finally:
        dv.close()
