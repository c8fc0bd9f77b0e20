"""gp_sgd_solve with one workgroup per column (n <= 131072 on the fp16 product paths) at the edges of the column lengths
and batch sizes its kernels are built for: the oracle's step run on exact rows of the same problem."""
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
                                       (16385, 9, 1025), (20003, 1, 64), (40001, 17, 1500), (131072, 2, 100), (131073, 2, 100)])
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
