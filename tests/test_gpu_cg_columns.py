"""gp_cg_solve with one workgroup per column (n <= 65536 on the fp16 product paths) and its neighbours: the oracle's
textbook CG run on the library's own product, at the edges of the column lengths the kernel is built for, of the
column counts that fill or pad the operand tiles, and past the last size, where the streaming kernels take over."""
import numpy as np
import pytest
import torch

from oracle import gp_oracle as orc
from tests.gpu_util import Dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,kind,t", [
    (1, 2, "se", 1), (31, 3, "matern32", 2), (33, 3, "se", 17), (4096, 5, "se", 33), (4097, 8, "matern32", 1),
    (8192, 4, "matern32", 97), (8193, 4, "se", 66), (16384, 26, "matern32", 65), (16385, 26, "se", 9), (40003, 20, "matern32", 17),
    (65536, 9, "se", 3), (65537, 9, "se", 3)])
def test_iterates_follow_the_textbook_recurrence(n, d, kind, t):
    rng = np.random.default_rng(n + t)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    B = rng.standard_normal((n, t)).astype(np.float32)
    X0 = (0.3 * rng.standard_normal((n, t))).astype(np.float32)
    if t > 1:
        B[:, t - 1] = 0.0          # a zero right-hand side: its solution is 0 whatever x0 says
    tol = np.full(t, 1e-6)
    if t > 2:
        tol[1] = 10.0              # stops at the start, and must be left as it is
    ell = np.full(d, 0.3 * np.sqrt(d))
    dv = Dev(X, kind, ell, 0.9, 1.1)
    try:
        def matvec(P):
            Pd = torch.from_numpy(np.ascontiguousarray(P, dtype=np.float32)).to(dv.dev)
            out = torch.empty_like(Pd)
            dv.gp.gp_kmv(dv.ctx, Pd, t, t, out, t, 1)
            torch.cuda.synchronize()
            return out.cpu().numpy().astype(np.float64)

        for x0 in (None, X0):
            print(f"[cg columns] n={n} t={t} warm={x0 is not None}", flush=True)
            Vref, itref, rr = orc.cg_batched(matvec, B, X0=x0, tol=tol, max_iters=3)
            rc, iters, kmv, relres, Vd = dv.solve(B, tol, max_iters=3, X0=None if x0 is None else dv.to(x0))
            V = Vd.cpu().numpy().astype(np.float64)
            assert iters == itref and kmv == iters + (x0 is not None)
            assert rc == (0 if (rr < tol).all() else 1)
            scale = np.linalg.norm(Vref, axis=0)
            err = np.linalg.norm(V - Vref, axis=0) / np.where(scale > 0, scale, 1.0)
            assert err.max() <= 1e-4, err
            live = rr > 1e-5
            assert np.abs(relres[live] / rr[live] - 1.0).max(initial=0.0) <= 1e-3
            if t > 1:
                assert not V[:, t - 1].any()
        # nothing to do: the solution as x0, tolerances it meets
        Vs = Vd.clone()
        rc, iters, _, _, V2 = dv.solve(B, 10.0, max_iters=5, X0=Vs)
        assert rc == 0 and iters == 0 and torch.equal(V2, Vs)
        # and the same again, bit for bit
        _, _, _, _, V3 = dv.solve(B, tol, max_iters=3, X0=dv.to(X0))
        assert torch.equal(V3, Vd)
    finally:
        dv.close()


@pytest.mark.parametrize("n,kinds", [(2000, ("CG_XR",)), (16384, ("CG_XR",)), (16385, ("CG_DOT", "CG_XR")),
                                     (65537, ("CG_DOT", "CG_XR", "CG_P"))])
def test_profile_counts_the_vector_kernels(n, kinds):
    """gp_profile times the vector work of every iteration, whichever kernels do it."""
    rng = np.random.default_rng(n)
    X = rng.uniform(-1.0, 1.0, size=(n, 3)).astype(np.float32)
    B = rng.standard_normal((n, 5)).astype(np.float32)
    dv = Dev(X, "se", np.full(3, 0.5), 0.9, 1.1)
    try:
        print(f"[cg columns] profile n={n}", flush=True)
        dv.gp.gp_profile(dv.ctx, (1 << dv.gp.GP_PROF_KINDS) - 1)
        _, iters, _, _, _ = dv.solve(B, 1e-7, max_iters=4)
        read = {k: dv.gp.gp_profile_read_kind(dv.ctx, getattr(dv.gp, "GP_PROF_" + k)) for k in ("TILE", "CG_DOT", "CG_XR", "CG_P")}
        dv.gp.gp_profile(dv.ctx, 0)
        assert iters == 4
        for k, (launches, ms) in read.items():
            assert launches == (iters if k == "TILE" or k in kinds else 0), read
            assert ms > 0.0 or not launches
    finally:
        dv.close()
