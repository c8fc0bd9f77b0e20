"""gp_kmv_static, the K V entry point for callers that cannot allocate: same results as gp_kmv.

Two calls in a row through the C ABI, the second on a smaller problem (the file-scope scratch then
still holds the first call's contents), each compared bit for bit with gp_kmv (same kernels, no
atomics on floats) and with the fp64 oracle at the 1e-5 normwise bar of the K V parity tests; a product
whose scratch would not fit is refused before anything is launched.  Collected last on purpose.
"""
import numpy as np
import pytest
import torch

from oracle import gp_oracle as orc
from paper_2405_18328_amd import binding as gp
from paper_2405_18328_amd.inputs import make
from tests.gpu_util import Dev, relerr

pytestmark = pytest.mark.gpu

KMV_TOL = 1e-5


def _both(dv, w, add_noise):
    """(gp_kmv_static output, gp_kmv output) on the workload's right-hand sides, padded leading dimensions."""
    t = w.s + 1
    ldv, ldo = t + 3, t + 2
    Vd = torch.full((w.n, ldv), float("nan"), device=dv.dev)
    Vd[:, :t] = dv.to(w.B)
    outs = []
    for fn in (gp.gp_kmv_static, gp.gp_kmv):
        out = torch.full((w.n, ldo), -777.0, device=dv.dev)
        print(f"[no-alloc] {fn.__name__} n={w.n} d={w.d} t={t} kind={w.kind}", flush=True)
        fn(dv.ctx, Vd, ldv, t, out, ldo, add_noise)
        torch.cuda.synchronize()
        o = out.cpu().numpy()
        assert (o[:, t:] == -777.0).all(), "padding columns of the output were written"
        outs.append(o[:, :t])
    return outs


def test_static_scratch_product_equals_gp_kmv_twice_in_a_row_second_call_smaller():
    cases = [("config2", dict(n=6000, s=64)),     # Matern-3/2, d = 26, t = 65: column-split partials, two N-tiles + y column
             ("config1", dict(n=1500, s=16)),     # SE, d = 8, t = 17: smaller in every dimension than the call before
             ("config2", dict(n=6000, s=64))]     # and the larger one again over what the small one left
    for name, kw in cases:
        w = make(name, **kw)
        dv = Dev(w.X, w.kind, w.ell, w.a, w.sigma)
        try:
            got, ref_gpu = _both(dv, w, 1)
            assert np.array_equal(got, ref_gpu), "gp_kmv_static differs from gp_kmv"
            ref = orc.kmv_dense(w.X, w.ell, w.a, w.kind, w.B, sigma=w.sigma)
            assert relerr(got, ref) <= KMV_TOL
            # a second call on the same context, without the noise term, reusing the scratch at once
            got0, ref0 = _both(dv, w, 0)
            assert np.array_equal(got0, ref0)
            assert relerr(got0, orc.kmv_dense(w.X, w.ell, w.a, w.kind, w.B)) <= KMV_TOL
        finally:
            dv.close()


def test_static_scratch_product_on_every_product_path(monkeypatch):
    w = make("config3", n=3000, s=8)
    for path in ("fp32", "f16x2", "f16x3"):
        monkeypatch.setenv("GPWS_PATH", path)
        dv = Dev(w.X, w.kind, w.ell, w.a, w.sigma)
        try:
            got, ref_gpu = _both(dv, w, 1)
            assert np.array_equal(got, ref_gpu), path
            assert relerr(got, orc.kmv_dense(w.X, w.ell, w.a, w.kind, w.B, sigma=w.sigma)) <= KMV_TOL
        finally:
            dv.close()


def test_static_scratch_product_refuses_what_does_not_fit_and_bad_arguments():
    n, d, t = 300000, 3, 65      # the packed images of V alone take 77 MB here (256 bytes per row)
    X = torch.zeros((n, d), device="cuda:0")
    ctx = gp.gp_create(gp.GP_SE_ARD, n, d, X, torch.cuda.current_stream().cuda_stream)
    try:
        gp.gp_set_theta(ctx, np.ones(d), 1.0, 0.1)
        V = torch.zeros((n, t), device="cuda:0")
        out = torch.full((n, t), 5.0, device="cuda:0")
        with pytest.raises(gp.GpError) as e:
            gp.gp_kmv_static(ctx, V, t, t, out, t, 1)
        assert e.value.code == gp.GP_ERR_WORKSPACE and "static" in str(e.value)
        torch.cuda.synchronize()
        assert (out == 5.0).all(), "a refused call wrote its output"
        with pytest.raises(gp.GpError) as e:
            gp.gp_kmv_static(ctx, V, t, t, V, t, 0)
        assert e.value.code == gp.GP_ERR_ARG
        with pytest.raises(gp.GpError) as e:
            gp.gp_kmv_static(ctx, V, t - 1, t, out, t, 0)
        assert e.value.code == gp.GP_ERR_ARG
    finally:
        gp.gp_destroy(ctx)


@pytest.mark.parametrize("n,d,kind,t", [
    (131073, 26, "matern32", 97),     # two column passes, the second without the vector-ALU column, on two kernels
    (70001, 26, "matern32", 34),      # wide kernel, a ragged last panel
    (131073, 12, "se", 65),           # one row past a full generation of workgroups
    (150000, 3, "se", 65), (230000, 26, "se", 17), (240001, 2, "matern32", 66)])
def test_static_scratch_product_whose_partial_images_do_not_fit(n, d, kind, t):
    """Sizes whose column splits leave more partial images than the static scratch holds: row panels, the same bits."""
    rng = np.random.default_rng(n)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    V = rng.standard_normal((n, t)).astype(np.float32)
    dv = Dev(X, kind, np.full(d, 0.6 * np.sqrt(d)), 0.9, 0.5)
    try:
        Vd = dv.to(V)
        outs, launches = [], []
        for fn in (gp.gp_kmv_static, gp.gp_kmv):
            out = torch.full((n, t + 1), -777.0, device=dv.dev)
            print(f"[no-alloc] {fn.__name__} n={n} d={d} t={t}", flush=True)
            gp.gp_profile(dv.ctx, 1 << gp.GP_PROF_TILE)
            fn(dv.ctx, Vd, t, t, out, t + 1, 1)
            launches.append(gp.gp_profile_read(dv.ctx)[0])
            gp.gp_profile(dv.ctx, 0)
            outs.append(out)
        assert launches[0] > launches[1], launches         # the panels were taken
        assert torch.equal(outs[0], outs[1]), "gp_kmv_static differs from gp_kmv"
        got = outs[0].cpu().numpy()
        assert (got[:, t:] == -777.0).all()
        rows = np.unique(np.r_[0, 255, 256, n - 1, rng.integers(0, n, 60)])
        ref = orc.kmv_rows(X, np.full(d, 0.6 * np.sqrt(d)), 0.9, kind, V, rows, sigma=0.5)
        assert relerr(got[rows, :t], ref) <= KMV_TOL
    finally:
        dv.close()


@pytest.mark.parametrize("n,d,t", [(3000, 26, 65), (20000, 3, 17), (131073, 3, 66)])
def test_static_scratch_product_in_a_captured_graph(n, d, t):
    """Recorded once and replayed on changing vectors, with eager products on the same scratch between the replays; the last
    size works in panels of rows."""
    rng = np.random.default_rng(n)
    X = torch.from_numpy(rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)).to("cuda:0")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ctx = gp.gp_create(gp.GP_SE_ARD, n, d, X, stream.cuda_stream)
        try:
            gp.gp_set_theta(ctx, np.full(d, 0.6 * np.sqrt(d)), 0.9, 0.5)
            V = torch.randn(n, t, device="cuda:0")
            out, want = torch.empty_like(V), torch.empty_like(V)
            gp.gp_kmv_static(ctx, V, t, t, out, t, 1)
            gp.gp_kmv(ctx, V, t, t, want, t, 1)
            torch.cuda.synchronize()
            print(f"[no-alloc] capture n={n} d={d} t={t}", flush=True)
            graph = torch.cuda.CUDAGraph()
            graph.capture_begin()
            gp.gp_kmv_static(ctx, V, t, t, out, t, 1)
            graph.capture_end()
            for _ in range(3):
                V.copy_(torch.randn(n, t, device="cuda:0"))
                out.fill_(float("nan"))
                gp.gp_kmv_static(ctx, V, t, t, want, t, 0)      # another product over the shared scratch
                gp.gp_kmv(ctx, V, t, t, want, t, 1)
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(out, want)
            del graph
        finally:
            torch.cuda.synchronize()
            gp.gp_destroy(ctx)
