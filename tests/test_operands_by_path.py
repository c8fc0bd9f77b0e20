"""Operands of the three product paths: allocated and packed for the paths that thetas and predictions ask for, and no others.

On the CPU: device memory of a context, counted on the stand-in for the HIP runtime.  On the GPU: one context led from path to path,
by thetas and by test inputs: products and gradients bit for bit those of a new context, and products and predictions within the
parity tests' bar of exact fp64 sums."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2405_18328_amd.build import LIB
from tests.test_solver_errors import RUNTIME

MEMORY = r"""
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
fake.fake_total.restype = C.c_size_t
fake.fake_memory.restype = C.c_size_t
lib.gp_last_error.restype = C.c_char_p
i64, p = C.c_int64, C.c_void_p
kind, n, d, path = map(int, sys.argv[3:7])
X, V, O = (C.c_float * (n * d))(), (C.c_float * n)(), (C.c_float * n)()
ctx = p()
assert lib.gp_create(C.byref(ctx), kind, i64(n), d, X, None) == 0
theta = lambda: lib.gp_set_theta(ctx, (C.c_double * d)(*[1.0] * d), C.c_double(1), C.c_double(0.5))
created = fake.fake_total()
if path:      # memory is refused once: the theta is, too, and leaves no error behind for the next
    fake.fake_memory(C.c_size_t(1 << 14))
    assert theta() == -2 and b"operands" in lib.gp_last_error(ctx), lib.gp_last_error(ctx)
    assert lib.gp_kmv(ctx, V, i64(1), 1, O, i64(1), 0) == -1
    fake.fake_memory(C.c_size_t(~0 & (1 << 63) - 1))
assert theta() == 0, lib.gp_last_error(ctx)
first = fake.fake_total()
assert theta() == 0 and fake.fake_total() == first
assert lib.gp_product_path(ctx) == {0: 1, 1: 0, 2: 2}[path]
print(created / n, first / n)
"""


@pytest.fixture(scope="module")
def counting_runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("counting")
    code = RUNTIME.replace("  if (n > most) most = n;\n", "  if (n > most) most = n;\n  total += n;\n").replace(
        "static size_t limit =", "static size_t total;\nsize_t fake_total() { return total; }      // bytes allocated so far\nstatic size_t limit =")
    assert code.count("total") == 3 + 1
    (d / "fake.cpp").write_text(code)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", str(d / "fake.cpp"),
                    "-o", str(d / "fake.so")], check=True)
    return str(d / "fake.so")


def _bytes(runtime, kind, n, d, path, env):
    e = dict(os.environ, OMP_NUM_THREADS="1", **({"GPWS_PATH": env} if env else {}))
    r = subprocess.run([sys.executable, "-c", MEMORY, runtime, LIB, str(kind), str(n), str(d), str(path)], capture_output=True, text=True,
                       timeout=60, env=e)
    assert r.returncode == 0, r.stderr[-2000:]
    return map(float, r.stdout.split())


@pytest.mark.parametrize("kind,d", [(0, 3), (0, 11), (1, 26), (1, 90), (1, 125)])
def test_memory_of_a_context(counting_runtime, kind, d):
    """A point's operands for fp16 on two pieces are 64 bytes per side and group of 32 slots for products (dist_f16.h) and
    2 x 32 for every 16 components of the gradient's, and its scaled row; three pieces and fp32 come on top when they are asked for."""
    n = 65536
    comps = d + 2 + (kind == 0)
    kh = next(b for b in (1, 2, 3, 4, 6, 8) if 16 * b >= comps)
    groups = {3: (1, 2), 11: (2, 3), 26: (2, 3), 90: (6, 9), 125: (8, 12)}[d]
    two = 2 * 64 * groups[0] + 4 * 32 * kh + 4 * d + 4
    fixed = ((1 << 22) + (1 << 14)) / n           # reductions and words that do not grow with n
    created, asked = _bytes(counting_runtime, kind, n, d, 0, "")
    assert created <= two + fixed and asked == created
    created, asked = _bytes(counting_runtime, kind, n, d, 2, "f16x3")
    assert created <= two + fixed and abs(asked - created - (2 * 64 * groups[1] + 2 * 32 * kh)) <= 0.1
    created, asked = _bytes(counting_runtime, kind, n, d, 1, "fp32")
    ks = next(b for b in (4, 7, 10, 14, 24, 46, 64) if 2 * b >= d + 2)
    assert created <= two + fixed and abs(asked - created - 2 * 8 * ks) <= 0.1


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["se", "matern32"])
@pytest.mark.parametrize("n,d,t", [(700, 5, 17), (1500, 26, 40)])
def test_one_context_from_path_to_path(kind, n, d, t):
    from oracle import gp_oracle as orc
    from tests.gpu_util import Dev, relerr
    rng = np.random.default_rng(n + d)
    X = rng.uniform(-1.0, 1.0, size=(n, d)).astype(np.float32)
    V, B = (rng.standard_normal((n, t)).astype(np.float32) for _ in range(2))
    near = rng.uniform(-1.0, 1.0, size=(77, d)).astype(np.float32)
    far, farther = near.copy(), near.copy()
    # scaled squared norms: d / 3 / ell^2 on average
    ells = [0.6 * np.sqrt(d), 0.1, 0.02 / np.sqrt(d), 0.2, 0.6 * np.sqrt(d), 0.004, 0.1, 0.6 * np.sqrt(d)]
    far[::2] *= 12.0 / np.sqrt(d / 3)
    farther[::2] *= 300.0
    dv = Dev(X, kind, np.full(d, 1.0), 1.1, 0.4)
    paths = []
    try:
        Vd, Bd = dv.to(V), dv.to(B)
        for step, e in enumerate(ells):
            ell = np.full(d, e) * rng.uniform(0.9, 1.1, size=d)
            dv.set_theta(ell, 1.1, 0.4)
            paths.append(dv.gp.gp_product_path(dv.ctx))
            print(f"[path] {kind} n={n} d={d} step {step} ell {e:.4g} path {paths[-1]}", flush=True)

            new = Dev(X, kind, ell, 1.1, 0.4)
            fresh = new.kmv(V, 1), new.grad(Vd, Bd)
            new.close()
            assert relerr(fresh[0], orc.kmv_dense(X, ell, 1.1, kind, V, sigma=0.4)) <= 1e-5

            def check():
                assert np.array_equal(dv.kmv(V, 1), fresh[0]) and np.array_equal(dv.grad(Vd, Bd), fresh[1])
            if step % 2:
                check()
            if e > 0.5:      # rows of test inputs that ask for the other paths
                for Xs in (near, farther, far, near):
                    assert relerr(dv.predict(Xs, V), orc.cross_kmv(Xs, X, ell, 1.1, kind, V)) <= 1e-5
            check()
    finally:
        dv.close()
    assert set(paths) == {0, 1, 2}, paths
