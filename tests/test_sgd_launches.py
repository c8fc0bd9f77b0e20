"""Launches of a step of the SGD column solver, counted on the stand-in for the HIP runtime."""
import os
import subprocess
import sys

import pytest

from paper_2405_18328_amd.build import LIB
from tests import test_gpu_sgd_columns as columns
from tests.test_solver_errors import runtime  # noqa: F401

STEPS = r"""
import ctypes as C, mmap, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
n, t, batch = map(int, sys.argv[3:6])
lib.gp_sgd_workspace_bytes.restype = C.c_size_t
lib.gp_last_error.restype = C.c_char_p
i64, p = C.c_int64, C.c_void_p
X, B, V = ((C.c_float * (n * k))() for k in (3, t, t))
ctx = p()
assert lib.gp_create(C.byref(ctx), 0, i64(n), 3, X, None) == 0
assert lib.gp_set_theta(ctx, (C.c_double * 3)(1, 1, 1), C.c_double(1), C.c_double(0.5)) == 0
size = lib.gp_sgd_workspace_bytes(ctx, t, batch)
work = mmap.mmap(-1, size + 4096)
at = C.addressof(C.c_char.from_buffer(work))
tol, it, kmv, rel = (C.c_float * t)(*[1e-3] * t), C.c_int(), C.c_int(), (C.c_float * t)()
I = (C.c_int * (batch * 9))()
def launches(steps):
    fake.fake_fail(0)
    fake.fake_launched()
    rc = lib.gp_sgd_solve(ctx, B, i64(t), None, V, i64(t), t, tol, I, batch, steps, C.c_double(1e-3), C.c_double(0.9), p(at), C.c_size_t(size),
                          C.byref(it), C.byref(kmv), rel)
    assert rc == 1, lib.gp_last_error(ctx)
    return fake.fake_launched()
print((launches(9) - launches(3)) / 6)
"""


@pytest.mark.parametrize("t,batch,launches", [(1, 1000, 3), (17, 1000, 3), (48, 1000, 3), (49, 1000, 2), (64, 199, 3), (64, 200, 2),
                                              (64, 2048, 2), (64, 2049, 3)])
def test_the_gradient_goes_along_with_the_step_where_there_are_many_columns(runtime, t, batch, launches):  # noqa: F811
    """One product, one step; the gradient in a launch of its own where a workgroup per column would be the slower way."""
    r = subprocess.run([sys.executable, "-c", STEPS, runtime, LIB, "3000", str(t), str(batch)], capture_output=True, text=True, timeout=60,
                       env=dict(os.environ, OMP_NUM_THREADS="1"))
    assert r.returncode == 0, r.stderr[-2000:]
    assert float(r.stdout) == launches


@pytest.mark.gpu
@pytest.mark.parametrize("n,t,batch", [(1100, 49, 1000), (2049, 64, 2048), (4097, 50, 200), (8193, 66, 1025), (16385, 65, 257)])
def test_iterates_with_the_gradient_in_the_step(n, t, batch):
    """Every form of the step that takes the gradient along: columns of up to 4096, 8192, 16384 rows and of more, with one and more
    rounds of 1024 rows."""
    columns.test_iterates_follow_the_step(n, t, batch, "matern32")


@pytest.mark.gpu
@pytest.mark.parametrize("n,t,batch,d", [(3000, 49, 800, 2), (17000, 66, 2048, 2)])
def test_columns_stop_with_the_gradient_in_the_step(n, t, batch, d):
    columns.test_columns_stop_at_their_own_steps(n, t, batch, d)
