"""Packing of points, as its launches look on the stand-in for the HIP runtime."""
import os
import subprocess
import sys

import pytest

from paper_2405_18328_amd.build import LIB
from tests.test_solver_errors import runtime  # noqa: F401

HEAD = r"""
import ctypes as C, os, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
fake.fake_threads.restype = C.c_ulonglong
lib.gp_last_error.restype = C.c_char_p
i64, p = C.c_int64, C.c_void_p
def create(kind, n, d, X):
    ctx = p()
    assert lib.gp_create(C.byref(ctx), kind, i64(n), d, X, None) == 0
    assert lib.gp_set_theta(ctx, (C.c_double * d)(*[1.0] * d), C.c_double(1), C.c_double(0.5)) == 0, lib.gp_last_error(ctx)
    return ctx
"""

LARGE = HEAD + r"""
few = (C.c_float * 64)()                 # no kernel runs: nothing behind the pointers is read
ctx = create(0, (1 << 29) + 33, 1, few)
assert 0 < fake.fake_threads() < 1 << 32
sys.stdout.flush()
os._exit(0)
"""

LARGE_PREDICT = HEAD + r"""
few = (C.c_float * 64)()
ctx = create(0, 64, 1, few)
fake.fake_threads()
assert lib.gp_predict(ctx, few, i64(1 << 30), few, i64(1), 1, few, i64(1)) == 0, lib.gp_last_error(ctx)
assert 0 < fake.fake_threads() < 1 << 32
sys.stdout.flush()
os._exit(0)
"""


def _run(runtime, code, *args, **env):  # noqa: F811
    r = subprocess.run([sys.executable, "-c", code, runtime, LIB, *map(str, args)], capture_output=True, text=True, timeout=60,
                       env=dict(os.environ, OMP_NUM_THREADS="1", **env))
    assert r.returncode == 0, r.stderr[-2000:]


def test_no_launch_of_more_than_two_to_the_32_threads(runtime):  # noqa: F811
    """2^29 points and more have 2^24 chunks of 32: a workgroup of 256 for each is more than one launch may have."""
    _run(runtime, LARGE)
    _run(runtime, LARGE_PREDICT)


WAITS = HEAD + r"""
n, d, m = 300, int(sys.argv[3]), 70
few = (C.c_float * (n * d))()
ctx = create(0, n, d, few)
fake.fake_posting(0)
assert lib.gp_predict(ctx, few, i64(m), few, i64(1), 1, few, i64(1)) == -2
assert b"not reported" in lib.gp_last_error(ctx), lib.gp_last_error(ctx)
"""


@pytest.mark.parametrize("d", [5, 126])
def test_a_prediction_returns_behind_the_packing_of_its_points(runtime, d):  # noqa: F811
    """X* is read during the call only: the call waits for the norm that is posted behind the packing (here: is told that there is
    none), also where the path is settled without it, as in 126 dimensions."""
    _run(runtime, WAITS, d)


SETTLED = HEAD + r"""
n, d, t = 9000, 5, 40
X, V, O = (C.c_float * (n * d))(), (C.c_float * (n * t))(), (C.c_float * (n * t))()
ctx = create(0, n, d, X)
fake.fake_launched()
assert lib.gp_kmv(ctx, V, i64(t), t, O, i64(t), 0) == 0
square = fake.fake_launched()
assert lib.gp_predict(ctx, X, i64(n), V, i64(t), t, O, i64(t)) == 0
assert fake.fake_launched() == square + 2, square       # + points packed, norm posted
"""


def test_a_prediction_whose_path_is_settled_prepares_no_other(runtime):  # noqa: F811
    """On the fp32 path of the training inputs neither the column maxima nor the fp16 operands of V are made."""
    _run(runtime, SETTLED, GPWS_PATH="fp32")
