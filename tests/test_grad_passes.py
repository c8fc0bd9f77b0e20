"""Tile passes of a gradient over its probes, counted on the stand-in for the HIP runtime: as few as blocks of 80 allow.

A pass works out distances and kernel values of all pairs again.  With 65 to 79 probes the time of a second pass, over no more
than 16 of them, was up to that of the first."""
import subprocess
import sys

import pytest

from paper_2405_18328_amd.build import LIB
from tests.test_solver_errors import runtime  # noqa: F401

COUNT = r"""
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
n, d, i64, p = 300, int(sys.argv[3]), C.c_int64, C.c_void_p
ctx, X = p(), (C.c_float * (n * d))()
assert lib.gp_create(C.byref(ctx), 1, i64(n), d, X, None) == 0
assert lib.gp_set_theta(ctx, (C.c_double * d)(*[1.0] * d), C.c_double(1), C.c_double(0.5)) == 0
g = (C.c_double * (d + 2))()
for t in map(int, sys.argv[4:]):
    V, B = (C.c_float * (n * t))(), (C.c_float * (n * t))()
    fake.fake_launched()
    assert lib.gp_mll_grad(ctx, V, i64(t), B, i64(t), t, g) == 0
    print(t, fake.fake_launched())
"""


@pytest.mark.parametrize("d", [5, 40])
def test_a_pass_for_every_eighty_probes(runtime, d):  # noqa: F811
    ts = [1, 2, 17, 65, 66, 80, 81, 82, 97, 146, 161, 162, 241, 242]
    r = subprocess.run([sys.executable, "-c", COUNT, runtime, LIB, str(d), *map(str, ts)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    got = {int(a): int(b) for a, b in (line.split() for line in r.stdout.splitlines())}
    per_pass = got[82] - got[81]
    assert per_pass > 2
    for t in ts:
        passes = max(1, -(-(t - 1) // 80))
        assert got[t] == got[1] + (passes - 1) * per_pass, (t, got)
