"""The wait for a set of points' largest norm asks the stream now and then, not all the time: a query costs many times what the wait does.

On the stand-in for the HIP runtime, with norms posted 200 us after their launch."""
import os
import subprocess
import sys

from paper_2405_18328_amd.build import LIB
from tests.test_points_host import HEAD
from tests.test_solver_errors import RUNTIME

PREDICT = HEAD + r"""
n, d, m = 300, 5, 70
few = (C.c_float * (n * d))()
ctx = create(0, n, d, few)
fake.fake_queries()
for _ in range(20):
    assert lib.gp_predict(ctx, few, i64(m), few, i64(1), 1, few, i64(1)) == 0, lib.gp_last_error(ctx)
q = fake.fake_queries()
assert q <= 20, q      # none, unless the thread that posts is held up by a millisecond
"""


def test_a_short_wait_does_not_ask_the_stream(tmp_path):
    code = RUNTIME
    for old, new in (("#include <cstdlib>", "#include <chrono>\n#include <cstdlib>\n#include <thread>"),
                     ("if (g.x * b.x == 1 && posting) **(unsigned long long**)args[1] = (unsigned long long)++posts << 32;",
                      "if (g.x * b.x == 1) std::thread([at = *(volatile unsigned long long**)args[1], w = (unsigned long long)++posts << 32] {\n"
                      "    std::this_thread::sleep_for(std::chrono::microseconds(200)); *at = w; }).detach();"),
                     ("hipError_t hipStreamQuery(hipStream_t) {\n", "static int queries;\nint fake_queries() { const int q = queries; queries = 0; return q; }\n"
                      "hipError_t hipStreamQuery(hipStream_t) {\n  ++queries;\n")):
        assert code.count(old) == 1
        code = code.replace(old, new)
    (tmp_path / "fake.cpp").write_text(code)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-pthread", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    str(tmp_path / "fake.cpp"), "-o", str(tmp_path / "fake.so")], check=True)
    r = subprocess.run([sys.executable, "-c", PREDICT, str(tmp_path / "fake.so"), LIB], capture_output=True, text=True, timeout=60,
                       env=dict(os.environ, OMP_NUM_THREADS="1"))
    assert r.returncode == 0, r.stderr[-2000:]
