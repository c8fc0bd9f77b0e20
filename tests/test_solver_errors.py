"""A column solver that ends with an error leaves nothing of itself on the stream.

The library runs on a stand-in for the HIP runtime, on the CPU: kernels do nothing, device memory is host memory, and
every query of the stream reports one more finished step in the place the solvers' kernels post to.  The stand-in fails
one runtime call after the other, through a whole solve; whatever was queued before has to be waited for, since a
kernel left over would write to the caller's workspace and post into the next solve.

On the way: the kernels with 1024 threads, of which a compute unit runs one workgroup at a time, are not launched with
a few workgroups more than there are compute units."""
import os
import subprocess
import sys

import pytest

from paper_2405_18328_amd.build import LIB

RUNTIME = r"""
#include <hip/hip_runtime.h>
#include <cstdlib>
#include <cstring>
#include <sys/mman.h>
static char* pinned;
static int queued, launched, until_failure, wide, posts, posting = 1;
static unsigned long long threads;
static unsigned steps;
static hipError_t fallible() { return until_failure > 0 && --until_failure == 0 ? hipErrorUnknown : hipSuccess; }
extern "C" {
int fake_queued() { return queued; }
int fake_launched() { const int n = launched; launched = 0; return n; }      // since the last time it was asked
void fake_posting(int on) { posting = on; }      // off: norms are not posted, and the stream is idle
unsigned long long fake_threads() { const unsigned long long m = threads; threads = 0; return m; }      // most in one dimension of a launch
int fake_wide() { return wide; }      // most workgroups of a launch with 1024 threads each
int fake_fail(int k) { const int left = until_failure; until_failure = k; steps = 0; queued = 0; return left; }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
static dim3 grid, block;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) { grid = g; block = b; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = grid; *b = block; *m = 0; *s = nullptr; return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
  ++queued;
  ++launched;
  if ((unsigned long long)g.x * b.x > threads) threads = (unsigned long long)g.x * b.x;
  // a single thread posts the largest norm, under one tag after the other
  if (g.x * b.x == 1 && posting) **(unsigned long long**)args[1] = (unsigned long long)++posts << 32;
  if (b.x == 1024 && (int)(g.x * g.y) > wide) wide = g.x * g.y;
  return hipSuccess;
}
static size_t limit = ~(size_t)0, most;
static hipError_t last_error = hipSuccess;
size_t fake_memory(size_t l) { const size_t m = most; most = 0; limit = l; return m; }      // most bytes allocated at once since; limit on them
hipError_t hipGetLastError() {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e == hipSuccess ? fallible() : e;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return fallible(); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (fallible() != hipSuccess) return hipErrorUnknown;
  ++queued; memcpy(d, s, n); return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  if (fallible() != hipSuccess) return hipErrorUnknown;
  ++queued; memset(d, v, n); return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) {
  if (!posting) return hipSuccess;
  unsigned long long* post = (unsigned long long*)(pinned + 32768);
  ++steps;
  for (int k = 0; k < 16; ++k) post[k] = steps;
  return hipErrorNotReady;
}
hipError_t hipStreamSynchronize(hipStream_t) { queued = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  if (n > limit) return last_error = hipErrorOutOfMemory;
  if (n > most) most = n;
  if (n >> 33) {      // never freed
    *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return *p == MAP_FAILED ? hipErrorOutOfMemory : hipSuccess;
  }
  *p = calloc(n, 1); return hipSuccess;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = pinned = (char*)calloc(n, 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p)); strcpy(p->gcnArchName, "gfx950"); p->multiProcessorCount = 256; return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stand-in failure"; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
}
"""

CHILD = r"""
import ctypes as C, mmap, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # found before the library's own runtime
lib = C.CDLL(sys.argv[2])
solver, n, t, batch, warm = sys.argv[3], int(sys.argv[4]), 9, 100, int(sys.argv[5])
for f in ("gp_workspace_bytes", "gp_ap_workspace_bytes", "gp_sgd_workspace_bytes"): getattr(lib, f).restype = C.c_size_t
lib.gp_last_error.restype = C.c_char_p
i64, p = C.c_int64, C.c_void_p
X, B, V = ((C.c_float * (n * k))() for k in (3, t, t))
ctx = p()
assert lib.gp_create(C.byref(ctx), 0, i64(n), 3, X, None) == 0
assert lib.gp_set_theta(ctx, (C.c_double * 3)(1, 1, 1), C.c_double(1), C.c_double(0.5)) == 0, lib.gp_last_error(ctx)
size = {"cg": lambda: lib.gp_workspace_bytes(ctx, t), "ap": lambda: lib.gp_ap_workspace_bytes(ctx, t, batch),
        "sgd": lambda: lib.gp_sgd_workspace_bytes(ctx, t, batch)}[solver]()
work = mmap.mmap(-1, size + 4096)                    # page-aligned, and only what is touched takes memory
at = C.addressof(C.c_char.from_buffer(work))
tol, it, kmv, rel = (C.c_float * t)(*[1e-3] * t), C.c_int(), C.c_int(), (C.c_float * t)()
I = (C.c_int * (batch * 6))()
head = (ctx, B, i64(t), V if warm else None, V, i64(t), t, tol)
tail = (p(at), C.c_size_t(size), C.byref(it), C.byref(kmv), rel)
def solve():
    if solver == "cg": return lib.gp_cg_solve(*head, 6, *tail)
    if solver == "ap": return lib.gp_ap_solve(*head, batch, 6, *tail, None)
    return lib.gp_sgd_solve(*head, I, batch, 6, C.c_double(1e-3), C.c_double(0.9), *tail)
assert fake.fake_fail(0) == 0 and solve() == 1, lib.gp_last_error(ctx)     # not converged after 6 steps
assert 0 < fake.fake_wide() <= 256, "%d workgroups of a launch on 256 compute units" % fake.fake_wide()
k = 0
while True:
    k += 1
    fake.fake_fail(k)
    rc = solve()
    left = fake.fake_queued()
    if fake.fake_fail(0) > 0: break                  # the solve ended before its k-th fallible call
    assert rc == -2, (k, rc)
    assert left == 0, "call %d failed: %d commands were left on the stream" % (k, left)
assert rc == 1 and k > 10, (rc, k)
print("calls", k - 1)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    (d / "fake.cpp").write_text(RUNTIME)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", str(d / "fake.cpp"),
                    "-o", str(d / "fake.so")], check=True)
    return str(d / "fake.so")


@pytest.mark.parametrize("warm", [0, 1])
@pytest.mark.parametrize("solver,n", [("cg", 3000), ("cg", 20000), ("ap", 3000), ("sgd", 3000), ("sgd", 16384), ("sgd", 20000)])
def test_an_error_return_leaves_nothing_queued(runtime, solver, n, warm):
    r = subprocess.run([sys.executable, "-c", CHILD, runtime, LIB, solver, str(n), str(warm)], capture_output=True, text=True,
                       timeout=300, env=dict(os.environ, OMP_NUM_THREADS="1"))
    assert r.returncode == 0, r.stderr[-2000:]


PRODUCTS = r"""
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
lib.gp_last_error.restype = C.c_char_p
n, i64, p = 9000, C.c_int64, C.c_void_p
X, V, O = (C.c_float * (n * 3))(), (C.c_float * (n * 40))(), (C.c_float * (n * 40))()
ctx = p()
assert lib.gp_create(C.byref(ctx), 0, i64(n), 3, X, None) == 0
assert lib.gp_set_theta(ctx, (C.c_double * 3)(1, 1, 1), C.c_double(1), C.c_double(0.5)) == 0
def launches(t, fail=0):
    fake.fake_fail(fail)
    rc = lib.gp_kmv(ctx, V, i64(t), t, O, i64(t), 1)
    return rc, fake.fake_queued(), fake.fake_fail(0)
assert launches(40)[0] == 0
plain = launches(9)[1], launches(40)[1]
for k in range(1, 20):
    rc, _, left = launches(40, k)
    if left > 0: break
    assert rc == -2
    # the failed product has taken its maxima (after its first launch) but may not have cleared them
    again = launches(9)
    assert again[0] == 0 and again[1] in (plain[0], plain[0] + 1), (k, again, plain)
    if k <= 3: assert again[1] == plain[0] + 1, (k, again, plain)
    assert launches(9)[1] == plain[0] and launches(40)[1] == plain[1]
assert k > 3, k
"""


def test_a_product_behind_a_failed_one_starts_from_clear_maxima(runtime):
    """gp_kmv accumulates its column maxima in words that its tile pass clears: where a call ends between the two, the next
    one clears them first, or it would scale its columns by the other call's maxima."""
    r = subprocess.run([sys.executable, "-c", PRODUCTS, runtime, LIB], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
