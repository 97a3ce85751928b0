"""A context's stream need not be ordered behind the null stream (a side stream of
torch is not), so nothing that the null stream may still have to do may be left when
the context's first kernel is enqueued.  The host side runs against a runtime that
records the order of its calls (no GPU)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# HIP calls of dmpt_init: memory on the host, kernels not run
RUNTIME = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
extern "C" {
struct D3 { unsigned x, y, z; };
static D3 g, b; static size_t shm; static void* str;
static void line(const char* op, const void* s) { std::printf("%s %p\n", op, s); }
int __hipPushCallConfiguration(D3 gg, D3 bb, size_t m, void* s) { g = gg; b = bb; shm = m; str = s; return 0; }
int __hipPopCallConfiguration(D3* gg, D3* bb, size_t* m, void** s) { *gg = g; *bb = b; *m = shm; *s = str; return 0; }
int hipLaunchKernel(const void*, D3, D3, void**, size_t, void* s) { line("launch", s); return 0; }
int hipMalloc(void** p, size_t n) { *p = std::calloc(n, 1); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(n, 1); return 0; }
int hipFree(void* p) { std::free(p); return 0; }
int hipHostFree(void* p) { std::free(p); return 0; }
int hipMemset(void* p, int v, size_t n) { line("fill", 0); std::memset(p, v, n); return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { line("fill", s); std::memset(p, v, n); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { line("sync", 0); std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void* q) { line("copy", q); std::memcpy(d, s, n); return 0; }
int hipStreamSynchronize(void* s) { line("sync", s); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipEventCreate(void** e) { *e = std::malloc(1); return 0; }
int hipEventDestroy(void* e) { std::free(e); return 0; }
int hipGetLastError() { return 0; }
}
"""

CALL = r"""
import ctypes, sys
runtime, lib, precision, ckpt = sys.argv[1], sys.argv[2], int(sys.argv[3]), int(sys.argv[4])
ctypes.CDLL(runtime, ctypes.RTLD_GLOBAL)
d = ctypes.CDLL(lib)
n = 300
opt = (ctypes.c_int32 * 8)()
d.dmpt_default_options(opt)
opt[0], opt[5] = precision, ckpt                       # precision, ckpt_every
h0 = (ctypes.c_double * (n * n))()
ctx = ctypes.c_void_p()
st = d.dmpt_init(ctypes.byref(ctx), h0, ctypes.c_int64(n), ctypes.c_int64(n // 2), 2, opt,
                 ctypes.c_void_p(0x1000))
assert st == 0, st
d.dmpt_destroy(ctx)
ctypes.CDLL(None).fflush(None)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("runtime")
    (d / "runtime.cpp").write_text(RUNTIME)
    so = str(d / "libruntime.so")
    subprocess.run([cxx, "-shared", "-fPIC", "-O1", str(d / "runtime.cpp"), "-o", so], check=True)
    return so


@pytest.mark.parametrize("precision,ckpt", [(0, 0), (0, 4), (1, 0), (2, 4), (3, 0)])
def test_nothing_is_pending_on_the_null_stream_at_the_first_launch(runtime, precision, ckpt):
    lib = os.path.join(ROOT, "paper_2203_09621_amd", "libdmpt.so")
    run = subprocess.run([sys.executable, "-c", CALL, runtime, lib, str(precision), str(ckpt)],
                         capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stderr
    log = [line.split() for line in run.stdout.splitlines()]
    assert sum(op == "launch" and s == "0x1000" for op, s in log) >= 3
    assert sum(op == "fill" for op, _ in log) >= 4
    pending = 0
    for op, s in log:
        if s == "(nil)":
            pending = 0 if op == "sync" else pending + 1
        elif op == "launch":
            assert pending == 0, "a fill on the null stream may run after this launch"
