"""Kernels that use more LDS than the default 64 KB ask for it on every device they are launched on, and again after a
refusal.  The library runs in a process of its own whose HIP calls end in a stub (loaded before the library, so its
symbols come first) that counts the requests per device and launches nothing.  Needs no GPU."""
import os
import subprocess
import sys

import pytest

from testing_lib import ROOT, TEST_LIB

STUB = r"""
#include <stddef.h>
#include <stdlib.h>
static int device = 0, refuse = 0, raised[8], launches = 0;
void stub_set(int dev, int fail) { device = dev; refuse = fail; }
int stub_raised(int dev) { return raised[dev]; }
int stub_launches(void) { return launches; }
int hipGetDevice(int* dev) { *dev = device; return 0; }
int hipFuncSetAttribute(const void* f, int attr, int value) { if (refuse) return 1; ++raised[device]; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { *v = 160 * 1024; return 0; }
int __hipPushCallConfiguration() { return 0; }
int __hipPopCallConfiguration() { return 0; }
int hipLaunchKernel() { ++launches; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* sym) { *p = malloc(1 << 20); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { return 0; }
"""

RUN = r"""
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
vp, i64, it = C.c_void_p, C.c_int64, C.c_int
class Cfg(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("bits", "block", "scale_block", "scale_bits", "v_dtype")]
L.lq_matmul.argtypes = [vp, i64, i64, i64, vp, vp, vp, Cfg, vp, vp, it, it, vp, vp, C.c_size_t, vp]
L.lq_test_sym_eig_fast.argtypes = [vp, it, vp, vp, vp]
L.lq_test_sym_eig.argtypes = [vp, it, vp, vp, vp, vp]
p = vp(4096)                                         # never dereferenced: nothing is launched
def product(precision):
    return L.lq_matmul(p, 600, 64, 64, p, p, p, Cfg(4, 16, 16, 8, 0), None, None, 0, precision, p, p, 1 << 40, None)
calls = {"plane_gemm": (lambda: product(1), 1), "qmatmul": (lambda: product(0), 1),
         "sym_eig": (lambda: L.lq_test_sym_eig_fast(p, 96, p, p, None), 1),
         "jacobi_eig": (lambda: L.lq_test_sym_eig(p, 160, p, p, p, None), 2)}       # two kernels
call, kernels = calls[sys.argv[3]]
def on(dev, fail=0):
    before, n = stub.stub_raised(dev), stub.stub_launches()
    stub.stub_set(dev, fail)
    rc = call()
    return rc, stub.stub_raised(dev) - before, stub.stub_launches() > n
assert on(0, 1)[:2] == (-7, 0), "a refused limit is an error"
r = on(0)
assert r == (0, kernels, True), (r, "asked for again")
assert on(0) == (0, 0, True)
assert on(1) == (0, kernels, True), "a second device has a limit of its own"
assert on(0) == (0, 0, True) and on(1) == (0, 0, True)
"""


@pytest.mark.parametrize("kernel", ["plane_gemm", "qmatmul", "sym_eig", "jacobi_eig"])
def test_lds_limit_is_raised_on_every_device(tmp_path, kernel):
    if not os.path.exists(TEST_LIB):
        from paper_2311_12023_amd import build
        build.build()
    src, lib, run = tmp_path / "stub.c", tmp_path / "libstub.so", tmp_path / "run.py"
    src.write_text(STUB)
    run.write_text(RUN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(lib), str(src)], check=True)
    out = subprocess.run([sys.executable, str(run), str(lib), TEST_LIB, kernel], capture_output=True, text=True, cwd=ROOT)
    assert out.returncode == 0, out.stderr
