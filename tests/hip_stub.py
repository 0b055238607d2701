"""Runs a piece of Python with the testing build of the library in a process of its own whose HIP calls end in a stub: it is
loaded before the library, so its symbols come first; it launches nothing and counts requests, launches and their
threads."""
import os
import subprocess
import sys

from testing_lib import ROOT, TEST_LIB

STUB = r"""
#include <stddef.h>
#include <stdlib.h>
struct dim { unsigned x, y, z; };
static int device = 0, refuse = 0, raised[8], launches = 0;
static double most = 0, total = 0;
void stub_set(int dev, int fail) { device = dev; refuse = fail; }
int stub_raised(int dev) { return raised[dev]; }
int stub_launches(void) { return launches; }
int hipGetDevice(int* dev) { *dev = device; return 0; }
int hipFuncSetAttribute(const void* f, int attr, int value) { if (refuse) return 1; ++raised[device]; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { *v = 160 * 1024; return 0; }
double stub_most_threads(void) { return most; }
double stub_all_threads(void) { return total; }
int __hipPushCallConfiguration(struct dim g, struct dim b, size_t shm, void* st) {
  double n = (double)g.x * g.y * g.z * b.x * b.y * b.z;
  if (n > most) most = n;
  total += n;
  return 0;
}
int __hipPopCallConfiguration() { return 0; }
int hipLaunchKernel() { ++launches; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* sym) { *p = malloc(1 << 20); return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventRecord(void* e, void* st) { return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 1.0f; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { return 0; }
"""

PRELUDE = r'''
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
args = sys.argv[3:]
stub.stub_most_threads.restype = stub.stub_all_threads.restype = C.c_double
vp, i64, it = C.c_void_p, C.c_int64, C.c_int
class Cfg(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("bits", "block", "scale_block", "scale_bits", "v_dtype")]
L.lq_nf_quantize.argtypes = [vp, i64, Cfg, vp, vp, vp, vp]
L.lq_matmul.argtypes = [vp, i64, i64, i64, vp, vp, vp, Cfg, vp, vp, it, it, vp, vp, C.c_size_t, vp]
L.lq_matmul_workspace_bytes.restype = L.lq_matmul_workspace_bytes_precision.restype = C.c_size_t
L.lq_matmul_workspace_bytes.argtypes = [i64, i64, i64, it]
L.lq_matmul_workspace_bytes_precision.argtypes = [i64, i64, i64, it, it]
L.lq_test_sym_eig_fast.argtypes = [vp, it, vp, vp, vp]
L.lq_test_sym_eig.argtypes = [vp, it, vp, vp, vp, vp]
L.lq_profile_class_name.restype = C.c_char_p
L.lq_profile_read.argtypes = [it, vp, vp, vp]
def classes_of(call):
    """Profile classes that the launches of call() are booked under: {name: work}."""
    L.lq_profile_enable(1); L.lq_profile_reset()
    assert call() == 0
    ran = {}
    for c in range(L.lq_profile_num_classes()):
        ms, n, w = C.c_double(), C.c_int64(), C.c_double()
        assert L.lq_profile_read(c, C.addressof(ms), C.addressof(n), C.addressof(w)) == 0
        if n.value:
            ran[L.lq_profile_class_name(c).decode()] = w.value
    L.lq_profile_enable(0)
    return ran
'''


def run(tmp_path, code, *args):
    if not os.path.exists(TEST_LIB):
        from paper_2311_12023_amd import build
        build.build()
    src, lib, script = tmp_path / "stub.c", tmp_path / "libstub.so", tmp_path / "run.py"
    src.write_text(STUB)
    script.write_text(PRELUDE + code)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(lib), str(src)], check=True)
    out = subprocess.run([sys.executable, str(script), str(lib), TEST_LIB, *map(str, args)], capture_output=True, text=True,
                         cwd=ROOT)
    assert out.returncode == 0, out.stderr
