"""Kernels that use more LDS than the default 64 KB ask for it on every device they are launched on, and again after a
refusal.  Needs no GPU: the library runs against the stub of hip_stub.py."""
import pytest

import hip_stub

RUN = r"""
p = vp(4096)                                         # never dereferenced: nothing is launched
def product(precision):
    return L.lq_matmul(p, 600, 64, 64, p, p, p, Cfg(4, 16, 16, 8, 0), None, None, 0, precision, p, p, 1 << 40, None)
calls = {"plane_gemm": (lambda: product(1), 1), "qmatmul": (lambda: product(0), 1),
         "sym_eig": (lambda: L.lq_test_sym_eig_fast(p, 96, p, p, None), 1),
         "jacobi_eig": (lambda: L.lq_test_sym_eig(p, 160, p, p, p, None), 2)}       # two kernels
call, kernels = calls[args[0]]
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
    hip_stub.run(tmp_path, RUN, kernel)
