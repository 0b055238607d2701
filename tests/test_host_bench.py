"""bench.py against the library: every product kernel of the forward product has a class of its own in the profile and a
roofline in the result line.  Needs no GPU."""
import importlib.util
import os

import pytest

from testing_lib import ROOT
import hip_stub


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("lq_bench", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


# rows, precision -> the kernel that multiplies X with the weights
ROUTES = [(1, 0, "qmatvec_kernel"), (8, 1, "qmatvec_kernel"), (9, 0, "qrows_kernel"), (128, 1, "qrows_kernel"),
          (129, 0, "qmatmul_kernel"), (512, 1, "qmatmul_kernel"), (513, 0, "qmatmul_kernel"), (513, 1, "plane_gemm_kernel")]


@pytest.mark.parametrize("m,precision,kernel", ROUTES)
def test_profile_names_the_kernel_that_runs(tmp_path, m, precision, kernel):
    hip_stub.run(tmp_path, r"""
m, precision, kernel = int(args[0]), int(args[1]), args[2]
p = vp(4096)
ran = classes_of(lambda: L.lq_matmul(p, m, 1024, 2048, p, p, p, Cfg(4, 16, 16, 8, 0), p, p, 64, precision, p, p, 1 << 40, None))
products = {"qmatvec_kernel", "qrows_kernel", "qmatmul_kernel", "plane_gemm_kernel"} & set(ran)
assert products == {kernel}, ran
if kernel not in ("qmatvec_kernel",):
    assert ran[kernel] >= 2.0 * m * 1024 * 2048
if kernel == "plane_gemm_kernel":
    assert "weight_plane_kernel" in ran
""", m, precision, kernel)


@pytest.mark.parametrize("m,precision,kernel", ROUTES)
def test_every_product_kernel_has_a_roofline(bench, m, precision, kernel):
    out = bench.matmul_roofline({kernel: (2.0, 4, 1e9), "misc": (0.5, 8, 1e6)}, precision, None)
    assert out["roofline"]["kernel"] == kernel and out["roofline"]["launches"] == 4
    assert out["roofline"]["bound"] == ("hbm" if kernel == "qmatvec_kernel" else "mfma")
    assert out["roofline"]["frac"] == out["roofline"]["achieved"] / out["roofline"]["peak"]
    assert out["kernels"]["misc"] == {"ms": 0.5, "launches": 8}
    assert bench.matmul_roofline({}, precision, None) == {}
