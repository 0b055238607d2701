"""Workspaces of the forward product over row counts and precisions: what a size serves.  Needs no GPU (hip_stub.py)."""
import pytest

import hip_stub
from testing_lib import load

RUN = r"""
d, k, rank = map(int, args)
p = vp(4096)                                         # never dereferenced: nothing is launched
def product(m, precision, size):
    return L.lq_matmul(p, m, d, k, p, p, p, Cfg(4, 16, 16, 8, 0), p, p, rank, precision, p, p, size, None)
# a workspace sized once for the largest batch serves every batch of 1 to 128 rows (ranks above 512 have no such kernels)
for top in (9, 12, 16, 24, 49, 63, 100, 128, 129, 300, 513, 1000) if rank <= 512 else ():
    size = L.lq_matmul_workspace_bytes(top, d, k, rank)
    for m in range(1, min(top, 128) + 1):
        for precision in (0, 1):
            assert product(m, precision, size) == 0, (top, m, precision, size)
for m in (1, 3, 8, 9, 40, 128, 129, 256, 400, 512, 513, 600, 1000, 4096):
    both = L.lq_matmul_workspace_bytes(m, d, k, rank)
    one = [L.lq_matmul_workspace_bytes_precision(m, d, k, rank, q) for q in (0, 1)]
    assert both == max(one)
    assert all(product(m, q, one[q]) == 0 for q in (0, 1))
    assert product(m, 0, 255) == product(m, 1, 255) == -6
    if m > 512:
        # fp32-grade products bring no room for weights in bf16: two planes of X, T and its planes, partial sums of at most
        # 256 tiles or 16 ranges, one scale for 16 weights
        rows, r32 = -(-m // 256) * 256, -(-rank // 32) * 32
        ranges = min(256 // max(1, -(-m // 256) * -(-k // 256)), 16)
        bound = 4 * rows * (d + 2 * r32 + 64 * 16) + 4 * m * ranges * max(k, r32 if rank > 64 else 0) * (ranges > 1) + d * k // 4 + 4096
        if rank <= 64:
            assert one[0] <= bound, (m, one[0], bound)
        # and a bf16 call takes such a workspace too
        assert product(m, 1, one[0]) == 0
"""


@pytest.mark.parametrize("d,k", [(4096, 4096), (4096, 11008), (8192, 8192), (5120, 13824), (8192, 28672), (768, 768), (32, 16)])
@pytest.mark.parametrize("rank", [0, 64, 200, 600])
def test_workspace_serves_smaller_batches(tmp_path, d, k, rank):
    hip_stub.run(tmp_path, RUN, d, k, rank)


def test_sizes_of_the_precisions(tmp_path):
    hip_stub.run(tmp_path, r"""
size = L.lq_matmul_workspace_bytes_precision
assert size(64, 250, 512, 8, 0) == size(64, 256, 512, 8, 2) == size(0, 256, 512, 8, 1) == 0
assert size(1000, 4096, 11008, 64, 0) < 40e6 and size(1000, 4096, 11008, 64, 1) > 2 * 4096 * 11008
assert L.lq_matmul_workspace_bytes(1000, 4096, 11008, 64) < 110e6          # nothing that a route leaves alone
assert L.lq_matmul_workspace_bytes(4096, 11008, 4096, 64) == size(4096, 11008, 4096, 64, 0)   # the plane in place of the lo half of X
assert L.lq_matmul_workspace_bytes(24, 4096, 11008, 64) == L.lq_matmul_workspace_bytes(9, 4096, 11008, 64) < 16e6
""")


# rows, weights, rank, bits -> the product kernel at precisions 0 and 1, as measured (us in lq_api_matmul.cpp)
ROUTES = [
    (64, 8192, 8192, 65, 3, "qrows qrows"), (96, 4096, 11008, 512, 4, "qrows qrows"), (96, 4096, 11008, 512, 3, "qmatmul qmatmul"),
    (80, 8192, 8192, 62, 4, "qrows qmatmul"), (128, 4096, 4096, 64, 3, "qrows qrows"), (128, 4096, 4096, 0, 3, "qmatmul qmatmul"),
    (128, 4096, 4096, 65, 4, "qrows qrows"), (97, 4096, 11008, 64, 3, "qmatmul qmatmul"), (97, 4096, 11008, 64, 4, "qrows qrows"),
    (128, 11008, 4096, 128, 3, "qrows qrows"), (112, 4096, 11008, 128, 3, "qmatmul qmatmul"), (128, 4096, 11008, 256, 4, "qrows qrows"),
    (128, 4096, 11008, 512, 8, "qmatmul qmatmul"), (128, 11008, 4096, 512, 8, "qrows qrows"), (100, 4096, 11008, 65, 4, "qrows qmatmul"),
    (100, 5120, 13824, 65, 4, "qmatmul qmatmul"), (128, 8192, 8192, 64, 4, "qrows qmatmul"), (128, 8192, 8192, 0, 2, "qmatmul qmatmul"),
    (128, 1024, 1024, 33, 3, "qrows qrows"),
]


@pytest.mark.parametrize("m,d,k,rank,bits,kernels", ROUTES)
def test_kernel_for_65_to_128_rows(tmp_path, m, d, k, rank, bits, kernels):
    """Large weights: the kernel that was measured to be the faster one runs when the workspace has the size that was asked
    for, and the other where only that one fits."""
    hip_stub.run(tmp_path, r"""
m, d, k, rank, bits = map(int, args[:5])
p = vp(4096)
def ran(precision, size):
    return [n.split("_")[0] for n in classes_of(lambda: L.lq_matmul(p, m, d, k, p, p, p, Cfg(bits, 16, 16, 8, 0), p, p, rank,
            precision, p, p, size, None)) if n in ("qrows_kernel", "qmatmul_kernel")]
for precision, kernel in enumerate(args[5].split()):
    assert ran(precision, L.lq_matmul_workspace_bytes_precision(m, d, k, rank, precision)) == [kernel]
    assert ran(precision, L.lq_matmul_workspace_bytes(9, d, k, rank)) == ["qrows"]
""", m, d, k, rank, bits, kernels)


@pytest.mark.parametrize("m,d,k,rank,kernel", [
    (512, 4096, 4096, 64, "qmatmul"), (513, 4096, 4096, 64, "plane"), (513, 2048, 2048, 0, "plane"), (640, 1024, 1024, 16, "qmatmul"),
    (640, 1024, 1024, 33, "plane"), (1024, 768, 3072, 32, "qmatmul"), (1025, 768, 3072, 32, "plane"), (600, 4096, 4096, 65, "qmatmul")])
def test_kernel_for_bf16_rows(tmp_path, m, d, k, rank, kernel):
    hip_stub.run(tmp_path, r"""
m, d, k, rank = map(int, args[:4])
p = vp(4096)
ran = classes_of(lambda: L.lq_matmul(p, m, d, k, p, p, p, Cfg(4, 16, 16, 8, 0), p, p, rank, 1, p, p, 1 << 40, None))
assert ("plane_gemm_kernel" in ran) == (args[4] == "plane") and ("qmatmul_kernel" in ran) == (args[4] == "qmatmul"), ran
""", m, d, k, rank, kernel)


# columns, rows, rank -> us of the whole call with rows_finish_kernel and with qmatvec_finish_kernel, at K of 2048 (28672 columns),
# 1024 (1024 columns) or 4096
FINISH = [
    (28672, 16, 17, 36.6, 38.9), (28672, 32, 17, 42.8, 46.6), (28672, 24, 64, 37.3, 38.3), (28672, 16, 65, 46.6, 50.1),
    (28672, 48, 65, 65.1, 75.1), (28672, 24, 256, 53.0, 58.5), (28672, 64, 512, 151.2, 176.6), (11008, 32, 17, 33.6, 34.9),
    (11008, 24, 65, 39.8, 41.6), (11008, 48, 256, 56.0, 59.3), (11008, 64, 512, 88.7, 98.3), (1024, 24, 17, 11.9, 12.6),
    (28672, 8, 64, 36.7, 35.3), (28672, 8, 512, 65.6, 53.0), (11008, 24, 64, 30.5, 29.8), (11008, 32, 64, 31.5, 30.8),
    (11008, 16, 256, 40.6, 38.0), (11008, 16, 512, 56.3, 51.4), (1024, 24, 64, 13.5, 12.4), (1024, 64, 512, 36.8, 30.2),
    (1024, 4, 256, 17.0, 13.3),
]


@pytest.mark.parametrize("k,m,rank,rows_us,few_us", FINISH)
def test_finishing_kernel(k, m, rank, rows_us, few_us):
    assert load().lq_test_rows_finish(m, k, rank) == (rows_us < few_us)
