"""The launch that adds the reduction ranges of X Q and X L1 and the product with L2: row counts around its workgroups of 1, 2, 4
and 8 rows, ranks around its chunks (16, 64), from one range to more than the sixteen that are in flight at a time, columns that do
not fill its last workgroup, and 6208 columns (97 workgroups for 8 rows), where 17 to 64 rows lie on both sides of every bound between
its two kernels (rows_finish_preferred: 256, 512 and 768 workgroups by rank).  Tolerance 4e-5 of |X| (|Q| + |L1| |L2|) as in
test_gpu_matmul.py."""
import numpy as np
import pytest

from paper_2311_12023_amd import gen
from testing_lib import load

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k", [(32, 16), (4096, 16), (1056, 208), (32, 6208)])
@pytest.mark.parametrize("rank", [0, 1, 16, 17, 32, 33, 64, 65, 128, 512])
def test_ranges_and_low_rank_product(oracle, d, k, rank):
    import torch
    from paper_2311_12023_amd import lq
    cfg = (4, 16, 64)
    ocfg = oracle.config(*cfg)
    w = gen.weight_matrix(d, k, 400 + rank, 4, outlier_frac=0.01)
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    l1, l2 = gen.low_rank_factors(d, k, rank, 401) if rank > 0 else (None, None)
    x = gen.activations(65, d, 402)
    ref, scale = oracle.matmul(x, codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    t = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    args = (t(oracle.pack(codes, 4)), t(sidx), t(v), lq.config(*cfg), k, t(l1), t(l2))
    for m in (1, 2, 3, 4, 5, 8, 9, 17, 32, 33, 64, 65):
        ws = lq.matmul_workspace(m, d, k, rank)
        ws.fill_(0xff)                                   # NaN patterns: every partial sum that is read was written
        y = lq.matmul(t(x[:m]), *args, workspace=ws).cpu().numpy()
        assert np.all(np.isfinite(y)), m
        assert np.max(np.abs(y - ref[:m]) - 4e-5 * scale[:m]) <= 0, (m, np.max(np.abs(y - ref[:m]) / scale[:m]))
    if k == 6208 and rank > 32:
        assert {load().lq_test_rows_finish(m, k, rank) for m in (9, 17, 32, 33, 64)} == {0, 1}
