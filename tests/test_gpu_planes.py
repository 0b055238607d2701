"""The bf16 forward product for more than 512 rows (precision 1: the weights decoded into a plane first) at the edges of its
tiles: rows and columns against 256, the reduction against the 32 of a step, the 64 of a decode tile and the four stages of
the pipeline, ranks against 32 and 64.  Tolerance as in test_gpu_matmul.py: 1e-2 of |X| (|Q| + |L1| |L2|)."""
import numpy as np
import pytest

from paper_2311_12023_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,k,cfg,rank", [
    (513, 32, 16, (2, 16, 16), 0),            # one step, one 16-column run
    (520, 96, 272, (3, 16, 64), 1),           # three steps and one of the low-rank part, a second column tile of 16
    (768, 160, 256, (4, 64, 256), 33),        # whole tiles, an odd number of half decode tiles
    (1025, 416, 528, (8, 16, 16), 64),        # one row in the fifth row tile
    (600, 2080, 128, (4, 32, 16, 5, "fp16"), 32), (2100, 64, 144, (3, 16, 256), 17),
    # the sizes above that go to the general kernel (small weights and ranks up to 32) at the rows from which they do not
    (1281, 32, 16, (2, 16, 16), 0), (1032, 96, 272, (3, 16, 64), 1), (1112, 2080, 128, (4, 32, 16, 5, "fp16"), 32),
    (1100, 1024, 1008, (4, 16, 64), 16),      # 20 tiles of 8 ranges: pairs are dealt out across tiles
    # more than 128 tiles: the reduction is not cut, tiles go straight to Y
    (1030, 64, 6928, (3, 16, 256), 17),       # a second band of row tiles with a single one, 28 column tiles
    (2305, 32, 3344, (4, 16, 64), 0),         # ten row tiles in three bands, the last of two, and one step
])
def test_planes_match_oracle(oracle, m, d, k, cfg, rank):
    import torch
    from paper_2311_12023_amd import lq
    ocfg = oracle.config(*cfg)
    w = gen.weight_matrix(d, k, 400 + m, 4, outlier_frac=0.01)
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    l1, l2 = gen.low_rank_factors(d, k, rank, 401 + m) if rank > 0 else (None, None)
    x = gen.activations(m, d, 402 + m)
    ref, scale = oracle.matmul(x, codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    t = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    args = (t(x), t(oracle.pack(codes, cfg[0])), t(sidx), t(v), lq.config(*cfg), k, t(l1), t(l2))
    ws = lq.matmul_workspace(m, d, k, rank)
    ws.fill_(0xff)                                       # NaN patterns: nothing stale is read
    y = lq.matmul(*args, precision=1, workspace=ws)
    assert torch.equal(y, lq.matmul(*args, precision=1))
    y = y.cpu().numpy()
    assert np.all(np.isfinite(y))
    assert np.max(np.abs(y - ref) - 1e-2 * scale) <= 0, np.max(np.abs(y - ref) / scale)
