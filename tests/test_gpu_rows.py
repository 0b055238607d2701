"""The forward product for 9 to 128 rows of X at the sizes where its kernel can go wrong: row tiles of 16 and groups of 48,
column tiles of 128 in half runs of 8, reductions shorter than its eight wavefronts, shares that end inside a tile, ranks
that are not multiples of 4 or of the 64 columns of a tile of L1.  Tolerances as in test_gpu_matmul.py: 4e-5 (precision 0)
and 1e-2 (precision 1) of |X| (|Q| + |L1| |L2|)."""
import numpy as np
import pytest

from paper_2311_12023_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,k,cfg,rank", [
    (9, 32, 16, (2, 16, 16), 0), (16, 64, 48, (3, 16, 64), 1), (17, 256, 144, (8, 16, 16), 3), (48, 288, 128, (4, 64, 256), 64),
    (49, 320, 272, (3, 16, 256), 65), (64, 1056, 528, (2, 16, 64), 33), (65, 512, 640, (8, 32, 16), 200), (97, 992, 384, (4, 128, 64), 62),
    (127, 224, 1040, (3, 16, 16), 512), (128, 2080, 64, (2, 64, 16), 5), (128, 128, 2064, (4, 16, 256, 5, "fp16"), 16),
    (9, 4096, 11008, (4, 64, 256, 8, "bf16"), 64),       # shares that end inside a tile
])
def test_rows_match_oracle(oracle, m, d, k, cfg, rank):
    import torch
    from paper_2311_12023_amd import lq
    ocfg = oracle.config(*cfg)
    w = gen.weight_matrix(d, k, 300 + m, 4, outlier_frac=0.01)
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    l1, l2 = gen.low_rank_factors(d, k, rank, 301 + m) if rank > 0 else (None, None)
    x = gen.activations(m, d, 302 + m)
    ref, scale = oracle.matmul(x, codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    t = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    args = (t(x), t(oracle.pack(codes, cfg[0])), t(sidx), t(v), lq.config(*cfg), k, t(l1), t(l2))
    for precision, tol in ((0, 4e-5), (1, 1e-2)):
        ws = lq.matmul_workspace(m, d, k, rank)
        ws.fill_(0xff)                                   # NaN patterns: every partial sum that is read was written
        y = lq.matmul(*args, precision=precision, workspace=ws)
        again = lq.matmul(*args, precision=precision)
        assert torch.equal(y, again)
        y = y.cpu().numpy()
        assert np.all(np.isfinite(y))
        assert np.max(np.abs(y - ref) - tol * scale) <= 0, (precision, np.max(np.abs(y - ref) / scale))


# (m, d, k, block) with three steps for one wavefront and two for the others, from which one row tile and 2-bit codes take the scales into
# X and the others do not: an odd number of 64 columns and one, two and three row tiles, blocks of a tile's columns and more
@pytest.mark.parametrize("m,d,k,block", [(9, 544, 16448, 64), (24, 544, 16448, 64), (40, 544, 16512, 128), (128, 544, 8256, 64), (17, 544, 16384, 1024)])
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
def test_rows_with_scales_in_x(oracle, m, d, k, block, bits):
    test_rows_match_oracle(oracle, m, d, k, (bits, block, 16), 33)


# Shares that end inside a tile: the next tile's first step is then asked for before this one's sums.  42 steps to a tile and 43 to
# a share (33 and 34 at 97 rows): every wavefront has five or more (four).
@pytest.mark.parametrize("m,d,k,cfg", [
    (48, 4096, 11072, (3, 64, 256)), (60, 1344, 16448, (8, 64, 16)), (60, 1344, 16448, (4, 64, 64)), (60, 1344, 16512, (3, 128, 16)),
    (97, 1056, 11008, (4, 128, 64)), (97, 1056, 11008, (8, 128, 16)),
])
def test_rows_shares_that_end_inside_a_tile(oracle, m, d, k, cfg):
    test_rows_match_oracle(oracle, m, d, k, cfg, 33)


@pytest.mark.parametrize("m", [12, 20])
@pytest.mark.parametrize("bits,block", [(3, 64), (4, 128)])
def test_rows_zero_scales_and_infinite_x(oracle, bits, block, m):
    """Blocks of zeros have scale 0 whatever X is multiplied with; a row of X that is not finite stays in its row."""
    import torch
    from paper_2311_12023_amd import lq
    d, k = 544, 16384
    ocfg = oracle.config(bits, block, 16)
    w = gen.weight_matrix(d, k, 77, 4)
    w[:, :block] = 0
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    x = gen.activations(m, d, 78)
    x[3, 5], x[11, 200] = np.inf, np.nan
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    y = lq.matmul(t(x), t(oracle.pack(codes, bits)), t(sidx), t(v), lq.config(bits, block, 16), k).cpu().numpy()
    ok = np.setdiff1d(np.arange(m), [3, 11])
    ref, scale = oracle.matmul(x[ok], codes, sidx, v, ocfg, k, want_abs=True)
    assert np.all(y[ok, :block] == 0) and np.all(np.abs(y[ok] - ref) <= 4e-5 * scale)
    assert not np.any(np.isfinite(y[[3, 11]][:, block:]))


def _noise(d, k, seed):
    return np.random.default_rng(seed).standard_normal((d, k), np.float32) * np.float32(0.02)


# one, two and three row tiles at sizes that take the scales into X, and without
@pytest.mark.parametrize("m,d,k,block,bits", [
    (16, 544, 16448, 64, 2), (16, 544, 16448, 64, 3), (16, 544, 16448, 64, 4), (16, 544, 16448, 64, 8), (60, 1344, 16448, 64, 4),
    (60, 1344, 16448, 64, 8), (60, 1344, 16512, 128, 3), (97, 1056, 11008, 128, 4), (97, 1056, 11008, 128, 8), (24, 544, 16448, 64, 4),
])
def test_rows_bf16_x_is_not_rounded(oracle, m, d, k, block, bits):
    """Rows of X with one element, exact in bf16, show every weight by itself.  Rounding the weight to the sum of two bf16
    (precision 0) or to one (precision 1) is off by 2^-17 or 2^-8 of it at most; X times a block's scale must not be rounded
    as coarsely on top of the values of the code book.  Beside that there are fp32 roundings of scale, product and sum and, for
    precision 1, 2^-17 of X times the scale."""
    import torch
    from paper_2311_12023_amd import lq
    ocfg = oracle.config(bits, block, 16)
    codes, sidx, v, _ = oracle.quantize(_noise(d, k, 500 + bits).ravel(), ocfg)
    x = np.zeros((m, d), np.float32)
    at = np.random.default_rng(bits).permutation(d)[:m]
    x[np.arange(m), at] = torch.from_numpy(gen.activations(1, m, 501)[0]).bfloat16().float().numpy()
    ref = x[np.arange(m), at].astype(np.float64)[:, None] * oracle.dequantize(codes, sidx, v, ocfg).reshape(d, k)[at]
    scale = np.abs(ref)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for precision, bound in ((0, 2.0 ** -17 + 2.0 ** -20), (1, 2.0 ** -8 + 2.0 ** -16)):
        y = lq.matmul(t(x), t(oracle.pack(codes, bits)), t(sidx), t(v), lq.config(bits, block, 16), k, precision=precision).cpu().numpy()
        assert np.max(np.abs(y - ref) - bound * scale) <= 0, (precision, np.max(np.abs(y - ref)[scale > 0] / scale[scale > 0]))


@pytest.mark.parametrize("m,d,k,bits,block", [
    (12, 544, 16448, 2, 64), (12, 544, 16448, 3, 64), (12, 544, 16448, 4, 64), (12, 544, 16448, 8, 64), (12, 544, 16512, 4, 128),
    (60, 1344, 16448, 4, 64), (60, 1344, 16512, 3, 128), (97, 1056, 11008, 4, 128), (97, 1056, 11008, 8, 128),
])
def test_rows_scale_times_x_past_the_largest_float(oracle, m, d, k, bits, block):
    """3e38 times a block's largest weight of 4 overflows, times its other weights (code 0, or small) it does not: columns whose
    result fits are as close to the oracle's as any other, the rest are infinite.  A row with an infinite element is not finite
    (split into bf16 it is NaN) and keeps to itself."""
    import torch
    from paper_2311_12023_amd import lq
    ocfg = oracle.config(bits, block, 16)
    w = _noise(d, k, 600 + bits)
    w[100], w[300] = 0, 0
    w[100, 7::block] = 4
    if bits == 8: w[100, 11::block] = -0.9
    w[300, 3::block], w[300, 5::block] = 2, -2
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    x = gen.activations(m, d, 601)
    x[:, [100, 300]] = 0
    x[1, 100] = x[m - 1, 100] = 3e38
    x[4, 300] = np.inf
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    keep = np.arange(m) != 4
    x64, q = x[keep].astype(np.float64), oracle.dequantize(codes, sidx, v, ocfg).reshape(d, k).astype(np.float64)
    ref, scale = x64 @ q, np.abs(x64) @ np.abs(q)
    fits = np.abs(ref) < 3.3e38
    assert 0 < np.sum(~fits) <= 2 * k // block + k // block
    for precision, tol in ((0, 4e-5), (1, 1e-2)):
        y = lq.matmul(t(x), t(oracle.pack(codes, bits)), t(sidx), t(v), lq.config(bits, block, 16), k, precision=precision).cpu().numpy()
        assert not np.any(np.isfinite(y[4]))
        y = y[keep]
        assert np.all(np.abs(y[fits] - ref[fits]) <= tol * scale[fits]) and np.all(np.isposinf(y[~fits]))
