"""GPU parity of the forward product Y = X (Q + L1 L2) with just-in-time dequantization (Section 3.2
"Implementation", Appendix A) against the oracle's fp64 definition.

Tolerance (derived from the arithmetic).  Precision 0 splits each operand into two bf16 halves: the split drops at
most 2^-18 of an operand, the omitted lo*lo term is at most 2^-18 of a product, so a product is off by at most
3 * 2^-18 = 1.1e-5 of |x||w|; fp32 accumulation over K terms adds about sqrt(K) * 2^-24 in practice.  The bound
used is 4e-5 * S with S = |X| (|Q| + |L1||L2|) elementwise, which the oracle returns.  Precision 1 (bf16 operands)
rounds each operand to 2^-9: 2^-8 per product, bound 1e-2 * S.  The quantized operand itself is exact: the kernel
multiplies the same fl32(code * scale) values that Dequantize returns.  Up to 8 rows of X (and rank <= 512) the product
runs in plain fp32 on the vector ALU whatever the precision argument says, and is held to the tighter bound as well.
"""
import numpy as np
import pytest

from paper_2311_12023_amd import gen

pytestmark = pytest.mark.gpu

TOL_SPLIT = 4e-5
TOL_BF16 = 1e-2


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2311_12023_amd import lq
    return torch, lq


def _case(oracle, d, k, cfg_tuple, rank, seed):
    ocfg = oracle.config(*cfg_tuple)
    w = gen.weight_matrix(d, k, seed, 4, outlier_frac=0.01)
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    l1, l2 = gen.low_rank_factors(d, k, rank, seed + 1) if rank > 0 else (None, None)
    return ocfg, codes, sidx, v, l1, l2


def _gpu_product(env, oracle, x, codes, sidx, v, cfg_tuple, k, l1, l2, precision):
    torch, lq = env
    t = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    packed = oracle.pack(codes, cfg_tuple[0])
    y = lq.matmul(t(x), t(packed), t(sidx), t(v), lq.config(*cfg_tuple), k, t(l1), t(l2), precision=precision)
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("m,d,k,cfg,rank", [
    (1, 32, 64, (4, 16, 16), 0),             # a single row, one reduction step, no low-rank part
    (7, 96, 192, (3, 32, 16), 5),            # ragged against every tile size, rank below one step
    (130, 256, 384, (4, 64, 256), 64),       # two row tiles (the second nearly empty), three column tiles
    (257, 160, 144, (2, 16, 16), 8),         # three row tiles, column tile cut at 144
    (64, 512, 128, (8, 64, 64), 40),         # 8-bit codes, rank that is not a multiple of 32
    (300, 64, 2048, (4, 32, 64), 33),        # wide output
    (8, 256, 384, (4, 64, 256), 64),         # few rows: the vector-ALU path, one full chunk of 8 rows
    (6, 160, 528, (3, 16, 16), 7),           # 3-bit runs, columns ragged against 128, rank not a multiple of anything
    (4, 1056, 272, (8, 16, 64), 40),         # 8-bit runs, reduction ranges of unequal length
    (2, 4192, 144, (2, 16, 16), 33),         # 2-bit runs, several ranges with the dense rows in the last one
    (20, 160, 528, (3, 16, 16), 7),          # just above that path's limit
    (3, 96, 64, (2, 32, 16), 1),             # rank 1
    (5, 64, 128, (4, 64, 16), 600),          # a rank beyond that path's limit goes to the MFMA kernel
    (520, 1120, 256, (4, 64, 256), 64),      # nine 64-row strips of X, 17.5 steps of 64 cut into reduction ranges
    (70, 224, 192, (3, 32, 32), 32),         # rank 32: T keeps one 32-deep step
    (40, 96, 128, (4, 32, 16), 0),           # MFMA path without a low-rank part
    (33, 128, 256, (4, 64, 64), 65),         # the smallest rank that takes the separate X L1 product
    (48, 1024, 512, (4, 64, 256), 64),       # a few dozen rows, reduction cut into ranges: T L2 joins the range sum
    (100, 2048, 320, (3, 32, 64), 17),       # the same with a ragged rank and column tile
    (9, 4096, 256, (2, 16, 16), 33),         # just above the vector path, one column tile, 16 ranges
])
def test_matmul_matches_oracle(env, oracle, m, d, k, cfg, rank):
    ocfg, codes, sidx, v, l1, l2 = _case(oracle, d, k, cfg, rank, 100 + m)
    x = gen.activations(m, d, 200 + m)
    ref, scale = oracle.matmul(x, codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    for precision, tol in ((0, TOL_SPLIT), (1, TOL_BF16)):
        y = _gpu_product(env, oracle, x, codes, sidx, v, cfg, k, l1, l2, precision)
        assert y.shape == (m, k) and np.all(np.isfinite(y))
        excess = np.abs(y - ref) - tol * scale
        assert np.max(excess) <= 0, (precision, np.max(np.abs(y - ref) / scale))


@pytest.mark.parametrize("seed", range(10))
def test_matmul_random_shapes(env, oracle, seed):
    """Seeded random shapes around the tile and strip sizes of all three paths (rows against 8, 64 and 256; the
    reduction against 32 and 64; columns against 256; ranks against 4, 32 and 64)."""
    rng = np.random.default_rng(5000 + seed)
    bits = int(rng.choice([2, 3, 4, 8]))
    block = int(rng.choice([16, 32, 64]))
    scale_block = int(rng.choice([16, 64, 256]))
    m = int(rng.choice([rng.integers(1, 9), rng.integers(9, 70), rng.integers(70, 600)]))
    d = 32 * int(rng.integers(1, 20))
    k = block * int(rng.integers(1, 1 + 640 // block))
    rank = int(rng.choice([0, rng.integers(1, 33), rng.integers(33, 65), rng.integers(65, 90)]))
    cfg = (bits, block, scale_block)
    ocfg, codes, sidx, v, l1, l2 = _case(oracle, d, k, cfg, rank, 6000 + seed)
    x = gen.activations(m, d, 7000 + seed)
    ref, scale = oracle.matmul(x, codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    for precision, tol in ((0, TOL_SPLIT), (1, TOL_BF16)):
        y = _gpu_product(env, oracle, x, codes, sidx, v, cfg, k, l1, l2, precision)
        assert y.shape == (m, k) and np.all(np.isfinite(y))
        assert np.max(np.abs(y - ref) - tol * scale) <= 0, (m, d, k, cfg, rank, precision, np.max(np.abs(y - ref) / scale))


def test_matmul_identity_returns_dequantized_weights(env, oracle):
    """X = I: every output is one stored weight; hi + lo of a weight carries 16 of its 24 bits."""
    torch, lq = env
    d, k, cfg = 128, 256, (4, 64, 256)
    ocfg, codes, sidx, v, _, _ = _case(oracle, d, k, cfg, 0, 31)
    q = oracle.dequantize(codes, sidx, v, ocfg).reshape(d, k).astype(np.float64)
    y = _gpu_product(env, oracle, np.eye(d, dtype=np.float32), codes, sidx, v, cfg, k, None, None, 0)
    assert np.max(np.abs(y - q) - 2.0 ** -16 * np.abs(q)) <= 0
    dq = lq.nf_dequantize(torch.from_numpy(oracle.pack(codes, 4)).cuda(), torch.from_numpy(sidx).cuda(),
                          torch.from_numpy(v).cuda(), d * k, lq.config(*cfg)).cpu().numpy()
    assert np.array_equal(dq.reshape(d, k).astype(np.float64), q)


def test_matmul_is_deterministic_and_ignores_workspace_contents(env, oracle):
    torch, lq = env
    m, d, k, cfg, rank = 48, 256, 256, (3, 64, 256), 16      # small grid: the reduction is cut, partial sums in scratch
    ocfg, codes, sidx, v, l1, l2 = _case(oracle, d, k, cfg, rank, 41)
    x = gen.activations(m, d, 42)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    args = (t(x), t(oracle.pack(codes, cfg[0])), t(sidx), t(v), lq.config(*cfg), k, t(l1), t(l2))
    ws = lq.matmul_workspace(m, d, k, rank)
    ws.fill_(0)
    a = lq.matmul(*args, workspace=ws).clone()
    ws.fill_(0xff)                                           # NaN patterns
    b = lq.matmul(*args, workspace=ws)
    assert torch.equal(a, b)


@pytest.mark.parametrize("shape", [(4096, 4096), (4096, 11008), (11008, 4096)])
def test_matmul_full_size_sampled_rows(env, oracle, shape):
    """The benchmark's shape (m = 4096 tokens, LLaMA-2-7B projections, NF4 with double quantization, rank 64):
    the oracle computes sampled rows of X one by one; the GPU result for those rows must agree, and must not depend
    on which other rows are in the batch."""
    torch, lq = env
    d, k = shape
    cfg, rank, m = (4, 64, 256, 8, "bf16"), 64, 4096
    ocfg = oracle.config(*cfg)
    w = gen.workload_matrix(3, {(4096, 4096): 0, (4096, 11008): 4, (11008, 4096): 6}[shape])
    assert w.shape == shape
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    l1, l2 = gen.low_rank_factors(d, k, rank, 77)
    x = gen.activations(m, d, 78)
    rows = [0, 127, 128, 2049, 4095]
    ref, scale = oracle.matmul(x[rows], codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    y = _gpu_product(env, oracle, x, codes, sidx, v, cfg, k, l1, l2, 0)
    assert np.max(np.abs(y[rows] - ref) - TOL_SPLIT * scale) <= 0, np.max(np.abs(y[rows] - ref) / scale)
    assert np.all(np.isfinite(y))
    y_small = _gpu_product(env, oracle, x[rows], codes, sidx, v, cfg, k, l1, l2, 0)
    assert np.max(np.abs(y_small - ref) - TOL_SPLIT * scale) <= 0


def test_matmul_full_size_few_dozen_rows(env, oracle):
    """96 rows against the 4096 x 4096 benchmark matrix: the path that adds T L2 together with the reduction ranges, at
    its real shape (16 column tiles x 16 ranges), checked on sampled rows."""
    d = k = 4096
    cfg, rank, m = (4, 64, 256, 8, "bf16"), 64, 96
    ocfg = oracle.config(*cfg)
    w = gen.workload_matrix(3, 1)
    codes, sidx, v, _ = oracle.quantize(w.ravel(), ocfg)
    l1, l2 = gen.low_rank_factors(d, k, rank, 79)
    x = gen.activations(m, d, 80)
    rows = [0, 31, 32, 95]
    ref, scale = oracle.matmul(x[rows], codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    for precision, tol in ((0, TOL_SPLIT), (1, TOL_BF16)):
        y = _gpu_product(env, oracle, x, codes, sidx, v, cfg, k, l1, l2, precision)
        assert np.all(np.isfinite(y))
        assert np.max(np.abs(y[rows] - ref) - tol * scale) <= 0, (precision, np.max(np.abs(y[rows] - ref) / scale))


@pytest.mark.parametrize("m", [4, 40, 300])
def test_matmul_in_a_hip_graph(env, oracle, m):
    """lq_matmul only launches kernels, so it can be recorded into a graph (after one eager call, which uploads the
    code-book tables and raises the kernel's LDS limit): every replay, with eager work on new inputs in between, must
    reproduce the eager result bit for bit."""
    torch, lq = env
    d, k, cfg, rank = 256, 512, (4, 64, 256), 16
    ocfg, codes, sidx, v, l1, l2 = _case(oracle, d, k, cfg, rank, 900 + m)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    packed, sidx_t, v_t, l1_t, l2_t = t(oracle.pack(codes, cfg[0])), t(sidx), t(v), t(l1), t(l2)
    gcfg = lq.config(*cfg)
    x = torch.empty((m, d), dtype=torch.float32, device="cuda")
    y = torch.empty((m, k), dtype=torch.float32, device="cuda")
    ws = lq.matmul_workspace(m, d, k, rank)
    x.copy_(t(gen.activations(m, d, 1)))
    lq.matmul(x, packed, sidx_t, v_t, gcfg, k, l1_t, l2_t, out=y, workspace=ws)          # eager warm-up
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lq.matmul(x, packed, sidx_t, v_t, gcfg, k, l1_t, l2_t, out=y, workspace=ws)
    for rep in range(4):
        xin = t(gen.activations(m, d, 10 + rep))
        eager = lq.matmul(xin, packed, sidx_t, v_t, gcfg, k, l1_t, l2_t)                  # own output and workspace
        torch.cuda.synchronize()
        x.copy_(xin)
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, eager), rep


@pytest.mark.parametrize("m,precision", [(1, 0), (8, 0), (24, 1), (300, 1), (600, 1), (1100, 1)])
def test_infinite_group_scale_is_infinite_weights(env, oracle, m, precision):
    """A group scale of infinity (a maximum above 65504 stored in fp16) makes infinite weights, as Dequantize returns them:
    the columns that hold one come out infinite, the others as ever."""
    torch, lq = env
    d, k, cfg = 64, 512, (4, 16, 16, 8, "fp16")
    rng = np.random.default_rng(m)
    ocfg = oracle.config(*cfg)
    codes, sidx, v, _ = oracle.quantize(rng.uniform(0.5, 1.0, d * k).astype(np.float32), ocfg)
    v[3] = np.inf                                            # row 1, columns 256 .. 511
    x = rng.uniform(0.5, 1.0, (m, d)).astype(np.float32)
    q = oracle.dequantize(codes, sidx, v, ocfg).reshape(d, k).astype(np.float64)
    ref = x.astype(np.float64) @ q
    assert np.all(np.isposinf(ref) == (np.arange(k) >= 256))
    y = _gpu_product(env, oracle, x, codes, sidx, v, cfg, k, None, None, precision)
    assert np.array_equal(np.isposinf(y), np.isposinf(ref))
    assert np.max(np.abs(y[:, :256] / ref[:, :256] - 1)) < TOL_BF16


@pytest.mark.parametrize("m,d,k,rank,precision,nbytes", [
    (128, 32, 2048, 16, 0, 200_000), (128, 32, 2048, 16, 1, 200_000),     # too small for the partial sums of 128 rows
    (600, 512, 1024, 40, 1, None),                                        # no room for the weights in bf16
])
def test_matmul_with_a_smaller_workspace(env, oracle, m, d, k, rank, precision, nbytes):
    """A workspace that only the general kernel can work with is accepted and the product is as good."""
    torch, lq = env
    cfg = (4, 32, 64)
    ocfg, codes, sidx, v, l1, l2 = _case(oracle, d, k, cfg, rank, 51)
    x = gen.activations(m, d, 52)
    ref, scale = oracle.matmul(x, codes, sidx, v, ocfg, k, l1, l2, want_abs=True)
    nbytes = nbytes or lq._lib.lq_matmul_workspace_bytes_precision(m, d, k, rank, 0)
    assert nbytes < lq._lib.lq_matmul_workspace_bytes_precision(m, d, k, rank, precision)
    ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device="cuda")
    start = -ws.data_ptr() % 256
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    y = lq.matmul(t(x), t(oracle.pack(codes, cfg[0])), t(sidx), t(v), lq.config(*cfg), k, t(l1), t(l2), precision=precision,
                  workspace=ws[start:start + nbytes]).cpu().numpy()
    assert np.max(np.abs(y - ref) - (TOL_SPLIT, TOL_BF16)[precision] * scale) <= 0
    assert torch.all(ws[start + nbytes:] == 0xff)                 # nothing is written past its end
