"""Cholesky-QR (Gram matrix, factor and inverse, rotation) over every number of rows and at column counts around the 16
columns of a Gram step and the 32 of a rotation tile, against what defines it: Q orthonormal, Q = C^-1 X with C lower
triangular.  The Gram matrix is exact to fp64, so what is left is C^-1 rounded to fp32 and fp32 sums over l terms: at a
condition of about 10 (rows drawn with 2 l columns or more), l * 2^-24 * 10 < 2e-4 for l <= 256."""
import numpy as np
import pytest

from paper_2311_12023_amd import gen
from testing_lib import load

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [32, 64, 96, 128, 160, 192, 224, 256])
@pytest.mark.parametrize("extra", [0, 1, 15, 17, 31, 2049])
def test_orthonormalize_ragged(l, extra):
    import torch
    L = load()
    m = 2 * l + extra
    ld = (m + 31) // 32 * 32
    rng = np.random.default_rng(l + extra)
    x = np.zeros((l, ld), np.float32)
    x[:, :m] = rng.standard_normal((l, m))
    xt = torch.from_numpy(x).cuda()
    scratch = torch.full((17 * l * l,), float("nan"), dtype=torch.float64, device="cuda")
    alt = torch.full((l, ld), float("nan"), dtype=torch.float32, device="cuda")
    assert L.lq_test_orthonormalize(xt.data_ptr(), l, m, ld, scratch.data_ptr(), alt.data_ptr(), None) == 0
    torch.cuda.synchronize()
    q = xt.cpu().numpy().astype(np.float64)
    assert np.all(q[:, m:] == 0)
    assert np.max(np.abs(q @ q.T - np.eye(l))) < 2e-4
    c = np.linalg.cholesky(x.astype(np.float64) @ x.T.astype(np.float64))
    assert np.max(np.abs(c @ q - x)) < 2e-4 * np.max(np.abs(x)) * np.sqrt(l)


@pytest.mark.parametrize("l", [32, 64, 96, 128])
@pytest.mark.parametrize("at", [1, 15, 16, 31])
def test_orthonormalize_dependent_rows(l, at):
    """Rows that are a multiple of an earlier one (a power of two, so exactly) or zero, at the edges of the 16-row blocks of
    the factorisation and in the last row: they come out zero and the others orthonormal.  The pivot that remains of such a
    row is rounding, l * 2^-53 of its squared norm, against the threshold of 1e-12."""
    import torch
    L = load()
    m = ld = 4 * l
    rng = np.random.default_rng(l + at)
    x = rng.standard_normal((l, m)).astype(np.float32)
    x[at], x[l - 1] = 4 * x[0], 0
    if l > 32:
        x[32 + at] = 0.5 * x[2]
    dependent = [at, l - 1] + ([32 + at] if l > 32 else [])
    xt = torch.from_numpy(x).cuda()
    scratch = torch.full((17 * l * l,), float("nan"), dtype=torch.float64, device="cuda")
    alt = torch.full((l, ld), float("nan"), dtype=torch.float32, device="cuda")
    assert L.lq_test_orthonormalize(xt.data_ptr(), l, m, ld, scratch.data_ptr(), alt.data_ptr(), None) == 0
    torch.cuda.synchronize()
    q = xt.cpu().numpy().astype(np.float64)
    assert np.all(q[dependent] == 0)
    want = np.eye(l)
    want[dependent, dependent] = 0
    assert np.max(np.abs(q @ q.T - want)) < 2e-4


@pytest.mark.parametrize("l", [64, 96, 128])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_orthonormalize_of_a_row_that_is_not_finite(l, bad):
    """A row of Q is a sum over the rows of X up to its own, taken 32 rows at a time: what is not finite reaches its own 32 rows and
    those after them, and the rows before are what they are without it."""
    import torch
    L = load()
    m = ld = 4 * l
    x = np.random.default_rng(l).standard_normal((l, m)).astype(np.float32)
    results = []
    for value in (1.0, bad):
        x[l - 20, 5] = value
        xt = torch.from_numpy(x).cuda()
        scratch = torch.full((17 * l * l,), float("nan"), dtype=torch.float64, device="cuda")
        alt = torch.full((l, ld), float("nan"), dtype=torch.float32, device="cuda")
        assert L.lq_test_orthonormalize(xt.data_ptr(), l, m, ld, scratch.data_ptr(), alt.data_ptr(), None) == 0
        results.append(xt.cpu().numpy())
    assert np.array_equal(results[0][:l - 32], results[1][:l - 32])
    assert not np.isfinite(results[1][l - 20]).any()


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("d,k,rank", [(96, 160, 4), (300, 272, 40)])
def test_factorize_of_a_matrix_that_is_not_finite(d, k, rank, bad):
    """It comes back, says so in its results, and they do not depend on what the workspace held."""
    import torch
    from paper_2311_12023_amd import lq
    w = torch.from_numpy(np.random.default_rng(d).standard_normal((d, k)).astype(np.float32)).cuda()
    w[7, 11] = bad
    results = []
    for fill in (0, 0x5b):
        ws = torch.full((lq._lib.lq_factorize_workspace_bytes(d, k, rank, None) + 256,), fill, dtype=torch.uint8, device="cuda")
        l1, l2, sigma = lq.factorize(w, rank, seed=3, workspace=ws)
        assert not np.isfinite(sigma).all() or not torch.isfinite(l1).all() or not torch.isfinite(l2).all()
        results.append((l1.cpu().numpy(), l2.cpu().numpy(), sigma))
    for a, b in zip(*results):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("l,m,batch,chunks", [(32, 100, 3, 16), (64, 1000, 5, 1), (96, 333, 12, 16), (128, 2049, 2, 128),
                                               (160, 500, 3, 7)])
def test_gram_of_a_batch(l, m, batch, chunks):
    """Problems a stride apart, scratch for one chunk of columns up to all of them.  A sum of m products of fp32 numbers in
    fp64: m roundings of 2^-53."""
    import torch
    L = load()
    ld, rng = (m + 15) // 16 * 16, np.random.default_rng(l)
    stride = l * ld + 64
    x = np.full((batch, stride), np.nan, np.float32)
    xs = x[:, :l * ld].reshape(batch, l, ld)
    xs[:, :, :m] = rng.standard_normal((batch, l, m)) * 10.0 ** np.arange(batch)[:, None, None]   # the padding stays NaN
    xt = torch.from_numpy(x).cuda()
    nd = batch * l * l * chunks
    part = torch.full((nd + 1,), float("nan"), dtype=torch.float64, device="cuda")
    g = torch.full((batch + 1, l, l), float("nan"), dtype=torch.float64, device="cuda")
    assert L.lq_test_gram(xt.data_ptr(), l, m, ld, stride, part.data_ptr(), nd, g.data_ptr(), batch, None) == 0
    torch.cuda.synchronize()
    v = xs[:, :, :m].astype(np.float64)
    assert np.all(np.abs(g[:batch].cpu().numpy() - v @ v.transpose(0, 2, 1)) <= 2.0 ** -52 * m * (np.abs(v) @ np.abs(v).transpose(0, 2, 1)))
    assert torch.isnan(g[batch]).all() and torch.isnan(part[nd])


@pytest.mark.parametrize("l", [32, 96])
@pytest.mark.parametrize("chunks", [1, 2, 15, 16, 17, 32, 33, 113, 127, 128])
def test_gram_adds_every_chunk(l, chunks):
    """Chunks of two groups of 16 columns, one to eight wavefronts that add them, the last range shorter than the others.
    Tolerance as for a batch."""
    import torch
    L = load()
    m, ld = 32 * chunks - 5, 32 * chunks
    x = torch.full((l, ld), float("nan"), device="cuda")
    x[:, :m] = torch.from_numpy(np.random.default_rng(chunks).standard_normal((l, m)).astype(np.float32)).cuda()
    nd = l * l * 128
    part = torch.full((nd,), float("nan"), dtype=torch.float64, device="cuda")
    g = torch.empty((l, l), dtype=torch.float64, device="cuda")
    assert L.lq_test_gram(x.data_ptr(), l, m, ld, 0, part.data_ptr(), nd, g.data_ptr(), 1, None) == 0
    torch.cuda.synchronize()
    v = x[:, :m].double().cpu().numpy()
    assert np.all(np.abs(g.cpu().numpy() - v @ v.T) <= 2.0 ** -52 * m * (np.abs(v) @ np.abs(v).T))


@pytest.mark.parametrize("l", [32, 64, 96, 128])
@pytest.mark.parametrize("lower", [False, True])
@pytest.mark.parametrize("batch,ld0,ld1", [(1, 32, 0), (3, 96, 0), (4, 160, 64), (2, 1056, 2080)])
def test_rotate_of_a_batch(l, lower, batch, ld0, ld1):
    """One or two matrices per problem, a stride apart.  fp32 sums over l terms: l * 2^-24 of the terms' magnitudes."""
    import torch
    L = load()
    rng = np.random.default_rng(l + ld0)
    u = rng.standard_normal((batch, l, l)).astype(np.float32)
    if lower:
        u = np.tril(u)
    put = lambda v: torch.from_numpy(v).cuda()
    mats = []
    for ld in (ld0, ld1):
        if ld:
            a = rng.standard_normal((batch, l + 1, ld)).astype(np.float32)        # a row between the problems
            mats.append((ld, a, put(a), torch.full(a.shape, 7.0, dtype=torch.float32, device="cuda")))
    ptr = lambda i, j: mats[i][j].data_ptr() if i < len(mats) else None
    ut = put(u)
    assert L.lq_test_rotate(l, ut.data_ptr(), l * l, int(lower), ptr(0, 2), ptr(0, 3), ld0, (l + 1) * ld0, ptr(1, 2), ptr(1, 3),
                            ld1, (l + 1) * ld1, batch, None) == 0
    torch.cuda.synchronize()
    for ld, a, _, c in mats:
        got, v = c.cpu().numpy(), a[:, :l].astype(np.float64)
        assert np.all(np.abs(got[:, :l] - u @ v) <= 2.0 ** -24 * (l + 1) * (np.abs(u).astype(np.float64) @ np.abs(v)))
        assert np.all(got[:, l] == 7.0)


@pytest.mark.parametrize("d,k,rank", [(192, 256, 4), (1500, 640, 16), (640, 1504, 16)])
def test_factorize_with_dominant_directions(d, k, rank):
    """Dominant directions that the cold start locks (the filter step then removes them from every row), up to more than the
    eight of its middle size: singular values against LAPACK at the 1e-4 of the decomposition's tests."""
    import torch
    from paper_2311_12023_amd import lq
    rng = np.random.default_rng(d + rank)
    for dominant in (1, 4, 7, 13):
        n = min(d, k)
        s = np.concatenate([40.0 * 0.9 ** np.arange(dominant), 1.0 + 0.1 * np.sort(rng.random(n - dominant))[::-1]])
        u, _ = np.linalg.qr(rng.standard_normal((d, n)))
        v, _ = np.linalg.qr(rng.standard_normal((k, n)))
        a = ((u * s) @ v.T).astype(np.float32)
        l1, l2, sigma = lq.factorize(torch.from_numpy(a).cuda(), rank, seed=3)
        ref = np.linalg.svd(a.astype(np.float64), compute_uv=False)[:rank]
        assert np.max(np.abs(sigma - ref) / ref) < 1e-4, dominant
        assert torch.isfinite(l1).all() and torch.isfinite(l2).all()


@pytest.mark.parametrize("d,k,rank", [(33, 48, 1), (65, 400, 15), (130, 144, 16), (96, 1040, 17), (192, 272, 97), (160, 256, 128)])
def test_error_with_packed_factors(d, k, rank):
    """The error that the decomposition reports comes from the factors packed as 16-bit pairs; it equals the error of the
    factors returned.  An entry is off by at most 2^-17 of itself and the product of the two low parts is left out, so the
    product is off by less than 2^-15 |L1| |L2|; 1e-6 covers the 32-bit subtraction."""
    import torch
    from paper_2311_12023_amd import lq
    w = gen.weight_matrix(d, k, 700 + rank, min(rank, 8))
    r = lq.decompose(torch.from_numpy(w).cuda(), rank, lq.config(4, 16, 16), 2, seed=5, want_dense=True)
    l1, l2, q = (r[n].cpu().numpy().astype(np.float64) for n in ("L1", "L2", "Q"))
    ref = np.linalg.norm(w - q - l1 @ l2)
    assert abs(r["err"] - ref) <= 2.0 ** -15 * np.linalg.norm(np.abs(l1) @ np.abs(l2)) + 1e-6 * ref
