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
