"""The eigen-solver of the Rayleigh-Ritz step over the spectra that decide its route: separated eigenvalues (tridiagonal
route), close ones (the same with a joint orthonormalisation), repeated and zero ones (one-sided Jacobi inside the same
launch), graded and diagonal matrices.

Tolerances: rows of fp32 numbers that are orthonormal to 2^-24 per entry, or to 1e-6 per pair on the Jacobi route and at
the smallest gap the tridiagonal route accepts (2e-9 of the largest eigenvalue): 4e-6.  A Rayleigh quotient misses its
eigenvalue by the square of the vector's error, or by the vector's rounding (2^-24 per entry, both factors, entries of G up
to lambda_1): 4e-7 of the largest eigenvalue covers both."""
import numpy as np
import pytest

from testing_lib import load

pytestmark = pytest.mark.gpu


def _spectrum(kind, l, rng):
    if kind == "flat":                       # a bulk under a few dominant values, as a weight matrix has it
        return np.concatenate([[900.0, 400.0, 120.0], 1.08 - 0.08 * np.sort(rng.random(l - 3))])
    if kind == "geometric":
        return 0.8 ** np.arange(l)
    if kind == "repeated":
        return np.repeat([7.0, 3.0], l // 2)
    if kind == "low_rank":
        return np.concatenate([np.linspace(2.0, 1.0, l // 4), np.zeros(l - l // 4)])
    if kind == "one_pair":                   # two eigenvalues 1e-11 apart among separated ones
        s = np.linspace(4.0, 1.0, l)
        s[5] = s[4] * (1 - 1e-11)
        return s
    if kind == "noise_floor":                # the residual of an 8-bit configuration: a cluster far below the rest
        return np.concatenate([np.linspace(900.0, 1.0, l - l // 3), 1e-6 * (1.0 + 0.03 * np.sort(rng.random(l // 3)))])
    if kind == "smallest_gap":               # just above the line of the tridiagonal route
        s = np.linspace(4.0, 1.0, l)
        s[5] = s[4] - 1.0e-8 * 4.0
        return s
    raise ValueError(kind)


def _solve(g):
    import torch
    L = load()
    l = g.shape[0]
    gt = torch.from_numpy(g.copy()).cuda()
    ut = torch.full((l, l), float("nan"), dtype=torch.float32, device="cuda")
    lam = torch.full((l,), float("nan"), dtype=torch.float64, device="cuda")
    assert L.lq_test_sym_eig_fast(gt.data_ptr(), l, ut.data_ptr(), lam.data_ptr(), None) == 0
    torch.cuda.synchronize()
    return ut.cpu().numpy().astype(np.float64), lam.cpu().numpy()


@pytest.mark.parametrize("l", [32, 64, 96, 128])
@pytest.mark.parametrize("kind", ["flat", "geometric", "repeated", "low_rank", "one_pair", "smallest_gap", "noise_floor"])
@pytest.mark.parametrize("scale", [1.0, 1e-13, 1e11])
def test_spectra(l, kind, scale):
    rng = np.random.default_rng(l)
    s = _spectrum(kind, l, rng)
    q, _ = np.linalg.qr(rng.standard_normal((l, l)))
    g = (q * s) @ q.T * scale
    g = (g + g.T) / 2
    u, lam = _solve(g)
    ref = np.sort(s)[::-1] * scale
    assert np.all(np.isfinite(u)) and np.all(np.diff(lam) <= 0)
    assert np.max(np.abs(u @ u.T - np.eye(l))) < 4e-6
    rq = np.einsum("ij,jk,ik->i", u, g, u)
    assert np.max(np.abs(rq - ref)) < 4e-7 * ref[0]
    # Eigenvalues of a route in fp64: the reduction and the multisection leave about l roundings of lambda_1.  The Jacobi
    # route, in fp32, misses this by orders of magnitude, so it also says that the others were not left for it.
    off_jacobi = kind not in ("repeated", "low_rank") and not (kind == "geometric" and l > 64)
    assert np.max(np.abs(lam - ref)) < (1e-13 * l if off_jacobi else 1e-4) * ref[0]


@pytest.mark.parametrize("l", [32, 64, 96, 128])
def test_diagonal_and_zero_matrices(l):
    d = np.arange(l, 0, -1.0)
    perm = np.random.default_rng(l).permutation(l)
    u, lam = _solve(np.diag(d[perm]))
    assert np.allclose(lam, d, rtol=1e-6)
    assert np.array_equal(np.abs(u), np.eye(l)[np.argsort(perm)])
    u, lam = _solve(np.zeros((l, l)))
    assert np.all(lam == 0) and np.max(np.abs(u @ u.T - np.eye(l))) == 0


@pytest.mark.parametrize("l", [32, 64, 96, 128])
def test_problems_of_a_batch_are_independent(l):
    """Problems of every route side by side in one launch, in scratch full of NaN: each comes out as it does alone."""
    import torch
    L = load()
    kinds = ["flat", "repeated", "noise_floor", "geometric", "low_rank", "smallest_gap"]
    rng = np.random.default_rng(l)
    gs = []
    for i, kind in enumerate(kinds):
        q, _ = np.linalg.qr(rng.standard_normal((l, l)))
        g = (q * _spectrum(kind, l, rng)) @ q.T * 10.0 ** (3 * i - 6)
        gs.append((g + g.T) / 2)
    n = len(kinds)
    gt = torch.from_numpy(np.stack(gs)).cuda()
    nan = lambda dtype, *shape: torch.full(shape, float("nan"), dtype=dtype, device="cuda")
    work, ut, lam = nan(torch.float64, n * 2 * l * l), nan(torch.float32, n + 1, l, l), nan(torch.float64, n + 1, l)
    assert L.lq_test_sym_eig_batch(gt.data_ptr(), l, n, work.data_ptr(), ut.data_ptr(), lam.data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert torch.isnan(ut[n]).all() and torch.isnan(lam[n]).all()
    for i in range(n):
        u1, lam1 = _solve(gs[i])
        assert np.array_equal(ut[i].cpu().numpy().astype(np.float64), u1), kinds[i]
        assert np.array_equal(lam[i].cpu().numpy(), lam1), kinds[i]


@pytest.mark.parametrize("l", [96, 128])
def test_which_launch_makes_the_vectors(l):
    """From l = 96 on the vectors of separated eigenvalues come from a second launch.  Whether a problem has left them to it is
    said by a word of the scratch, which is written for every problem, and not by what stood in Ut before."""
    import torch
    L = load()
    rng = np.random.default_rng(l)
    q, _ = np.linalg.qr(rng.standard_normal((l, l)))
    work = torch.full((2 * l * l,), float("nan"), dtype=torch.float64, device="cuda")
    lam = torch.empty(l, dtype=torch.float64, device="cuda")
    ne = l // 16                             # behind the packed reflectors, {d, e^2}, e, h, the eigenvalues and their bound
    at = 8 * 256 * (ne * ne - ne * (ne - 1) // 2) + 16 * (l + 1) + 3 * 8 * l + 8
    wanted = work.view(torch.int32)[at // 4]
    for kind, second in (("flat", 1), ("noise_floor", 0), ("smallest_gap", 1), ("repeated", 0)):
        g = (q * _spectrum(kind, l, rng)) @ q.T
        g = (g + g.T) / 2
        gt = torch.from_numpy(g.copy()).cuda()
        wanted.fill_(7)
        ut = torch.full((l, l), float("nan"), dtype=torch.float32, device="cuda")
        assert L.lq_test_sym_eig_batch(gt.data_ptr(), l, 1, work.data_ptr(), ut.data_ptr(), lam.data_ptr(), None) == 0
        assert wanted.item() == second, kind
        u = ut.cpu().numpy().astype(np.float64)
        assert np.max(np.abs(u @ u.T - np.eye(l))) < 4e-6, kind


@pytest.mark.parametrize("l", [32, 64, 96, 128, 160])
@pytest.mark.parametrize("kind", ["nan", "one_nan", "inf"])
def test_every_row_is_written_for_a_matrix_that_is_not_finite(l, kind):
    """Nothing of what the outputs held before is left, so the result does not depend on it."""
    import torch
    L = load()
    g = np.random.default_rng(l).standard_normal((l, l))
    g = g @ g.T
    if kind == "nan":
        g[:] = np.nan
    elif kind == "one_nan":
        g[3, 17] = g[17, 3] = np.nan
    else:
        g[5, 5] = np.inf
    results = []
    for before in (7.0, -3.0):
        gt = torch.from_numpy(g.copy()).cuda()
        work = torch.full((2 * l * l,), before, dtype=torch.float64, device="cuda")
        ut = torch.full((l, l), before, dtype=torch.float32, device="cuda")
        lam = torch.full((l,), before, dtype=torch.float64, device="cuda")
        if l <= 128:
            assert L.lq_test_sym_eig_batch(gt.data_ptr(), l, 1, work.data_ptr(), ut.data_ptr(), lam.data_ptr(), None) == 0
        else:
            assert L.lq_test_sym_eig(gt.data_ptr(), l, ut.data_ptr(), lam.data_ptr(), work.data_ptr(), None) == 0
        assert not (ut == before).any() and not (lam == before).any()
        results.append((ut.cpu().numpy(), lam.cpu().numpy()))
    for a, b in zip(*results):
        assert np.array_equal(a, b, equal_nan=True)


def _nested_clusters(l, seed):
    """Clusters of 1 to 7 eigenvalues that start on points of a grid of 1/64, each point once, 1e-2, 1e-4 or 1e-7 apart inside;
    the largest is 1 and no two are within 1e-8, which leaves them all to the tridiagonal route (its line: 2e-9 of a bound below 3)."""
    rng = np.random.default_rng(100 * l + seed)
    s, tops = [1.0], iter(rng.permutation(np.arange(8, 64)) / 64)
    while len(s) < l:
        m = min(int(rng.integers(1, 8)), l - len(s))
        s += list(next(tops) - 10.0 ** -float(rng.choice([2, 4, 7])) * (np.arange(m) + 0.3 * rng.random(m)))
    s = np.array(s)
    assert np.min(np.diff(np.sort(s))) > 1e-8 and np.min(s) > 0
    q, _ = np.linalg.qr(rng.standard_normal((l, l)))
    return s, q


@pytest.mark.parametrize("l", [32, 64, 96, 128])
@pytest.mark.parametrize("seed", range(4))
def test_eigenvalues_of_nested_clusters(l, seed):
    """Groups of every size share an interval of the eigenvalue search for a while, also on the points of a uniform grid.  The
    reduction and the search leave about l roundings of lambda_1."""
    s, q = _nested_clusters(l, seed)
    g = (q * s) @ q.T
    g = (g + g.T) / 2
    u, lam = _solve(g)
    assert np.max(np.abs(lam - np.linalg.eigvalsh(g)[::-1])) < 1e-13 * l
    assert np.max(np.abs(u @ u.T - np.eye(l))) < 4e-6


@pytest.mark.parametrize("l", [32, 64, 96, 128])
def test_eigenvalues_of_repeated_clusters(l):
    """The same with eigenvalues that coincide, which may end on the Jacobi route (fp32: 1e-4 as in test_spectra)."""
    s, q = _nested_clusters(l, 0)
    s[l // 2:] = s[:l // 2]
    g = (q * s) @ q.T
    g = (g + g.T) / 2
    u, lam = _solve(g)
    assert np.max(np.abs(lam - np.linalg.eigvalsh(g)[::-1])) < 1e-4
    assert np.max(np.abs(u @ u.T - np.eye(l))) < 4e-6
