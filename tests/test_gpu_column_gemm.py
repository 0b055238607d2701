"""The cold start's products of one problem (column_gemm_kernel, the sum of its ranges, operand layout in and out) and the filter
step that reads and writes them, at the edges of tiles, steps and ranges, against numpy in fp64.

Tolerance of a product: three bf16 MFMAs per product leave 2^-16 of it, which over K terms of random sign grows like sqrt(K):
2e-5 sqrt(K) in the root mean square, 1.5e-4 sqrt(K) at worst, as for wide_gemm_kernel's split mode."""
import numpy as np
import pytest

from testing_lib import load

pytestmark = pytest.mark.gpu


def up64(x):
    return (x + 63) // 64 * 64


def _bf16(v):
    """fp32 -> bf16, to nearest even, as bits and as fp32."""
    u = np.ascontiguousarray(v, np.float32).view(np.uint32)
    r = ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    return r, (r.astype(np.uint32) << 16).view(np.float32)


def _pack(x):
    """[k / 32][row / 16][hi, lo][lane = 16 q + n][8]: row n of the tile, k = 4 q + 0..3 and 16 + 4 q + 0..3."""
    l, ld = x.shape
    hi, back = _bf16(x)
    lo, _ = _bf16(x - back)
    out = np.stack([hi, lo])                                            # part, row, k
    out = out.reshape(2, l // 16, 16, ld // 32, 2, 4, 4)                # part, tile, n, step, half, q, 4
    return out.transpose(3, 1, 0, 5, 2, 4, 6).reshape(-1)


@pytest.mark.parametrize("l", [32, 64, 96, 128])
@pytest.mark.parametrize("mode,big,K", [(0, 1, 16), (0, 65, 48), (0, 200, 1040), (0, 515, 752), (1, 16, 1), (1, 64, 33), (1, 208, 1031),
                                        (1, 528, 769)])
@pytest.mark.parametrize("nt,ranges", [(0, 0), (1, 1), (2, 1), (4, 1), (1, 3), (2, 8), (4, 2)])
def test_column_gemm(l, mode, big, K, nt, ranges):
    import torch
    L = load()
    rng = np.random.default_rng(l + big + K)
    ldx, ldc = up64(K), up64(big)
    x = np.zeros((l, ldx), np.float32)
    x[:, :K] = rng.standard_normal((l, K))
    a = rng.standard_normal((big, K) if mode == 0 else (K, big)).astype(np.float32)
    xt, at = torch.from_numpy(x).cuda(), torch.from_numpy(a).cuda()
    ct = torch.full((l, ldc), 7.0, device="cuda")
    packed = torch.full((2 * l * ldc,), -1, dtype=torch.int16, device="cuda")
    scratch = torch.full((l * (ldx + 8 * ldc),), float("nan"), device="cuda")
    args = (mode, l, big, K, xt.data_ptr(), ldx, at.data_ptr(), a.shape[1], ct.data_ptr(), ldc, packed.data_ptr(), nt, ranges,
            scratch.data_ptr(), None)
    assert L.lq_test_column_gemm(*args) == 0
    torch.cuda.synchronize()
    got = ct.cpu().numpy()
    ref = x[:, :K].astype(np.float64) @ (a.T if mode == 0 else a).astype(np.float64)
    err = got[:, :big] - ref
    assert np.max(np.abs(err)) < 1.5e-4 * np.sqrt(K) and np.sqrt(np.mean(err ** 2)) < 2e-5 * np.sqrt(K)
    assert np.all(got[:, big:] == 7.0)
    full = np.where(np.arange(ldc) < big, got, np.float32(0))
    assert np.array_equal(packed.cpu().numpy().view(np.uint16), _pack(full))
    again = torch.full((l, ldc), 7.0, device="cuda")
    assert L.lq_test_column_gemm(*args[:8], again.data_ptr(), *args[9:]) == 0 and torch.equal(ct, again)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("mode,big,K", [(0, 65, 48), (0, 515, 752), (1, 64, 33), (1, 528, 769)])
@pytest.mark.parametrize("nt,ranges", [(0, 0), (1, 3), (4, 2)])
def test_column_gemm_keeps_what_is_not_finite_where_it_belongs(mode, big, K, nt, ranges, bad):
    """An entry of A reaches its own column of the product (every row: X has no zeros), one of X its own row, also where they lie
    at the end of a ragged reduction or in the last column of a tile, whose neighbours past the edge are read in its place."""
    import torch
    L = load()
    l, rng, ldx, ldc = 64, np.random.default_rng(big), up64(K), up64(big)
    x = np.zeros((l, ldx), np.float32)
    x[:, :K] = rng.standard_normal((l, K))
    a = rng.standard_normal((big, K)).astype(np.float32)
    a[big - 1, K - 1] = a[3, 0] = bad
    x[17, K - 1] = x[40, 5] = bad
    at = torch.from_numpy(np.ascontiguousarray(a if mode == 0 else a.T)).cuda()
    xt, ct = torch.from_numpy(x).cuda(), torch.full((l, ldc), 7.0, device="cuda")
    packed = torch.full((2 * l * ldc,), -1, dtype=torch.int16, device="cuda")
    scratch = torch.full((l * (ldx + 8 * ldc),), float("nan"), device="cuda")
    assert L.lq_test_column_gemm(mode, l, big, K, xt.data_ptr(), ldx, at.data_ptr(), at.shape[1], ct.data_ptr(), ldc, packed.data_ptr(),
                                 nt, ranges, scratch.data_ptr(), None) == 0
    got = ct.cpu().numpy()[:, :big]
    hit = np.zeros((l, big), bool)
    hit[[17, 40]] = True
    hit[:, [3, big - 1]] = True
    assert np.array_equal(~np.isfinite(got), hit)
    with np.errstate(invalid="ignore"):
        ref = x[:, :K].astype(np.float64) @ a.T.astype(np.float64)
    assert np.max(np.abs(got - ref)[~hit]) < 1.5e-4 * np.sqrt(K)


@pytest.mark.parametrize("l,m", [(32, 100), (96, 1003), (128, 16400)])
@pytest.mark.parametrize("locked", [0, 3, 16])
@pytest.mark.parametrize("ranges", [0, 1, 4])
@pytest.mark.parametrize("terms", [1, 2, 3])
def test_filter_step_of_ranges(l, m, locked, ranges, terms):
    """X as the sum of ranges, the combination, the deflation (rows longer than 16384 columns take separate launches) and the operand
    layout.  Everything is fp32 arithmetic on a few terms and one sum over m: 1e-5 of the largest entry."""
    import torch
    L = load()
    ld, rng = up64(m), np.random.default_rng(l + m + locked)
    pad = lambda *shape: np.concatenate([rng.standard_normal((*shape, m)), np.zeros((*shape, ld - m))], -1).astype(np.float32)
    q, _ = np.linalg.qr(rng.standard_normal((m, 16)))
    lrows = np.zeros((l, ld), np.float32)
    lrows[:16, :m] = q.T
    x, y, z, parts = pad(l), pad(l), pad(l), pad(max(ranges, 1), l)
    dev = lambda v: torch.from_numpy(v).cuda()
    xt, yt, zt, lt, pt = dev(x), dev(y), dev(z), dev(lrows), dev(parts)
    packed = torch.full((2 * l * ld,), -1, dtype=torch.int16, device="cuda")
    ptr = lambda t, want: t.data_ptr() if want else None
    assert L.lq_test_filter_step_packed(xt.data_ptr(), 0.75, ptr(yt, terms > 1), -2.0, ptr(zt, terms > 2), 0.5, lt.data_ptr(), l, locked,
                                        m, ld, ptr(pt, ranges), ranges or 1, packed.data_ptr(), None) == 0
    torch.cuda.synchronize()
    got = xt.cpu().numpy()
    v = parts.astype(np.float64).sum(0) if ranges else x.astype(np.float64)
    if terms > 1:
        v = 0.75 * v - 2.0 * y
    if terms > 2:
        v = v + 0.5 * z
    lk = lrows[:locked].astype(np.float64)
    v = v - (v @ lk.T) @ lk
    v[:locked] = lk
    assert np.max(np.abs(got - v)) < 1e-5 * np.max(np.abs(v))
    assert np.all(got[:, m:] == 0)
    assert np.array_equal(packed.cpu().numpy().view(np.uint16), _pack(got))
