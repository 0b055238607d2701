"""Quantize of more weights than one grid can hold: a grid has fewer than 2^32 threads.  Needs no GPU (hip_stub.py)."""
import pytest

import hip_stub


@pytest.mark.parametrize("block,scale_block", [(16, 16), (64, 128), (64, 256)])     # 256, 512 and 1024 lanes
@pytest.mark.parametrize("runs", [1, 1 << 30, (1 << 30) + 64, (1 << 32) + 64])
def test_every_run_has_a_lane(tmp_path, block, scale_block, runs):
    hip_stub.run(tmp_path, r"""
block, scale_block, runs = map(int, args)
p = vp(4096)
n = max(16 * runs, block) // block * block
assert L.lq_nf_quantize(p, n, Cfg(2, block, scale_block, 8, 0), p, p, p, None) == 0
assert stub.stub_most_threads() < 2.0 ** 32
assert n // 16 <= stub.stub_all_threads() < n // 16 + 1024
""", block, scale_block, runs)
