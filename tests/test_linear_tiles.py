"""The projection's smaller workgroup tiles (128 x 128 and 64 x 128 outputs, FA_OPT_LINEAR_TILE of include/fa.h): every
tile sums an output's products in the same order, so y is the 128 x 256 tile's bit for bit, and that one's error bounds
against the fp64 oracle hold."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
from gpu_util import run_attn_linear


# B, H, Nq, D, N: one k-tile, fewer k-tiles than loads run ahead, as many, more; rows that end at, before and after a
# 64- and a 128-row tile
SHAPES = [(1, 1, 64, 64, 256), (2, 3, 129, 64, 512), (1, 5, 200, 64, 256), (1, 3, 65, 128, 768), (2, 9, 191, 128, 256)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("rows_per_block", [0, 100])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_tiles_change_no_bit(oracle, shape, rows_per_block, dtype):
    B, H, Nq, D, N = shape
    print(f"case linear tiles shape={shape} rpb={rows_per_block} dtype={dtype}", flush=True)
    rng = np.random.default_rng(hash((shape, dtype)) % (2**32))
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, Nq, D), dtype=np.float32), dtype) for _ in range(3))
    w = I.f32_to_bits(rng.standard_normal((H * D, N), dtype=np.float32) / np.float32(math.sqrt(H * D)), dtype)
    scale = 1.0 / math.sqrt(D)
    y_ref = oracle.attention_linear(q, k, v, w, scale, True, dtype)
    ys = []
    for tile in (128, 128128, 64128, fa.FA_AUTO):
        fa.fa_set_option(fa.FA_OPT_LINEAR_TILE, tile)
        ys.append(run_attn_linear(q, k, v, w, scale, True, dtype, rows_per_block=rows_per_block)[2])
        assert np.abs(ys[-1].astype(np.float64) - y_ref).max() <= 1e-2      # one error of o, see test_attn_linear.py
        assert np.array_equal(ys[-1], ys[0]), tile
