"""The decoding step where B * H does not divide 256: the tiles of all heads laid end to end and cut into 256 equal pieces,
so that a workgroup's piece may end in one head and begin in the next, and a head's runs are merged by as many as it has."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
import options
from gpu_util import check_against_oracle, run_fa_fwd_splitkv


def test_a_head_has_no_more_runs_than_the_plan_reports():
    for heads in (3, 5, 7, 36, 40, 48, 60, 84, 150, 255, 257, 300, 384):
        for tiles in (1, 14, 15, 20, 35, 137, 1000, 4097):
            p = fa.fa_fwd_splitkv_plan(1, heads, 1, tiles * 64 - 3, 64, 1, 0)
            total = heads * tiles
            if total < 256 * 20:
                assert (p.grid_x, p.grid_y) == (heads, p.nsplit)
                continue
            assert (p.grid_x, p.grid_y) == (256, 1)
            bounds = np.arange(257, dtype=np.int64) * total // 256
            owner = np.searchsorted(bounds, np.arange(total), side="right") - 1
            first, last = owner[::tiles], owner[tiles - 1::tiles]
            assert (last - first + 1).max() <= p.nsplit <= math.ceil(256 / heads) + 1
            assert p.workspace_bytes == p.nsplit * heads * (64 + 2) * 4
    for heads in (8, 32, 256, 385, 1000):      # equal runs, or one per head
        p = fa.fa_fwd_splitkv_plan(1, heads, 1, 64000, 128, 1, 1)
        assert (p.grid_x, p.grid_y) == (heads, max(1, 256 // heads))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("B,H,Nk,D", [(1, 40, 8200, 64), (1, 48, 6913, 128), (3, 100, 1153, 64), (1, 3, 110001, 128),
                                      (1, 255, 1400, 64), (1, 257, 1344, 128), (2, 192, 900, 64)])
def test_pieces_elementwise(oracle, B, H, Nk, D, dtype):
    print(f"case pieces B={B} H={H} Nk={Nk} D={D} dtype={dtype}", flush=True)
    rng = np.random.default_rng(hash((B, H, Nk, D, dtype)) % (2**32))
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, n, D), dtype=np.float32), dtype) for n in (1, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, True, dtype)
    o, lse, plan = run_fa_fwd_splitkv(q, k, v, scale, True, dtype)
    assert plan.streaming and (plan.grid_x, plan.grid_y) == (256, 1)
    check_against_oracle(o, lse, o_ref, lse_ref, dtype, f"pieces {(B, H, Nk, D)} dt={dtype}")
    options.set_decode("mfma")            # the tile kernel, equal runs
    o2, lse2, plan2 = run_fa_fwd_splitkv(q, k, v, scale, True, dtype)
    assert not plan2.streaming
    check_against_oracle(o2, lse2, o_ref, lse_ref, dtype, f"pieces, tile kernel {(B, H, Nk, D)}")
