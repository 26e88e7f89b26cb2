"""FA_MODE_WIDE on workgroups of four waves (FA_MODE_WIDE4 forces it): at D = 128 persistent workgroups that take block of
128 rows after block of rows from a list, at D = 64 one workgroup per block.  Same tolerances as the other modes."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
from gpu_util import check_against_oracle, run_fa_fwd


def force():
    fa.fa_set_option(fa.FA_OPT_FWD_MODE, fa.FA_MODE_WIDE4)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [0, 1])
def test_plan_of_the_four_wave_form(D, causal):
    force()
    for B, H, Nq, Nk in ((1, 1, 1000, 1000), (3, 20, 1531, 1531), (2, 5, 257, 100), (9, 40, 300, 700)):
        p = fa.fa_fwd_plan(B, H, Nq, Nk, D, causal, 0)
        nqt = -(-Nq // 128)
        assert (p.mode, p.block_m, p.threads, p.work_items) == (fa.FA_MODE_WIDE, 128, 256, B * H * nqt)
        visited = 0
        for b in range(nqt):
            last = min(b * 128 + 127, Nq - 1) + Nk - Nq if causal else Nk - 1
            visited += max(min(last, Nk - 1), -1) // 64 + 1 if last >= 0 else 0
        assert p.tiles_visited == visited * B * H
        assert p.grid % 8 == 0 and (p.grid <= 512 if D == 128 else p.grid >= p.work_items)


# B, H, Nq, Nk: an odd and an even number of tiles per block; one tile; rows past the end in the last block; more keys than
# queries and fewer (causal: blocks without a key, in the middle of a workgroup's list too); list layouts at D = 128: one
# entry per workgroup, several with all heads mixed, head by head (under five blocks per head), groups of eight heads,
# heads that do not divide by 8
SHAPES = [(1, 1, 128, 64), (1, 3, 129, 129), (1, 2, 300, 385), (2, 5, 640, 1000), (1, 9, 1100, 1100), (3, 27, 700, 500),
          (5, 14, 1000, 1000), (25, 8, 300, 320), (8, 45, 700, 700), (70, 8, 200, 190)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", SHAPES)
def test_four_wave_form_elementwise(oracle, shape, D, causal, dtype):
    B, H, Nq, Nk = shape
    print(f"case four waves shape={shape} D={D} causal={causal} dtype={dtype}", flush=True)
    force()
    rng = np.random.default_rng(hash((shape, D, causal, dtype)) % (2**32))
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, n, D), dtype=np.float32), dtype) for n in (Nq, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, causal, dtype)
    o, lse = run_fa_fwd(q, k, v, scale, causal, dtype)
    check_against_oracle(o, lse, o_ref, lse_ref, dtype, f"four waves {shape} D={D} causal={causal} dt={dtype}")


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [-0.3, 0.0, 0.7])
@pytest.mark.parametrize("D", [64, 128])
def test_four_wave_form_with_moving_maxima_and_any_scale(oracle, D, scale):
    """Logits that rise along the keys by far more than the exponent reference tolerates; a workgroup's blocks follow each
    other with references of their own, and the sign of the scale is put into Q for every block."""
    print(f"case four waves maxima D={D} scale={scale}", flush=True)
    force()
    rng = np.random.default_rng(5)
    B, H, N = 2, 41, 1000
    q, k, v = (rng.standard_normal((B, H, N, D), dtype=np.float32) for _ in range(3))
    k *= np.linspace(0.05, 4.0, N, dtype=np.float32)[None, None, :, None]
    q, k, v = (I.f32_to_bits(x, I.F16) for x in (q, k, v))
    o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, True, I.F16)
    o, lse = run_fa_fwd(q, k, v, scale, True, I.F16)
    check_against_oracle(o, lse, o_ref, lse_ref, I.F16, f"four waves maxima D={D} scale={scale}")


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
def test_four_wave_lse_counts_the_unrounded_exponentials(oracle, D):
    """fp16, two or three tiles, logits of standard deviation 4: rows ruled by one or two keys.  With the sum over rounded
    exponentials one dominant term is off by up to 2^-11, 5e-4 in lse; over the unrounded ones lse carries fp32 rounding
    only: logits up to 32 whose dot product and exponent take a few steps of 2^-19 each, 1e-5."""
    print(f"case four waves lse D={D}", flush=True)
    force()
    rng = np.random.default_rng(77 + D)
    q, k, v = (I.f32_to_bits(2 * rng.standard_normal((2, 12, n, D), dtype=np.float32), I.F16) for n in (82, 168, 168))
    scale = 1.0 / math.sqrt(D)
    _, lse_ref = oracle.attention_fwd(q, k, v, scale, True, I.F16)
    _, lse = run_fa_fwd(q, k, v, scale, True, I.F16)
    assert np.abs(lse - lse_ref).max() <= 1e-5
