"""fa_fwd's choice at D = 64 between two groups of waves on alternate tiles (FA_MODE_SPLIT) and the other forms, on either side of its
lines for many blocks of rows; the calls beside the lines against the oracle on sampled rows."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
from gpu_util import check_against_oracle, run_fa_fwd

D = 64
SPLIT, WIDE, FOLD = fa.FA_MODE_SPLIT, fa.FA_MODE_WIDE, fa.FA_MODE_WIDE_FOLD


@pytest.mark.parametrize("B,H,Nq,Nk,causal,mode,rows", [
    (13, 5, 1896, 1896, 0, SPLIT, 128), (1, 20, 7058, 7058, 0, SPLIT, 128), (8, 8, 2560, 2560, 0, SPLIT, 128),
    (10, 8, 1587, 1683, 0, WIDE, 256), (8, 8, 2049, 1535, 0, WIDE, 128), (8, 8, 2561, 2561, 0, WIDE, 256), (8, 8, 2048, 2048, 0, WIDE, 256),
    (2, 12, 9332, 9332, 1, SPLIT, 128), (3, 12, 7581, 7581, 1, SPLIT, 128), (4, 40, 2700, 3700, 1, SPLIT, 128),
    (2, 32, 4096, 4096, 1, FOLD, 256), (4, 20, 4300, 4300, 1, WIDE, 128),
    (1, 70, 6912, 6912, 1, SPLIT, 128), (1, 71, 6912, 6912, 1, WIDE, 128),
    (1, 16, 4000, 30000, 1, SPLIT, 128)])
def test_plan(B, H, Nq, Nk, causal, mode, rows):
    p = fa.fa_fwd_plan(B, H, Nq, Nk, D, causal, I.BF16)
    assert (p.mode, p.block_m) == (mode, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("B,H,Nq,Nk,causal", [(13, 5, 1896, 1896, False), (4, 40, 2700, 3700, True)])
def test_sampled_rows(oracle, B, H, Nq, Nk, causal, dtype):
    print(f"case form choice {(B, H, Nq, Nk, causal)} dtype={dtype}", flush=True)
    assert fa.fa_fwd_plan(B, H, Nq, Nk, D, int(causal), dtype).mode == SPLIT
    rng = np.random.default_rng(Nq + dtype)
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, n, D), dtype=np.float32), dtype) for n in (Nq, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    o, lse = run_fa_fwd(q, k, v, scale, causal, dtype)
    rows = np.unique(np.concatenate([rng.integers(0, B * H * Nq, 1000), [0, Nq - 1, B * H * Nq - 1]]))
    o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, causal, dtype, rows=rows)
    check_against_oracle(o.reshape(-1, D)[rows], lse.reshape(-1)[rows], o_ref, lse_ref, dtype, f"form choice {(B, H, Nq, Nk)}")
