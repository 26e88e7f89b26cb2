"""The kernel on waves of 64 rows where fa_fwd takes it for walks below 4096 keys (plans report FA_MODE_WIDE on 256 rows, 256 threads):
either side of the lines, and results against the oracle on sampled rows: ragged and whole tiles at the end of the walk,
odd numbers of tiles, diagonals that do not start on a tile, and both row sums in fp16."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
from gpu_util import check_against_oracle, run_fa_fwd, run_fa_fwd_splitkv

D = 128


def on_rows64(B, H, Nq, Nk, causal, dtype=I.BF16):
    p = fa.fa_fwd_plan(B, H, Nq, Nk, D, causal, dtype)
    return p.mode == fa.FA_MODE_WIDE and p.block_m == 256 and p.threads == 256


@pytest.mark.parametrize("B,H,Nq,Nk,causal,want", [
    (1, 32, 2048, 960, 0, True), (1, 32, 2048, 896, 0, False), (4, 32, 1024, 1216, 0, True), (4, 32, 1024, 1152, 0, False),
    (1, 32, 2048, 2047, 0, False), (1, 32, 2048, 2049, 0, True), (1, 40, 2048, 2048, 0, False),
    (1, 32, 2048, 4096, 1, True), (1, 32, 2048, 3072, 1, False), (1, 32, 2048, 4095, 1, False), (1, 32, 6144, 6144, 1, False),
    (1, 40, 2048, 4096, 1, False), (1, 128, 4096, 4096, 1, False), (4, 32, 1024, 2880, 1, False), (4, 32, 1024, 2944, 1, True)])
def test_plan(B, H, Nq, Nk, causal, want):
    assert on_rows64(B, H, Nq, Nk, causal) is want


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("B,H,Nq,Nk,causal", [
    (1, 64, 1000, 1088, False), (1, 64, 1024, 2111, False), (1, 128, 512, 1216, False), (1, 128, 400, 2944, True),
    (1, 128, 511, 3008, True), (1, 256, 257, 2560, True)])
def test_sampled_rows(oracle, B, H, Nq, Nk, causal, dtype):
    print(f"case rows64 choice {(B, H, Nq, Nk, causal)} dtype={dtype}", flush=True)
    assert on_rows64(B, H, Nq, Nk, int(causal), dtype)
    rng = np.random.default_rng(Nq + Nk + dtype)
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, n, D), dtype=np.float32), dtype) for n in (Nq, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    o, lse = run_fa_fwd(q, k, v, scale, causal, dtype)
    rows = np.unique(np.concatenate([rng.integers(0, B * H * Nq, 1000), [0, Nq - 1, B * H * Nq - 1]]))
    o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, causal, dtype, rows=rows)
    check_against_oracle(o.reshape(-1, D)[rows], lse.reshape(-1)[rows], o_ref, lse_ref, dtype, f"rows64 {(B, H, Nq, Nk)}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("H,Nq,Nk,nsplit,causal", [
    (4, 300, 2950, 2, True), (3, 520, 4480, 3, True), (2, 257, 2801, 2, False), (2, 513, 3071, 2, True)])
def test_runs_of_1400_keys_and_more(oracle, H, Nq, Nk, nsplit, causal, dtype):
    """Split-KV runs of several query blocks on that kernel: runs that start and end anywhere, ragged last tiles."""
    print(f"case rows64 runs {(H, Nq, Nk, nsplit, causal)} dtype={dtype}", flush=True)
    assert (Nk - Nq // 2 if causal else Nk) // nsplit >= 1400
    rng = np.random.default_rng(Nq + Nk + dtype)
    q, k, v = (I.f32_to_bits(rng.standard_normal((1, H, n, D), dtype=np.float32), dtype) for n in (Nq, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    o, lse, plan = run_fa_fwd_splitkv(q, k, v, scale, causal, dtype, nsplit)
    assert plan.nsplit == nsplit
    o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, causal, dtype)
    check_against_oracle(o, lse, o_ref, lse_ref, dtype, f"rows64 runs {(H, Nq, Nk, nsplit)}")
