"""The number of runs fa_fwd_splitkv picks for more than one query (host logic; the results at any number of runs are
checked in test_splitkv.py)."""
import math

import pytest

from paper_2410_16663_amd import binding as fa

MIB64 = 64 << 20


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("heads", [1, 5, 24, 40, 48, 64, 161, 352])
def test_runs_of_a_few_queries_fill_one_round_per_xcd(D, heads):
    slots = 32 if D == 128 else 64              # workgroups an XCD holds at a time
    for Nq in (2, 9, 16):
        for Nk in (70, 1000, 30000):
            n = fa.fa_fwd_splitkv_plan(1, heads, Nq, Nk, D, 1, 0).nsplit
            tiles = -(-Nk // 64)
            assert n == 1 or (-(-heads // 8) * n <= slots and tiles // n >= 4)
            assert n <= max(1, math.ceil(8 * slots / heads))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [0, 1])
def test_runs_of_a_chunk_stay_within_bounds(D, causal):
    for heads in (1, 5, 20, 40, 96, 400):
        for Nq in (17, 225, 512, 1000, 2049):
            for Nk in (100, 2049, 9000, 60000):
                p = fa.fa_fwd_splitkv_plan(1, heads, Nq, Nk, D, causal, 1)
                tiles = -(-Nk // 64)
                assert p.nsplit == 1 or (p.nsplit <= 64 and tiles // p.nsplit >= 4)
                # what a workgroup count alone would ask for: one per compute unit at D = 128, two at D = 64
                by_count = max(1, min(-(-(256 if D == 128 else 512) // p.work_items), tiles // 4))
                row_bytes = heads * Nq * (D + 2) * 4
                assert p.nsplit == 1 or p.workspace_bytes <= max(MIB64, by_count * row_bytes)
    # a short walk gains nothing from being cut; a long one of few query blocks does
    assert fa.fa_fwd_splitkv_plan(1, 40, 562, 690, D, 1, 0).nsplit == 1
    assert fa.fa_fwd_splitkv_plan(1, 8, 200, 40000, D, 1, 0).nsplit >= 8
