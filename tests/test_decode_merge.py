"""The decoding step in several runs per head, merged by the workgroup that finishes a head's last run: up to D/4 runs in the
decode kernel itself, more through the second kernel.  Marks of the runs stand in o meanwhile, so o is not cleared between calls
here: it holds the previous call's results, and under a replayed graph those of the same call."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
from gpu_util import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("D,runs", [(64, 2), (64, 15), (64, 16), (64, 17), (128, 3), (128, 8), (128, 9), (128, 31), (128, 32), (128, 33)])
def test_merge_in_the_decode_kernel(oracle, D, runs, dtype):
    import torch
    print(f"case merge D={D} runs={runs} dtype={dtype}", flush=True)
    rng = np.random.default_rng(1000 * D + 10 * runs + dtype)
    B, H, Nk = 2, 3, 64 * runs + 37
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, n, D), dtype=np.float32), dtype) for n in (1, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    klen = [Nk, 5]                       # the second entry has fewer keys than runs: most of its runs see none
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(a.view(np.int16)).to(dev) for a in (q, k, v))
    tlen = torch.tensor(klen, dtype=torch.int32, device=dev)
    plan = fa.fa_fwd_splitkv_plan(B, H, 1, Nk, D, 1, dtype, runs)
    assert plan.nsplit == runs and plan.streaming
    ws = torch.full((plan.workspace_bytes // 4,), float("nan"), dtype=torch.float32, device=dev)
    out = [(torch.full((B, H, 1, D), 0x7E00, dtype=torch.int16, device=dev), torch.full((B, H, 1), float("nan"), device=dev)) for _ in range(2)]

    def call(i, stream):
        o, lse = out[i]
        if i == 0:
            fa.fa_fwd_splitkv(tq, tk, tv, o, lse, B, H, 1, Nk, D, scale, 1, dtype, runs, ws, plan.workspace_bytes, stream)
        else:
            fa.fa_decode_masked(tq, tk, tv, o, lse, B, H, Nk, D, scale, -1, 0, 0, tlen, dtype, runs, ws, plan.workspace_bytes, stream, 1)

    def check(i, name):
        torch.cuda.synchronize()
        o, lse = (x.cpu().numpy() for x in out[i])
        for b in range(B):
            n = Nk if i == 0 else klen[b]
            o_ref, lse_ref = oracle.attention_fwd(q[b:b + 1], k[b:b + 1, :, :n].copy(), v[b:b + 1, :, :n].copy(), scale, True, dtype)
            check_against_oracle(o[b:b + 1].view(np.uint16), lse[b:b + 1], o_ref, lse_ref, dtype, f"{name} D={D} runs={runs} entry {b}")
        return o, lse

    side = torch.cuda.Stream()
    for i in range(2):
        for _ in range(3):
            call(i, torch.cuda.current_stream().cuda_stream)
        first = check(i, "eager")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(i, side.cuda_stream)
        for _ in range(3):
            graph.replay()
            again = check(i, "replay")
            assert all(np.array_equal(a, b) for a, b in zip(first, again))
            call(i, torch.cuda.current_stream().cuda_stream)     # another call, another mark, in the same o
