"""The decoding step in several runs per head, merged by the workgroup that finishes a head's last run: up to D/4 runs in the
decode kernel itself, more through the second kernel.  Marks of the runs stand in o meanwhile, so o is not cleared between calls
here: it holds the previous call's results, and under a replayed graph those of the same call."""
import math
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import build
from paper_2410_16663_amd import inputs as I
from gpu_util import check_against_oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

ORDER_KERNEL = """
#include <hip/hip_runtime.h>
using f32x2 = float __attribute__((ext_vector_type(2)));
FRAGMENT
extern "C" __global__ void probe(float *part, unsigned long long *tags, unsigned long long tag, float a, float b, unsigned long long *out) {
    const float x[2] = {a, b};
    store_shared<1>(part + 2, x);
    store_shared<2>(part, x);
    wait_memory();
    __hip_atomic_store(tags, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_memory();
    const unsigned long long seen = __hip_atomic_load(tags + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (seen == tag) {
        wait_memory();
        const f32x2 y = load_shared(part + 4);
        out[0] = __builtin_bit_cast(unsigned long long, y);
    }
}
"""


def test_accesses_the_merge_is_ordered_by_are_compiled_as_it_assumes(tmp_path):
    """store_shared, load_shared and the tags' accesses bear sc1 on gfx950 (past the XCD's L2) and stay on their sides of
    wait_memory; on another target the fragment does not compile."""
    with open(os.path.join(ROOT, "paper_2410_16663_amd", "csrc", "fa_decode_kernels.inc")) as f:
        src = f.read()
    begin, end = "#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)", "constexpr int DECODE_WAVES"
    assert src.count(begin) == 1 and src.count(end) == 1
    hip = tmp_path / "order.hip"
    hip.write_text(ORDER_KERNEL.replace("FRAGMENT", src[src.index(begin):src.index(end)]))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "--offload-arch=gfx950") and not f.startswith("-Rpass")]

    def compile_for(arch):
        return subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), f"--offload-arch={arch}"] + flags +
                              ["--cuda-device-only", "-S", str(hip), "-o", str(tmp_path / "order.s")], capture_output=True, text=True)

    r = compile_for("gfx950")
    assert r.returncode == 0, r.stderr
    asm = (tmp_path / "order.s").read_text()
    body = asm[asm.index("probe:"):asm.index("s_endpgm")]
    steps = re.findall(r"(global_store_\w+ .*|global_load_\w+ .*|s_waitcnt vmcnt\(0\)\s*$)", body, flags=re.M)
    kinds = ["wait" if x.startswith("s_wait") else re.match(r"global_(store|load)", x).group(1) + (" sc1" if re.search(r"\bsc1\b", x) else "")
             for x in steps]
    squeezed = [k for i, k in enumerate(kinds) if k != "wait" or i == 0 or kinds[i - 1] != "wait"]
    assert squeezed[:8] == ["store sc1", "store sc1", "wait", "store sc1", "wait", "load sc1", "wait", "load sc1"], steps
    r = compile_for("gfx1100")
    assert r.returncode != 0 and "argued for gfx950 only" in r.stderr


@pytest.mark.gpu
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


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("B,H,Nk,D", [(1, 40, 8200, 64), (1, 48, 6913, 128), (3, 100, 1153, 64)])
def test_pieces_over_their_own_results(oracle, B, H, Nk, D, dtype):
    """Equal pieces of all heads' tiles: heads of one, two and more runs beside each other, called and replayed over what the calls
    before left in o (their own results, other calls' marks overwritten)."""
    import torch
    print(f"case merge of pieces B={B} H={H} Nk={Nk} D={D} dtype={dtype}", flush=True)
    rng = np.random.default_rng(7 * Nk + D + dtype)
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, n, D), dtype=np.float32), dtype) for n in (1, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(a.view(np.int16)).to(dev) for a in (q, k, v))
    plan = fa.fa_fwd_splitkv_plan(B, H, 1, Nk, D, 1, dtype)
    assert (plan.grid_x, plan.grid_y, plan.combine_grid) == (256, 1, 0)
    ws = torch.full((plan.workspace_bytes // 4,), float("nan"), dtype=torch.float32, device=dev)
    o = torch.full((B, H, 1, D), 0x7E00, dtype=torch.int16, device=dev)
    lse = torch.full((B, H, 1), float("nan"), device=dev)

    def call(stream):
        fa.fa_fwd_splitkv(tq, tk, tv, o, lse, B, H, 1, Nk, D, scale, 1, dtype, 0, ws, plan.workspace_bytes, stream)

    def results():
        torch.cuda.synchronize()
        return o.cpu().numpy().view(np.uint16), lse.cpu().numpy()

    call(torch.cuda.current_stream().cuda_stream)
    first = results()
    check_against_oracle(*first, *oracle.attention_fwd(q, k, v, scale, True, dtype), dtype, f"pieces replayed {(B, H, Nk, D)}")
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for _ in range(3):
            call(side.cuda_stream)
    for _ in range(3):
        graph.replay()
        assert all(np.array_equal(a, b) for a, b in zip(first, results()))
        call(torch.cuda.current_stream().cuda_stream)
        assert all(np.array_equal(a, b) for a, b in zip(first, results()))
