"""fa_fwd_splitkv launches what fa_fwd_splitkv_plan says: the kernel nodes of a captured call, their number and grids."""
import ctypes
import os

import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
import options


def test_second_kernel_of_the_plan():
    """None where a single query's runs, up to D/4, are merged by the kernel that computes them; one for more, for more queries and
    through the tile kernel."""
    for D in (64, 128):
        for runs in (1, 2, D // 4, D // 4 + 1, 40):
            for B, H in ((1, 1), (2, 24), (1, 70000)):
                p = fa.fa_fwd_splitkv_plan(B, H, 1, 64 * 100, D, 1, I.BF16, runs)
                blocks = -(-B * H // (1024 // D))
                assert (p.nsplit, p.grid_x, p.grid_y) == (runs, B * H, runs)
                assert p.combine_grid == (blocks if runs > D // 4 else 0)
                assert fa.fa_fwd_splitkv_plan(B, H, 2, 64 * 100, D, 1, I.BF16, runs).combine_grid == (0 if runs == 1 else -(-2 * B * H // (1024 // D)))
    assert fa.fa_fwd_splitkv_plan(1, 48, 1, 32768, 128, 1, I.BF16).combine_grid == 0          # pieces, six runs at most
    assert fa.fa_fwd_splitkv_plan(1, 3, 1, 2000000, 128, 1, I.BF16).combine_grid == 1         # pieces, 86 runs
    options.set_decode("mfma")
    assert fa.fa_fwd_splitkv_plan(1, 16, 1, 6400, 128, 1, I.BF16, 4).combine_grid == 2


class KernelNode(ctypes.Structure):
    """hipKernelNodeParams"""
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint)]


def kernel_grids(graph):
    import torch
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    g = ctypes.c_void_p(graph.raw_cuda_graph())
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(g, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(g, nodes, ctypes.byref(n)) == 0
    grids = []
    for node in nodes:
        p = KernelNode()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        grids.append(tuple(p.grid)[:2])
    return grids


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,Nq,Nk,D,nsplit", [
    (1, 32, 1, 1000, 128, 0), (1, 12, 1, 3000, 64, 0), (1, 3, 1, 3000, 64, 17), (2, 4, 1, 6400, 128, 33), (1, 48, 1, 32768, 128, 0),
    (1, 5, 1, 1200000, 64, 0), (8, 32, 1, 500, 128, 0), (1, 8, 4, 9000, 128, 0)])
def test_launches(B, H, Nq, Nk, D, nsplit):
    import torch
    print(f"case launches {(B, H, Nq, Nk, D, nsplit)}", flush=True)
    dev = torch.device("cuda:0")
    q, k, v = (torch.zeros((B, H, n, D), dtype=torch.bfloat16, device=dev) for n in (Nq, Nk, Nk))
    o, lse = torch.empty_like(q), torch.empty((B, H, Nq), device=dev)
    plan = fa.fa_fwd_splitkv_plan(B, H, Nq, Nk, D, 1, I.BF16, nsplit)
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device=dev)

    def call(stream):
        fa.fa_fwd_splitkv(q, k, v, o, lse, B, H, Nq, Nk, D, 0.1, 1, I.BF16, nsplit, ws, plan.workspace_bytes, stream)

    call(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=side):
        call(side.cuda_stream)
    want = [(plan.grid_x, plan.grid_y)] + ([(plan.combine_grid, 1)] if plan.combine_grid else [])
    assert kernel_grids(graph) == want
