"""fa_attn_linear in blocks of rows gives the o, lse and y of fa_attn_linear_block over the same blocks bit for bit, whatever
FA_OPT_LINEAR_OVERLAP says: on one stream, on two, and on two under capture."""
import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
import options
from gpu_util import run_attn_linear

pytestmark = pytest.mark.gpu


def split_rows(Nq, rows):
    blocks, r = [], 0
    while r < Nq:
        n = min(max(rows // 2, 1) if r == 0 else rows, Nq - r)
        blocks.append((r, n))
        r += n
    return blocks


def make(Nq, D, dtype, B=2, H=2, N=512):
    rng = np.random.default_rng(Nq + D + dtype)
    bits = lambda shape, m=1.0: I.f32_to_bits(rng.standard_normal(shape, dtype=np.float32) * np.float32(m), dtype)
    return bits((B, H, Nq, D)), bits((B, H, Nq, D)), bits((B, H, Nq, D)), bits((H * D, N), (H * D) ** -0.5)


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Nq,rows", [(1100, 256), (700, 699), (333, 1), (2600, 1024)])
def test_blocks_whatever_the_option(Nq, rows, D, dtype):
    print(f"case attn_linear blocks Nq={Nq} rows={rows} D={D} dtype={dtype}", flush=True)
    q, k, v, w = make(Nq, D, dtype)
    one_by_one = run_attn_linear(q, k, v, w, 0.1, True, dtype, blocks=split_rows(Nq, rows))
    for on in (None, True, False):
        options.set_linear_overlap(on)
        got = run_attn_linear(q, k, v, w, 0.1, True, dtype, rows_per_block=rows)
        assert all(np.array_equal(a, b) for a, b in zip(one_by_one, got)), on


@pytest.mark.parametrize("overlap", [None, True, False])
def test_blocks_under_capture(overlap):
    import torch
    print(f"case attn_linear blocks captured overlap={overlap}", flush=True)
    B, H, Nq, D, N, dtype, rows = 2, 2, 1100, 128, 512, I.BF16, 256
    q, k, v, w = make(Nq, D, dtype)
    one_by_one = run_attn_linear(q, k, v, w, 0.1, True, dtype, blocks=split_rows(Nq, rows))
    options.set_linear_overlap(overlap)
    dev = torch.device("cuda:0")
    tq, tk, tv, tw = (torch.from_numpy(a.view(np.int16)).to(dev) for a in (q, k, v, w))
    to = torch.zeros((B, H, Nq, D), dtype=torch.int16, device=dev)
    tl = torch.zeros((B, H, Nq), dtype=torch.float32, device=dev)
    ty = torch.zeros((B, Nq, N), dtype=torch.float32, device=dev)

    def call(stream):
        fa.fa_attn_linear(tq, tk, tv, tw, to, tl, ty, B, H, Nq, Nq, D, N, 0.1, 1, dtype, rows, stream)

    call(torch.cuda.current_stream().cuda_stream)                  # (the second stream comes into being outside of a capture)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(side.cuda_stream)
    for _ in range(3):
        for t in (to, tl, ty):
            t.zero_()
        graph.replay()
        copy = ty.clone()                                          # behind the replay: sees the finished y
        torch.cuda.synchronize()
        got = to.cpu().numpy().view(np.uint16), tl.cpu().numpy(), copy.cpu().numpy()
        assert all(np.array_equal(a, b) for a, b in zip(one_by_one, got))
