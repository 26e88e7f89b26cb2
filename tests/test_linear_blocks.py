"""fa_attn_linear computes all rows at once; with FA_OPT_LINEAR_OVERLAP = 1 block after block, the projections on a second
stream: then o, lse and y are those of fa_attn_linear_block over the same blocks."""
import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
import options
from gpu_util import run_attn_linear, run_fa_fwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Nq,rows", [(1100, 256), (700, 699), (333, 1)])
def test_blocks_on_two_streams_and_all_rows_at_once(Nq, rows, D):
    import torch
    print(f"case attn_linear blocks Nq={Nq} rows={rows} D={D}", flush=True)
    rng = np.random.default_rng(Nq + D)
    B, H, N = 2, 2, 512
    bits = lambda shape, m=1.0: I.f32_to_bits(rng.standard_normal(shape, dtype=np.float32) * np.float32(m), I.BF16)
    q, k, v, w = bits((B, H, Nq, D)), bits((B, H, Nq, D)), bits((B, H, Nq, D)), bits((H * D, N), (H * D) ** -0.5)
    blocks, r = [], 0
    while r < Nq:
        n = min(max(rows // 2, 1) if r == 0 else rows, Nq - r)
        blocks.append((r, n))
        r += n
    one_by_one = run_attn_linear(q, k, v, w, 0.1, True, I.BF16, blocks=blocks)
    options.set_linear_overlap(True)
    for _ in range(3):
        got = run_attn_linear(q, k, v, w, 0.1, True, I.BF16, rows_per_block=rows)
        assert all(np.array_equal(a, b) for a, b in zip(one_by_one, got))
    for on in (False, None):
        options.set_linear_overlap(on)
        o, lse, y = run_attn_linear(q, k, v, w, 0.1, True, I.BF16, rows_per_block=rows)
        whole = run_attn_linear(q, k, v, w, 0.1, True, I.BF16, rows_per_block=0)
        assert all(np.array_equal(a, b) for a, b in zip((o, lse, y), whole))
        o_fwd, lse_fwd = run_fa_fwd(q, k, v, 0.1, True, I.BF16)
        assert np.array_equal(o, o_fwd) and np.array_equal(lse, lse_fwd)
    # work enqueued on the caller's stream right behind the call sees the finished y and does not overtake it
    options.set_linear_overlap(True)
    dev = torch.device("cuda:0")
    tq, tk, tv, tw = (torch.from_numpy(a.view(np.int16)).to(dev) for a in (q, k, v, w))
    to = torch.zeros((B, H, Nq, D), dtype=torch.int16, device=dev)
    tl = torch.zeros((B, H, Nq), dtype=torch.float32, device=dev)
    ty = torch.empty((B, Nq, N), dtype=torch.float32, device=dev)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fa.fa_attn_linear(tq, tk, tv, tw, to, tl, ty, B, H, Nq, Nq, D, N, 0.1, 1, I.BF16, rows, side.cuda_stream)
        copy = ty.clone()
        ty.zero_()
    side.synchronize()
    assert np.array_equal(copy.cpu().numpy(), one_by_one[2])


@pytest.mark.parametrize("B,H,N,D", [(1, 16, 1334, 128), (1, 8, 2048, 128), (1, 10, 2500, 64), (2, 24, 1024, 64)])
def test_fp16_lse_of_blocks_given_at_once(oracle, B, H, N, D):
    """Small blocks carry both row sums in fp16 (lse from the unrounded exponentials), and so does the one launch that stands for
    them, whatever form it takes: logits of standard deviation 4, fp32 rounding of logits up to 32, 1e-5."""
    print(f"case attn_linear lse {(B, H, N, D)}", flush=True)
    rng = np.random.default_rng(N + D)
    q, k, v = (I.f32_to_bits(2 * rng.standard_normal((B, H, N, D), dtype=np.float32), I.F16) for _ in range(3))
    w = I.f32_to_bits(rng.standard_normal((H * D, 256), dtype=np.float32) * np.float32((H * D) ** -0.5), I.F16)
    _, lse, _ = run_attn_linear(q, k, v, w, D ** -0.5, True, I.F16, rows_per_block=256)
    rows = np.unique(np.concatenate([rng.integers(0, B * H * N, 2000), [0, N - 1, B * H * N - 1]]))
    _, lse_ref = oracle.attention_fwd(q, k, v, D ** -0.5, True, I.F16, rows=rows)
    assert np.abs(lse.reshape(-1)[rows] - lse_ref).max() <= 1e-5
