"""fa_fwd_masked on waves of 64 rows (windows and key counts without a prefix, D = 128), forced on small problems: limits on either side
of a unit of 32 keys, of a tile and of the pipelined loop's first and last tiles, walks that start past tile 0, ragged ends,
empty rows, and the diagonal on each batch entry's own last key; against the oracle element by element."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import inputs as I
import options
from gpu_util import check_against_oracle, run_fa_fwd_masked

pytestmark = pytest.mark.gpu
D = 128


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("Nq,Nk,left,right,kv_len,anchor", [
    (640, 640, 127, 0, None, 0), (640, 640, 128, 0, None, 0), (640, 640, 129, 31, None, 0), (640, 640, 63, 32, None, 0),
    (640, 640, 0, 0, None, 0), (640, 640, -1, 0, None, 0), (640, 640, -1, -1, None, 0), (640, 640, 300, -1, None, 0),
    (700, 700, 200, 0, None, 0), (700, 777, 333, 40, None, 0), (300, 1408, 500, 0, None, 0), (900, 300, 100, 0, None, 0),
    (512, 1024, -1, -1, (1024, 479), 0), (512, 1024, -1, 0, (993, 960), 0), (512, 1024, 160, 0, (544, 1023), 0),
    (512, 1024, 160, 0, (544, 700), 1), (320, 1024, -1, 0, (0, 321), 1), (256, 832, 95, 33, (1, 832), 0)])
def test_elementwise(oracle, Nq, Nk, left, right, kv_len, anchor, dtype):
    print(f"case masked rows64 {(Nq, Nk, left, right, kv_len, anchor)} dtype={dtype}", flush=True)
    options.set_fwd_mode("wide64")
    rng = np.random.default_rng(Nq + 3 * Nk + left + dtype)
    q, k, v = (I.f32_to_bits(rng.standard_normal((2, 2, n, D), dtype=np.float32), dtype) for n in (Nq, Nk, Nk))
    scale = 1.0 / math.sqrt(D)
    o_ref, lse_ref = oracle.attention_fwd_masked(q, k, v, scale, dtype, left, right, 0, kv_len, diag_from_kv_len=anchor)
    o, lse = run_fa_fwd_masked(q, k, v, scale, dtype, left, right, 0, kv_len, diag_from_kv_len=anchor)
    check_against_oracle(o, lse, o_ref, lse_ref, dtype, f"rows64 {(Nq, Nk, left, right, kv_len, anchor)}")
    assert (I.bits_to_f64(o, dtype)[np.isneginf(lse_ref)] == 0).all()
