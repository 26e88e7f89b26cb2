"""A wave whose last tile holds keys for it in its first half only leaves the other half out (D = 64, four-wave workgroups and eight
waves on 256 rows): lengths on both sides of every 32 keys, the diagonal at either half.  Leaving masked keys out changes no bit
of bf16 results against the kernel for descriptor masks, which computes whole tiles (fp16 carries other row sums there)."""
import math

import numpy as np
import pytest

from paper_2410_16663_amd import binding as fa
from paper_2410_16663_amd import inputs as I
import options
from gpu_util import check_against_oracle, run_fa_fwd, run_fa_fwd_masked

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("Nq,Nk", [(40, 1), (64, 32), (33, 33), (130, 63), (197, 197), (161, 224), (96, 257), (290, 97), (300, 352)])
def test_last_tiles(oracle, Nq, Nk, dtype):
    D = 64
    print(f"case half tiles Nq={Nq} Nk={Nk} D={D} dtype={dtype}", flush=True)
    B, H, scale = 1, 3, 1.0 / math.sqrt(D)
    rng = np.random.default_rng(1000 * Nq + Nk + D)
    # (v stays N(0, 1): the tolerance is stated for it.  Of 2 N(0, 1) half a unit of bf16 in [2, 4), 7.8e-3, and the rounding of a
    # dominant probability, 2^-9 |v - o|, pass 1e-2 together.)
    q, k, v = (I.f32_to_bits(rng.standard_normal((B, H, n, D), dtype=np.float32), dtype) for n in (Nq, Nk, Nk))
    options.set_fwd_mode("wide4")
    for causal in (False, True):
        o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, causal, dtype)
        o, lse = run_fa_fwd(q, k, v, scale, causal, dtype)
        check_against_oracle(o, lse, o_ref, lse_ref, dtype, f"half tiles {(Nq, Nk, D)} causal={causal} dt={dtype}")
        if dtype == I.BF16:
            om, lm = run_fa_fwd_masked(q, k, v, scale, dtype, -1, 0 if causal else -1)
            assert np.array_equal(o, om) and np.array_equal(lse, lm)
    options.set_fwd_mode("wide")
    for causal in (False, True):
        o_ref, lse_ref = oracle.attention_fwd(q, k, v, scale, causal, dtype)
        o, lse = run_fa_fwd(q, k, v, scale, causal, dtype)
        check_against_oracle(o, lse, o_ref, lse_ref, dtype, f"half tiles wide {(Nq, Nk, D)} causal={causal} dt={dtype}")
