"""Few units are divided over few shares.  That must not cost precision: the 24 bits of a probability are multiplied in three parts."""
import numpy as np
import pytest

import oracle
import workloads as wl
from oracle.kv_int8 import dequantize_rows, quantize_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("B,Hq,Hkv,D,ctx,nq", [(1, 32, 32, 128, 1270, 8), (1, 8, 2, 64, 33, 3), (2, 4, 4, 128, 700, 1),
                                               (3, 8, 8, 64, 31, 2)])
def test_error_against_64_bits(dtype, B, Hq, Hkv, D, ctx, nq):
    from paper_2404_15778_amd import harness as hip
    w = wl.make_attention("short", B, Hq, Hkv, D, "bf16", np.full(B, ctx, np.int32), np.full(B, nq, np.int32), seed=ctx)
    K, V, Q = (wl.bf16_bits_to_f32(x) for x in (w.K, w.V, w.Q))
    if dtype == "int8kv":
        K, V, Q = (dequantize_rows(*quantize_rows(x)) for x in (K, V, Q))
        w.dtype = dtype
    want, _ = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    O, _, status, _ = hip.run_attention_workload(w, fused=True)
    assert status == 0
    # Scores of a few units in log2 and their exponentials are rounded to 24 bits a few times each, the parts of a probability to nothing
    # (without the third, 2^-17 of each would be lost: 3.6e-6)
    assert np.linalg.norm(O - want) <= 1e-6 * np.linalg.norm(want)
