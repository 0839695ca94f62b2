"""Short block lists are divided over fewer shares.  That must not cost precision: what the rounding of the probabilities
to bf16 leaves over is multiplied as well there."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,D,ctx,nq", [(1, 32, 32, 128, 1270, 8), (1, 8, 2, 64, 33, 3), (2, 4, 4, 128, 700, 1),
                                               (3, 8, 8, 64, 31, 2)])
def test_error_against_64_bits(B, Hq, Hkv, D, ctx, nq):
    from paper_2404_15778_amd import harness as hip
    w = wl.make_attention("short", B, Hq, Hkv, D, "bf16", np.full(B, ctx, np.int32), np.full(B, nq, np.int32), seed=ctx)
    K, V, Q = (wl.bf16_bits_to_f32(x) for x in (w.K, w.V, w.Q))
    want, _ = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    O, _, status, _ = hip.run_attention_workload(w, fused=True)
    assert status == 0
    # a probability and its remainder have 8 bits each: 2^-18 of it is lost; fp32 scores and exponentials: about 1e-6
    assert np.linalg.norm(O - want) <= 2e-5 * np.linalg.norm(want)
