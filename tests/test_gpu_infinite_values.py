"""An infinite element of V makes its outputs infinite wherever its probability is positive, and leaves the others alone:
also where short block lists are divided over fewer shares and remainders of the probabilities are multiplied."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu
INF, MINUS_INF = 0x7F80, 0xFF80  # bf16


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,D,ctx,nq", [(1, 4, 4, 128, 200, 3), (1, 8, 2, 64, 700, 2), (2, 16, 16, 128, 1000, 1),
                                               (8, 32, 32, 64, 100, 2)])  # the last one over all shares
def test_infinite_values_of_the_context(B, Hq, Hkv, D, ctx, nq, fused):
    from paper_2404_15778_amd import harness as hip
    w = wl.make_attention("inf", B, Hq, Hkv, D, "bf16", np.full(B, ctx, np.int32), np.full(B, nq, np.int32), seed=ctx)
    K, Q, V = (wl.bf16_bits_to_f32(x) for x in (w.K, w.Q, w.V))
    # tokens of blocks that every query sees in whole: the first, one in the middle, two signs in one unit
    marks = [(5, 0, 7, INF), (40, Hkv - 1, 3, MINUS_INF), (70, 0, D - 1, MINUS_INF), (95, 1, 0, INF)]
    for tok, head, d, bits in marks:
        w.V[B - 1, tok, head, d] = bits
        V[B - 1, tok, head, d] = 0.0
    want, _ = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    O, lse, status, _ = hip.run_attention_workload(w, fused=fused)
    assert status == 0 and np.isfinite(lse).all()
    g = Hq // Hkv
    for tok, head, d, bits in marks:
        rows = (B - 1, slice(None), slice(head * g, (head + 1) * g), d)
        assert (O[rows] == (np.inf if bits == INF else -np.inf)).all(), (tok, head, d)
        O[rows] = want[rows] = 0.0
    assert np.isfinite(O).all() and np.abs(O - want).max() <= 2e-2
