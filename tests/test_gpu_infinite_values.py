"""An infinite element of V makes its outputs infinite wherever its probability is positive, and leaves the others alone:
also where the probabilities of few units are multiplied in three parts of 8 bits, none of which may become zero."""
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


# Units of 8 tokens and the new ones, the first of which has the score 0, the eighth `below` less, the others 200 less (in powers of two)
@pytest.mark.parametrize("dtype,least", [("bf16", 126), ("fp32", 148)])  # exponent of the smallest probability that is not taken as 0
@pytest.mark.parametrize("Hq,Hkv,D,nq", [(1, 1, 64, 3), (4, 1, 128, 4), (4, 1, 128, 6), (2, 1, 64, 16), (8, 1, 128, 8), (5, 1, 64, 8),
                                         (264, 33, 128, 8), (85, 17, 64, 8), (81, 81, 128, 4)])  # up to 64 rows, and each kernel
@pytest.mark.parametrize("below", [20, 90, 97, 98, 110, 126, 140])
def test_infinite_values_of_small_probability(Hq, Hkv, D, nq, dtype, least, below):
    from paper_2404_15778_amd import harness as hip
    w = wl.make_attention("tiny", 1, Hq, Hkv, D, dtype, np.array([8], np.int32), np.array([nq], np.int32), seed=1, Lcap=800)
    w.scale = float(np.log(2.0))
    Q, K, V = np.zeros(w.Q.shape, np.float32), np.zeros(w.K.shape, np.float32), np.ones(w.V.shape, np.float32)
    Q[..., 0], K[:, 1:, :, 0], K[:, 7, :, 0] = 1.0, -200.0, -float(below)
    V[:, 7, :, 3], V[:, 7, :, 5] = np.inf, -np.inf
    to = wl.to_bf16_bits if dtype == "bf16" else np.float32
    w.Q, w.K, w.V = to(Q), to(K), to(V)
    O, lse, status, _ = hip.run_attention_workload(w, fused=True)
    assert status == 0 and np.isfinite(lse).all()
    if below <= least:
        assert (O[..., 3] == np.inf).all() and (O[..., 5] == -np.inf).all()
    O[..., 3] = O[..., 5] = 1.0
    assert np.abs(O - 1.0).max() <= 1e-6
