"""Rows of extreme but finite size.  Scores far beyond what a softmax resolves: all of a query's weight is on its largest score, which has
the probability 1.  Keys and queries whose sizes cancel: ordinary scores, whatever the order in which their scales are multiplied."""
import math

import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("Hq,Hkv,D,kmax", [(4, 2, 64, 4), (4, 4, 128, 16), (8, 2, 128, 6), (4, 1, 64, 8), (8, 1, 128, 8), (8, 1, 64, 5),
                                           (136, 17, 128, 8), (63, 9, 64, 5), (100, 100, 64, 2)])
@pytest.mark.parametrize("size", [32.0, 2.0 ** 15, 2.0 ** 24])  # of K and Q: scores of 2^12, 2^32 and 2^50
def test_one_token_takes_all(dtype, Hq, Hkv, D, kmax, size):
    from paper_2404_15778_amd import harness
    from oracle.kv_int8 import dequantize_rows, quantize_rows
    w = wl.make_attention("far", 2, Hq, Hkv, D, "bf16", [900, 40], [kmax, kmax], 3, kmax=kmax, Lcap=960)
    w.scale = 1.0 / math.sqrt(D)
    Q, K, V = (wl.bf16_bits_to_f32(x) for x in (w.Q, w.K, w.V))
    Q *= size / np.sqrt((Q ** 2).mean())
    K *= size
    w.Q, w.K = wl.to_bf16_bits(Q), wl.to_bf16_bits(K)
    Q, K = wl.bf16_bits_to_f32(w.Q), wl.bf16_bits_to_f32(w.K)
    if dtype == "int8kv":
        Q, K, V = (dequantize_rows(*quantize_rows(x)) for x in (Q, K, V))
        w.dtype = dtype
    want, want_lse = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    O, lse, status, _ = harness.run_attention_workload(w, fused=True)
    assert status == 0
    # a score is rounded to 24 bits a few times on its way (and in lse)
    assert np.abs(lse - want_lse).max() <= 2e-6 * np.abs(want_lse).max()
    # The probability 1 and, over bf16 caches, V are represented as they are; an INT8 row's V scale is rounded to bf16 (2^-9).
    # Two scores nearer to each other than their rounding, 2^-21 of them, may change places or share a row.
    g = Hq // Hkv
    for b in range(2):
        for i in range(kmax):
            for h in range(Hq):
                s = np.sort(K[b, :w.ctx_len[b] + i + 1, h // g].astype(np.float64) @ Q[b, i, h].astype(np.float64))[::-1][:2] * w.scale
                if s[0] - s[1] > 40 + 2.0 ** -20 * abs(s[0]):
                    err = np.abs(O[b, i, h] - want[b, i, h]).max()
                    assert err <= (2.0 ** -8 if dtype == "int8kv" else 1e-6) * np.abs(want[b, i, h]).max(), (b, i, h)
    assert np.isfinite(O).all()


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("Hq,Hkv,D,kmax", [(4, 2, 64, 4), (4, 4, 128, 16), (8, 2, 128, 6), (4, 1, 64, 8), (8, 1, 128, 8), (8, 1, 64, 5),
                                           (136, 17, 128, 8), (63, 9, 64, 5), (100, 100, 64, 2)])
@pytest.mark.parametrize("power", [120, 110, -110])
def test_keys_and_queries_of_opposite_size(dtype, Hq, Hkv, D, kmax, power):
    from paper_2404_15778_amd import harness
    from oracle.kv_int8 import dequantize_rows, quantize_rows
    w = wl.make_attention("opposite", 2, Hq, Hkv, D, "bf16", [900, 40], [kmax, kmax], 4, kmax=kmax, Lcap=960)
    w.K = wl.to_bf16_bits(np.ldexp(wl.bf16_bits_to_f32(w.K), power))
    w.Q = wl.to_bf16_bits(np.ldexp(wl.bf16_bits_to_f32(w.Q), -power))
    Q, K, V = (wl.bf16_bits_to_f32(x) for x in (w.Q, w.K, w.V))
    if dtype == "int8kv":
        Q, K, V = (dequantize_rows(*quantize_rows(x)) for x in (Q, K, V))
        w.dtype = dtype
    want, want_lse = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    O, lse, status, _ = harness.run_attention_workload(w, fused=True)
    # probabilities are rounded to bf16 (2^-9) for outputs of magnitude up to about 4; lse stays in 32 bits
    assert status == 0 and np.abs(O - want).max() <= 2e-2 and np.abs(lse - want_lse).max() <= 1e-4
