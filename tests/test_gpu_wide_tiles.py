"""More than 16 query rows per kv head, at the edges of the dispatch: 17, 32, 33 and 64 rows, caches of 24 and 25 blocks (the
kernels that share a block's rows, and those that share the blocks), any sign of the softmax scale."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu
# probabilities and V are rounded to bf16 (2^-9 each) for outputs of magnitude up to about 4
TOL = 2e-2
# scores, exponentials and their sum stay in 32 bits: a few roundings of values up to about 20
LSE_TOL = 1e-4


@pytest.mark.parametrize("blocks", [24, 25])
@pytest.mark.parametrize("D,Hq,Hkv,kmax", [(128, 17, 1, 1), (128, 8, 2, 8), (128, 33, 1, 1), (128, 16, 2, 8), (64, 6, 2, 6), (64, 2, 2, 32),
                                           (64, 7, 1, 7), (64, 3, 3, 64)])
@pytest.mark.parametrize("fused", [False, True])
def test_rows_and_cache_sizes(D, Hq, Hkv, kmax, blocks, fused):
    from paper_2404_15778_amd import harness
    ctx = [32 * blocks - kmax, 0, 31, 32, 200, 5]  # the first unit ends with the cache; one block, part of one, several
    nq = [kmax, kmax, 1, max(1, kmax - 1), kmax, 0]
    w = wl.make_attention("wide", 6, Hq, Hkv, D, "bf16", ctx, nq, 41, kmax=kmax, Lcap=32 * blocks)
    Or, lser = oracle.verify_attention(w.Q, w.K, w.V, w.ctx_len, w.draft_len, w.scale)
    O, lse, status, _ = harness.run_attention_workload(w, poison=True, fused=fused)
    assert status == 0 and np.isfinite(O).all()
    assert np.abs(O - Or).max() <= TOL and np.abs(lse - lser).max() <= LSE_TOL


@pytest.mark.parametrize("Hq,kmax", [(4, 6), (4, 16)])  # 24 and 64 rows
def test_zero_scale_is_the_mean_of_the_visible_values(Hq, kmax):
    from paper_2404_15778_amd import harness
    w = wl.make_attention("flat", 3, Hq, 1, 128, "bf16", [900, 40, 0], [kmax, 3, kmax], 5, kmax=kmax, Lcap=900 + kmax)
    w.scale = 0.0
    Or, lser = oracle.verify_attention(w.Q, w.K, w.V, w.ctx_len, w.draft_len, 0.0)
    O, lse, status, _ = harness.run_attention_workload(w, poison=True)
    assert status == 0
    assert np.abs(O - Or).max() <= TOL and np.abs(lse - lser).max() <= 1e-4


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("D,Hq,kmax", [(128, 4, 6), (128, 4, 16), (64, 4, 6), (64, 4, 16)])
def test_negative_scale_is_negative_queries(dtype, D, Hq, kmax):
    import torch
    import paper_2404_15778_amd as bass
    dev, ctx, nq = "cuda:0", [900, 65, 3], [kmax, kmax, 2]
    gen = torch.Generator(device=dev)
    gen.manual_seed(D + kmax)
    rows = lambda n, H: torch.randn((3, n, H, D), generator=gen, device=dev).to(torch.bfloat16)  # noqa: E731
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)  # noqa: E731
    d = bass.make_desc(3, kmax, Hq, 1, D, 900 + kmax, dtype, 0.1)
    caches = [torch.zeros(bass.bass_kv_cache_bytes(d), dtype=torch.uint8, device=dev) for _ in range(2)]
    bass.bass_kv_append(d.replace(kmax=900), *caches, rows(900, 1), rows(900, 1), i32([0] * 3), i32(ctx))
    bass.bass_kv_append(d, *caches, rows(kmax, 1), rows(kmax, 1), i32(ctx), i32(nq))
    Q, ws, out = rows(kmax, Hq), bass.alloc_workspace(d, dev), []
    for desc, q in ((d, -Q), (d.replace(scale=-0.1), Q)):
        O, lse = torch.zeros((3, kmax, Hq, D), device=dev), torch.zeros((3, kmax, Hq), device=dev)
        bass.bass_verify_attention(desc, q, *caches, i32(ctx), i32(nq), O, lse, ws)
        out.append((O, lse))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][0].isfinite().all() and out[0][0].abs().sum() > 0


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("D,g,kmax", [(128, 1, 16), (128, 4, 3), (64, 2, 8), (64, 1, 1)])
@pytest.mark.parametrize("Hkv", [80, 81])  # one workgroup per stretch of the list, one wavefront
def test_units_at_the_edge_of_one_tile(dtype, D, g, kmax, Hkv):
    from paper_2404_15778_amd import harness
    from oracle.kv_int8 import dequantize_rows, quantize_rows
    w = wl.make_attention("narrow", 1, g * Hkv, Hkv, D, "bf16", [333], [kmax], 7, kmax=kmax, Lcap=333 + kmax)
    Q, K, V = w.Q, w.K, w.V
    if dtype == "int8kv":
        Q, K, V = (dequantize_rows(*quantize_rows(wl.bf16_bits_to_f32(x))) for x in (Q, K, V))
        w.dtype = dtype
    Or, lser = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    for fused in (False, True):
        O, lse, status, _ = harness.run_attention_workload(w, poison=True, fused=fused)
        assert status == 0 and np.abs(O - Or).max() <= TOL and np.abs(lse - lser).max() <= LSE_TOL


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("D,g,kmax,B,Hkv", [(64, 4, 8, 3, 85), (64, 3, 8, 4, 64), (64, 2, 10, 32, 32), (64, 2, 10, 25, 41),  # 255, 256, 1024, 1025 units
                                            (128, 6, 6, 4, 16), (128, 8, 8, 5, 13)])  # 64 and 65: a row merged in four parts or in one
def test_units_at_the_edge_of_several_tiles(dtype, D, g, kmax, B, Hkv):
    from paper_2404_15778_amd import harness
    from oracle.kv_int8 import dequantize_rows, quantize_rows
    ctx = [(333, 820, 0, 31)[b % 4] if B < 9 else (70, 33, 0, 129, 12)[b % 5] for b in range(B)]
    w = wl.make_attention("units", B, g * Hkv, Hkv, D, "bf16", ctx, [kmax - b % 3 for b in range(B)], 11, kmax=kmax, Lcap=820 + kmax)
    Q, K, V = w.Q, w.K, w.V
    if dtype == "int8kv":
        Q, K, V = (dequantize_rows(*quantize_rows(wl.bf16_bits_to_f32(x))) for x in (Q, K, V))
        w.dtype = dtype
    Or, lser = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    for fused in (False, True):
        O, lse, status, _ = harness.run_attention_workload(w, poison=True, fused=fused)
        assert status == 0 and np.abs(O - Or).max() <= TOL and np.abs(lse - lser).max() <= LSE_TOL
