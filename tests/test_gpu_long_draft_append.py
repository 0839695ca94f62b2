"""Drafts too long to be staged, more than one query tile: a planned launch appends them block by block.  The caches and
outputs are those of an append by a launch of its own (bass_append_verify_attention at these sizes)."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("D,kmax,Hq,Hkv", [(128, 17, 4, 2), (128, 20, 6, 2), (128, 32, 3, 3), (128, 64, 2, 2), (64, 33, 2, 2),
                                           (64, 64, 1, 1)])
def test_planned_append_of_long_drafts(dtype, D, kmax, Hq, Hkv):
    import torch
    import paper_2404_15778_amd as bass
    dev = "cuda:0"
    ctx, nq = [0, 31, 32, 5, 100, 7, 63], [kmax, kmax, 1, kmax - 1, kmax, 0, 2]
    B, Lcap = len(ctx), 100 + kmax
    gen = torch.Generator(device=dev)
    gen.manual_seed(D + kmax)
    rows = lambda H: torch.randn((B, kmax, H, D), generator=gen, device=dev).to(torch.bfloat16)  # noqa: E731
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)  # noqa: E731
    d = bass.make_desc(B, kmax, Hq, Hkv, D, Lcap, dtype, 1.0 / math.sqrt(D))
    caches = [torch.zeros(bass.bass_kv_cache_bytes(d), dtype=torch.uint8, device=dev) for _ in range(2)]
    for i in range(0, 100, kmax):
        bass.bass_kv_append(d, *caches, rows(Hkv), rows(Hkv), i32([i] * B), i32([min(kmax, max(0, c - i)) for c in ctx]))
    Q, K, V, status = rows(Hq), rows(Hkv), rows(Hkv), torch.zeros(1, dtype=torch.int32, device=dev)
    ws, plan = bass.alloc_workspace(d, dev), bass.alloc_plan(d, dev)

    def run(planned):
        c = [t.clone() for t in caches]
        O = torch.full((B, kmax, Hq, D), 7.0, device=dev)
        lse = torch.full((B, kmax, Hq), 7.0, device=dev)
        if planned:
            bass.bass_attention_plan(d, i32(ctx), i32(nq), bass.PLAN_APPEND, 0, plan, status)
            bass.bass_verify_attention_planned(d, Q, K, V, *c, plan, O, lse, ws, status)
        else:
            bass.bass_append_verify_attention(d, Q, K, V, *c, i32(ctx), i32(nq), O, lse, ws, status)
        return [*c, O, lse]

    got, want = run(True), run(False)
    assert status.item() == 0
    for a, b in zip(got, want):
        assert torch.equal(a, b)


# Stretches of several blocks: 32 workgroups share 65 - 170 blocks, so a stretch has 2 - 6 of them, even and odd counts, new
# tokens in either or both blocks of a phase and in later phases, and units that begin and end inside a stretch.
@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("ctx", [[900, 333, 640, 64, 5], [31, 400, 1000, 959, 0]])
@pytest.mark.parametrize("D,kmax,Hq,Hkv", [(128, 20, 2, 2), (128, 32, 1, 1), (128, 64, 2, 2), (128, 24, 4, 2), (64, 32, 2, 2), (64, 60, 2, 2),
                                           (64, 9, 208, 104), (128, 32, 60, 60)])  # the last two: more than 256 units
def test_stretches_of_several_blocks(dtype, ctx, D, kmax, Hq, Hkv):
    import numpy as np
    import torch
    import oracle
    import paper_2404_15778_amd as bass
    from oracle.kv_int8 import dequantize_rows, quantize_rows
    dev, B = "cuda:0", len(ctx)
    nq = [kmax, kmax - 3, 1, kmax, kmax]
    Lcap = max(ctx) + kmax
    gen = torch.Generator(device=dev)
    gen.manual_seed(D + kmax + ctx[0])
    rand = lambda n, H: torch.randn((B, n, H, D), generator=gen, device=dev).to(torch.bfloat16)  # noqa: E731
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)  # noqa: E731
    d = bass.make_desc(B, kmax, Hq, Hkv, D, Lcap, dtype, 1.0 / math.sqrt(D))
    old, new, Q = [rand(max(ctx), Hkv) for _ in range(2)], [rand(kmax, Hkv) for _ in range(2)], rand(kmax, Hq)
    caches = [torch.full((bass.bass_kv_cache_bytes(d),), 0x7F, dtype=torch.uint8, device=dev) for _ in range(2)]
    bass.bass_kv_append(d.replace(kmax=max(ctx)), *caches, *old, i32([0] * B), i32(ctx))
    by_append = [t.clone() for t in caches]
    bass.bass_kv_append(d, *by_append, *new, i32(ctx), i32(nq))
    rows = []  # keys and values as the oracle takes them
    for o, n in zip(old, new):
        r = np.zeros((B, Lcap, Hkv, D), np.float32)
        for b in range(B):
            r[b, :ctx[b]], r[b, ctx[b]:ctx[b] + nq[b]] = o[b, :ctx[b]].float().cpu().numpy(), n[b, :nq[b]].float().cpu().numpy()
        rows.append(r)
    q = Q.float().cpu().numpy()
    if dtype == "int8kv":
        q, *rows = [dequantize_rows(*quantize_rows(x)) for x in (q, *rows)]
    want, want_lse = oracle.verify_attention(q, *rows, np.array(ctx, np.int32), np.array(nq, np.int32), d.scale)
    O, lse = torch.full((B, kmax, Hq, D), 7.0, device=dev), torch.full((B, kmax, Hq), 7.0, device=dev)
    status, plan, ws = torch.zeros(1, dtype=torch.int32, device=dev), bass.alloc_plan(d, dev), bass.alloc_workspace(d, dev)
    bass.bass_set_attention_waves(64)
    try:
        bass.bass_attention_plan(d, i32(ctx), i32(nq), bass.PLAN_APPEND, 0, plan, status)
        bass.bass_verify_attention_planned(d, Q, *new, *caches, plan, O, lse, ws, status)
    finally:
        bass.bass_set_attention_waves(0)
    assert status.item() == 0
    # valid tokens: the same codes and scales (stale ones may differ)
    def tokens(c):
        out = [torch.zeros((B, Lcap, Hkv, D), dtype=torch.int8 if dtype == "int8kv" else torch.bfloat16, device=dev) for _ in range(2)]
        start, n = i32([0] * B), i32([c_ + n_ for c_, n_ in zip(ctx, nq)])
        if dtype == "int8kv":
            out += [torch.zeros((B, Lcap, Hkv), device=dev) for _ in range(2)]
            bass.bass_kv_gather_int8(d.replace(kmax=Lcap), *c, *out, start, n)
        else:
            bass.bass_kv_gather(d.replace(kmax=Lcap), *c, *out, start, n)
        return out
    assert all(torch.equal(a, b) for a, b in zip(tokens(caches), tokens(by_append)))
    # probabilities are rounded to bf16: 2^-9 of each, times values of up to 5; the rows' sums stay in 32 bits
    assert np.abs(O.cpu().numpy() - want).max() <= 2e-2 and np.abs(lse.cpu().numpy() - want_lse).max() <= 1e-3


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("ctx", [[600, 333, 640, 64, 5]])
@pytest.mark.parametrize("D,kmax,Hq,Hkv", [(128, 40, 56, 56), (64, 33, 60, 60)])
def test_long_drafts_of_many_units_in_small_caches(dtype, ctx, D, kmax, Hq, Hkv):
    """280 and 300 units of more than 32 rows, caches of at most 24 blocks: appended by a launch of their own over bf16 caches too."""
    test_stretches_of_several_blocks(dtype, ctx, D, kmax, Hq, Hkv)


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("kmax", [32, 33])
def test_refused_launch_of_many_long_drafts_appends_nothing(dtype, kmax):
    """More than 256 units of 32 row slots and more: the rows are appended by a launch of their own, but for 32 rows over bf16 caches, which
    the attention launch appends.  Either way a plan of another shape stops it before anything is written."""
    import torch
    import paper_2404_15778_amd as bass
    dev, B, H, D, Lcap = "cuda:0", 17, 16, 128, 96
    d = bass.make_desc(B, kmax, H, H, D, Lcap, dtype, 1.0 / math.sqrt(D))
    gen = torch.Generator(device=dev)
    gen.manual_seed(1)
    Q, K, V = [torch.randn((B, kmax, H, D), generator=gen, device=dev).to(torch.bfloat16) for _ in range(3)]
    lens = [torch.full((B,), x, dtype=torch.int32, device=dev) for x in (40, 32)]
    caches = [torch.full((bass.bass_kv_cache_bytes(d),), 3, dtype=torch.uint8, device=dev) for _ in range(2)]
    O, status = torch.full((B, kmax, H, D), 7.0, device=dev), torch.zeros(1, dtype=torch.int32, device=dev)
    plan, ws = bass.alloc_plan(d, dev), bass.alloc_workspace(d, dev)
    bass.bass_attention_plan(d.replace(Lcap=Lcap + 32), *lens, bass.PLAN_APPEND, 0, plan, status)  # another shape
    bass.bass_verify_attention_planned(d, Q, K, V, *caches, plan, O, None, ws, status)
    assert status.item() == bass.STATUS_PLAN_MISMATCH
    assert (O == 7.0).all() and all((c == 3).all() for c in caches)
    status.zero_()
    bass.bass_attention_plan(d, *lens, bass.PLAN_APPEND, 0, plan, status)
    want = [c.clone() for c in caches]
    bass.bass_kv_append(d, *want, K, V, *lens)
    bass.bass_verify_attention_planned(d, Q, K, V, *caches, plan, O, None, ws, status)
    assert status.item() == 0 and all(torch.equal(a, b) for a, b in zip(caches, want)) and not (O == 7.0).any()
