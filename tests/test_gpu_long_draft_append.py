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
