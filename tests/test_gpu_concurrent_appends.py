"""Appends to disjoint tokens may run at the same time on two streams, also where the tokens share a 32-token block: each
writes nothing but its own rows."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("split", [13, 32 + 2, 64 + 31])  # the second append goes on inside a block of the first
def test_two_streams_fill_one_block(dtype, D, split):
    import torch
    import paper_2404_15778_amd as bass
    dev, B, H, total = "cuda:0", 16, 32, 120
    kmax = max(split, total - split, 32)  # by blocks
    d = bass.make_desc(B, kmax, H, H, D, total, dtype, 1.0)
    gen = torch.Generator(device=dev)
    gen.manual_seed(D + split)
    rows = [[torch.randn((B, kmax, H, D), generator=gen, device=dev).to(torch.bfloat16) for _ in range(2)] for _ in range(2)]
    lens = [[torch.full((B,), x, dtype=torch.int32, device=dev) for x in pair] for pair in ((0, split), (split, total - split))]
    size = bass.bass_kv_cache_bytes(d)
    make = lambda: [torch.full((size,), 0x5A, dtype=torch.uint8, device=dev) for _ in range(2)]  # noqa: E731
    want = make()
    for i in range(2):
        bass.bass_kv_append(d, *want, *rows[i], *lens[i])
    streams = [torch.cuda.Stream() for _ in range(2)]
    caches = [make() for _ in range(8)]
    torch.cuda.synchronize()
    for c in caches:
        for i in range(2):
            bass.bass_kv_append(d, *c, *rows[i], *lens[i], stream=streams[i])
    torch.cuda.synchronize()
    for c in caches:
        assert all(torch.equal(a, b) for a, b in zip(c, want))


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("D,kmax,Hq,Hkv", [(128, 20, 16, 16), (64, 33, 16, 16), (128, 32, 32, 16)])
def test_attention_appends_a_long_draft_beside_an_append(dtype, D, kmax, Hq, Hkv):
    """A planned launch appends its drafts itself; the tokens behind them, in the same block, come from another stream."""
    import torch
    import paper_2404_15778_amd as bass
    dev, B, ctx, more = "cuda:0", 8, 75, 24
    nq = kmax - 1
    d = bass.make_desc(B, kmax, Hq, Hkv, D, ctx + kmax + more, dtype, 1.0 / D**0.5)
    gen = torch.Generator(device=dev)
    gen.manual_seed(D + kmax)
    rand = lambda n, H: torch.randn((B, n, H, D), generator=gen, device=dev).to(torch.bfloat16)  # noqa: E731
    fill = lambda x: torch.full((B,), x, dtype=torch.int32, device=dev)  # noqa: E731
    head, draft, tail, Q = [[rand(n, Hkv) for _ in range(2)] for n in (ctx, kmax, more)] + [rand(kmax, Hq)]
    base = [torch.zeros(bass.bass_kv_cache_bytes(d), dtype=torch.uint8, device=dev) for _ in range(2)]
    bass.bass_kv_append(d.replace(kmax=ctx), *base, *head, fill(0), fill(ctx))
    lens, behind = (fill(ctx), fill(nq)), (fill(ctx + nq), fill(more))
    plan, status = bass.alloc_plan(d, dev), torch.zeros(1, dtype=torch.int32, device=dev)
    bass.bass_attention_plan(d, *lens, bass.PLAN_APPEND, 0, plan, status)

    def run(first, second):
        c = [t.clone() for t in base]
        O, ws = torch.zeros((B, kmax, Hq, D), device=dev), bass.alloc_workspace(d, dev)
        torch.cuda.synchronize()
        bass.bass_verify_attention_planned(d, Q, *draft, *c, plan, O, None, ws, status, stream=first)
        bass.bass_kv_append(d.replace(kmax=more), *c, *tail, *behind, stream=second)
        torch.cuda.synchronize()
        return [O, *c]

    streams = [torch.cuda.Stream() for _ in range(2)]
    want = run(streams[0], streams[0])
    for _ in range(8):
        assert all(torch.equal(a, b) for a, b in zip(run(*streams), want))
    assert status.item() == 0
