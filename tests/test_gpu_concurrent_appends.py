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
