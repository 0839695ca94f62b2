"""Appends and gathers of 32 rows and more go by cache blocks, fewer by single rows: both must leave the same bytes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

#        offset, rows: nothing, one row, around a block's edges, several blocks, past the end, before the start
SPANS = [(0, 0), (0, 32), (31, 1), (1, 31), (5, 70), (32, 64), (90, 33), (63, 2), (120, 20), (-3, 40), (130, 4)]


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hkv", [1, 3, 8, 9])
def test_blocks_and_rows_leave_the_same_bytes(dtype, D, Hkv):
    import torch
    import paper_2404_15778_amd as bass
    dev, B, kmax, Lcap, piece = "cuda:0", len(SPANS), 75, 133, 25
    gen = torch.Generator(device=dev)
    gen.manual_seed(D + Hkv)
    desc = bass.make_desc(B, kmax, Hkv, Hkv, D, Lcap, dtype, 1.0)
    size = bass.bass_kv_cache_bytes(desc)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)  # noqa: E731
    off, cnt = np.array([o for o, _ in SPANS]), np.array([n for _, n in SPANS])
    rows = [torch.randn((B, kmax, Hkv, D), generator=gen, device=dev).to(torch.bfloat16) for _ in range(2)]
    rows[0][:, 1] = 0  # a row of zeros
    old = [torch.randint(0, 255, (size,), generator=gen, device=dev, dtype=torch.uint8) for _ in range(2)]

    by_blocks, by_rows = [t.clone() for t in old], [t.clone() for t in old]
    st = torch.zeros(2, dtype=torch.int32, device=dev)
    bass.bass_kv_append(desc, *by_blocks, *rows, i32(off), i32(cnt), st[:1])
    for i in range(0, kmax, piece):
        part = [t[:, i:i + piece].contiguous() for t in rows]
        bass.bass_kv_append(desc.replace(kmax=piece), *by_rows, *part, i32(off + i), i32(np.clip(cnt - i, 0, piece)), st[1:])
    assert all(torch.equal(a, b) for a, b in zip(by_blocks, by_rows))
    assert st[0].item() == st[1].item() != 0  # the rows outside the cache are reported

    def gather(k, o, n):
        shape = (B, k, Hkv, D)
        if dtype == "int8kv":
            out = [torch.full(shape, 7, dtype=torch.int8, device=dev) for _ in range(2)]
            out += [torch.full(shape[:3], 7.0, device=dev) for _ in range(2)]
            bass.bass_kv_gather_int8(desc.replace(kmax=k), *by_rows, *out, i32(o), i32(n))
        else:
            out = [torch.full(shape, 7, dtype=torch.bfloat16, device=dev) for _ in range(2)]
            bass.bass_kv_gather(desc.replace(kmax=k), *by_rows, *out, i32(o), i32(n))
        return out

    whole = gather(kmax, off, cnt)
    parts = [gather(piece, off + i, np.clip(cnt - i, 0, piece)) for i in range(0, kmax, piece)]
    for j, t in enumerate(whole):
        want = torch.cat([p[j] for p in parts], 1)
        assert torch.equal(t.view(torch.uint8), want.contiguous().view(torch.uint8))
