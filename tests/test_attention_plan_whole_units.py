"""Short units are not cut apart by the virtual entries of their pads: where every unit can have stretches of its own, of four blocks or
eight, in no more shares than an even division would take, it gets them (CPU: the host planner)."""
import pytest

import paper_2404_15778_amd as bass
from test_attention_plan import check_plan, parse_plan, segments_of


# heads, query slots, type, context of every sequence, blocks of the longest stretch
@pytest.mark.parametrize("Hq,Hkv,D,kmax,dtype,ctx,most", [
    (32, 8, 128, 8, "bf16", [60], 3), (32, 8, 128, 8, "int8kv", [60, 90, 5, 118], 4), (32, 8, 64, 4, "bf16", [100] * 4, 4),  # one stretch a unit
    (32, 32, 128, 8, "bf16", [370], 4),                      # a tile of 16 rows: 12 blocks, three stretches
    (32, 8, 128, 8, "bf16", [3900], 4),                      # 256 stretches of four blocks
    (64, 8, 128, 6, "bf16", [150] * 32, 5), (64, 8, 128, 6, "int8kv", [400] * 16, 8), (64, 8, 128, 8, "bf16", [60] * 32, 3),  # two tiles
])
def test_stretches_of_whole_units(Hq, Hkv, D, kmax, dtype, ctx, most):
    B = len(ctx)
    d = bass.make_desc(B, kmax, Hq, Hkv, D, 4096, dtype, 1.0)
    plan = check_plan(d, ctx, [kmax] * B, bass.PLAN_APPEND, 0)
    shares = [segments_of(plan, w) for w in range(plan["nshares"])]
    assert all(len(s) <= 1 for s in shares)
    assert max(n for s in shares for (_, _, _, _, _, n, _, _) in s) == most
    per = 4 if most <= 4 else 8
    assert sum(len(s) for s in shares) == sum(-(-(-(-(c + kmax) // 32)) // per) for c in ctx) * Hkv <= 256


# lists that are longer than 256 such stretches, or would take more shares: divided evenly, units end inside stretches
@pytest.mark.parametrize("Hq,Hkv,D,kmax,dtype,ctx", [(32, 8, 128, 8, "bf16", [4000] * 16), (64, 8, 128, 8, "int8kv", [1200, 3000] * 8),
                                                     (32, 32, 128, 8, "bf16", [1800, 2900]), (32, 32, 128, 32, "bf16", [100] * 9)])
def test_longer_lists_are_divided_evenly(Hq, Hkv, D, kmax, dtype, ctx):
    B = len(ctx)
    plan = check_plan(bass.make_desc(B, kmax, Hq, Hkv, D, 4096, dtype, 1.0), ctx, [kmax] * B, 0, 0)
    assert any(len(segments_of(plan, w)) > 1 for w in range(plan["nshares"]))


# More than 32 rows of few units in a large cache: the kernels that share rows (pads of 3 entries), whose shares have at least two entries,
# over INT8 caches four, where the units are long
@pytest.mark.parametrize("dtype,D,ctx,shares", [("bf16", 128, 60, 24), ("bf16", 128, 1000, 140), ("int8kv", 128, 1000, 70),
                                                ("int8kv", 64, 1000, 70), ("int8kv", 128, 500, 76)])
def test_few_units_share_rows(dtype, D, ctx, shares):
    d = bass.make_desc(1, 6, 64, 8, D, 4096, dtype, 1.0)
    plan = check_plan(d, [ctx], [6], bass.PLAN_APPEND, 0, expect_shares=256 if dtype == "bf16" else 1024)
    assert int(plan["hdr"][6]) == 3
    assert shares - 8 <= sum(1 for r in plan["records"] if int(r[16])) <= shares


# (300 sequences: two rounds of the planning workgroups' threads, 512 shares; 1500: planned through global memory, not whole)
@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,D,kmax,dtype,longest", [(1, 32, 8, 128, 8, "bf16", 370), (32, 64, 8, 128, 6, "int8kv", 200), (7, 8, 8, 64, 3, "bf16", 500),
                                                           (300, 1, 1, 64, 20, "bf16", 100), (1500, 2, 1, 64, 10, "int8kv", 70)])
@pytest.mark.parametrize("padded", [0, 90])
def test_device_plan_is_the_host_plan(B, Hq, Hkv, D, kmax, dtype, longest, padded):
    import numpy as np
    import torch
    rng = np.random.default_rng(B)
    ctx, nq = rng.integers(-2, longest, B), rng.integers(0, kmax + 1, B)
    ctx[0], nq[0] = longest, kmax
    d = bass.make_desc(B, kmax, Hq, Hkv, D, longest + kmax, dtype, 1.0)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda:0")  # noqa: E731
    plan, status = torch.zeros(bass.bass_attention_plan_bytes(d), dtype=torch.uint8, device="cuda:0"), i32([0])
    bass.bass_attention_plan(d, i32(ctx), i32(nq), 0, padded, plan, status)
    host, host_status = bass.bass_attention_plan_host(d, ctx, nq, 0, padded)
    words = check_plan(d, ctx, nq, 0, padded)
    got = plan.cpu().numpy()
    got_parts, want_parts = parse_plan(got, B, Hkv), parse_plan(host, B, Hkv)
    for part in ("hdr", "records", "seq_L", "seq_nq", "seq_inc", "owners"):
        assert (got_parts[part] == want_parts[part]).all(), part
    for w in range(words["nshares"]):
        assert segments_of(got_parts, w) == segments_of(want_parts, w)
    assert status.item() == host_status


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("Hq,Hkv,D,kmax", [(8, 4, 128, 3), (12, 4, 64, 7), (48, 6, 128, 8), (40, 8, 64, 7)])  # 6, 21, 64 and 35 rows
@pytest.mark.parametrize("ctx", [[60, 3, 0, 31, 90], [128, 200, 5, 255, 33]])  # stretches of four blocks; of eight with more rows
def test_attention_over_whole_units(dtype, Hq, Hkv, D, kmax, ctx):
    import numpy as np
    import oracle
    import workloads as wl
    from oracle.kv_int8 import dequantize_rows, quantize_rows
    from paper_2404_15778_amd import harness
    nq = [kmax, 1, kmax, 0, kmax - 1]
    w = wl.make_attention("whole", 5, Hq, Hkv, D, "bf16", ctx, nq, 23, kmax=kmax, Lcap=900)
    Q, K, V = w.Q, w.K, w.V
    if dtype == "int8kv":
        Q, K, V = (dequantize_rows(*quantize_rows(wl.bf16_bits_to_f32(x))) for x in (Q, K, V))
        w.dtype = dtype
    want, want_lse = oracle.verify_attention(Q, K, V, w.ctx_len, w.draft_len, w.scale)
    for fused in (False, True):
        O, lse, status, da = harness.run_attention_workload(w, poison=True, fused=fused)
        # probabilities and V are rounded to bf16 (2^-9 each) for outputs of magnitude up to about 4; lse stays in 32 bits
        assert status == 0 and np.abs(O - want).max() <= 2e-2 and np.abs(lse - want_lse).max() <= 1e-4
    O, lse = da.verify(harness.to_device(w.Q), harness.i32(ctx), harness.i32(nq), variant="pad", padded_len=300)
    assert np.abs(O.cpu().numpy() - want).max() <= 2e-2 and np.abs(lse.cpu().numpy() - want_lse).max() <= 1e-4
