"""Short block lists go to fewer shares than the launch has wavefronts or workgroups (CPU: the host planner)."""
import pytest

import paper_2404_15778_amd as bass
from test_attention_plan import check_plan


def busy_shares(plan):
    return sum(1 for r in plan["records"] if int(r[16]))


# blocks of the 8 units: stretches of 4 real blocks unless a fifth of the entries (7 virtual ones per unit) is less, then of 8
@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("ctx,shares", [(0, 8), (28, 8), (29, 8), (32, 8), (124, 8), (125, 16), (330, 24), (380, 24), (420, 32), (530, 24), (1240, 40), (4000, 128)])
def test_shares_of_few_units(dtype, ctx, shares):
    Hkv = 8
    d = bass.make_desc(1, 4, Hkv, Hkv, 128, 4096, dtype, 1.0)
    plan = check_plan(d, [ctx], [4], bass.PLAN_APPEND, 0, expect_shares=768)
    entries, blocks = int(plan["hdr"][10]), -(-(ctx + 4) // 32)
    assert entries == (blocks + 7) * Hkv
    assert busy_shares(plan) == shares <= max(entries // 5, Hkv)
    assert shares == Hkv * (-(-blocks // 4) if Hkv * -(-blocks // 4) <= max(entries // 5, Hkv) else -(-blocks // 8))


def test_explicit_spread_and_fp32_are_left_alone():
    d = bass.make_desc(1, 4, 8, 8, 128, 4096, "fp32", 1.0)
    plan = check_plan(d, [600], [4], 0, 0)
    assert max(int(r[8 * i + 5]) for r in plan["records"] for i in range(min(2, int(r[16])))) == 1  # one block each
    try:
        bass.bass_set_attention_waves(512)
        d = bass.make_desc(1, 4, 8, 8, 128, 4096, "bf16", 1.0)
        plan = check_plan(d, [600], [4], 0, 0, expect_shares=512)
        assert max(int(r[8 * i + 5]) for r in plan["records"] for i in range(min(2, int(r[16])))) == 1
    finally:
        bass.bass_set_attention_waves(0)


# At most 80 units: fewer than 256 shares where a fifth of the entries is at most 128, or at most 25 units; of whole units, as above.  More units:
# all 768 wavefronts, 3 virtual entries per unit (a share of virtual entries only has nothing to do).
@pytest.mark.parametrize("B,ctx,shares", [(1, 20, 32), (2, 20, 64), (1, 1000, 256), (2, 1000, 256), (1, 3000, 256), (3, 640, 768), (4, 20, 128), (3, 200, 768)])
def test_fewer_shares_only_where_they_are_worth_it(B, ctx, shares):
    d = bass.make_desc(B, 4, 32, 32, 128, 4096, "bf16", 1.0)
    plan = check_plan(d, [ctx] * B, [4] * B, bass.PLAN_APPEND, 0, expect_shares=768)
    assert shares - 3 * B * 32 <= busy_shares(plan) <= shares
    if B * 32 <= 80 and ctx <= 1000:
        assert busy_shares(plan) == shares


# More than 32 rows of few units, which share rows: at least 1 entry for a share, 2 from units of 17 entries on, 4 from 34 over INT8 caches,
# where that leaves less than all (256, INT8 512) of them
@pytest.mark.parametrize("dtype,ctx,shares", [("bf16", 20, 32), ("bf16", 180, 72), ("bf16", 400, 128), ("bf16", 440, 68), ("bf16", 1500, 204), ("bf16", 1900, 252), ("bf16", 2000, 256), ("bf16", 4000, 256),
                                              ("int8kv", 180, 72), ("int8kv", 400, 128), ("int8kv", 440, 68), ("int8kv", 930, 132), ("int8kv", 970, 68), ("int8kv", 1000, 70), ("int8kv", 4000, 258)])
def test_shares_of_few_units_that_share_rows(dtype, ctx, shares):
    d = bass.make_desc(1, 6, 64, 8, 128, 4096, dtype, 1.0)
    plan = check_plan(d, [ctx], [6], bass.PLAN_APPEND, 0)
    entries = int(plan["hdr"][10])
    most, least = (256, 1 if entries < 136 else 2) if dtype == "bf16" else (512, 1 if entries < 136 else 2 if entries < 272 else 4)
    assert entries == (-(-(ctx + 6) // 32) + 3) * 8 and shares == min(most, entries // least)
    assert shares - 3 * 8 <= busy_shares(plan) <= shares
