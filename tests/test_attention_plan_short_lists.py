"""Short block lists go to fewer shares than the launch has wavefronts (CPU: the host planner)."""
import pytest

import paper_2404_15778_amd as bass
from test_attention_plan import check_plan


@pytest.mark.parametrize("dtype,per_unit", [("bf16", 5), ("int8kv", 8)])
@pytest.mark.parametrize("ctx", [0, 31, 32, 330, 1240, 4000])
def test_shares_per_unit(dtype, per_unit, ctx):
    Hkv = 8
    d = bass.make_desc(1, 4, Hkv, Hkv, 128, 4096, dtype, 1.0)
    plan = check_plan(d, [ctx], [4], bass.PLAN_APPEND, 0, expect_shares=768)
    entries = int(plan["hdr"][10])
    busy = sum(1 for r in plan["records"] if int(r[16]))
    assert busy <= min(768, max(entries // 5, per_unit * Hkv))
    if entries >= 5 * 768:
        assert busy >= 768 - Hkv  # at most the stretches of virtual blocks have no segment


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


@pytest.mark.parametrize("B,ctx,few", [(1, 1000, True), (2, 1000, True), (3, 640, False), (4, 20, False), (3, 200, False), (2, 20, True)])
def test_fewer_shares_only_where_they_are_worth_it(B, ctx, few):
    d = bass.make_desc(B, 4, 32, 32, 128, 4096, "bf16", 1.0)
    plan = check_plan(d, [ctx] * B, [4] * B, bass.PLAN_APPEND, 0, expect_shares=768)
    assert all(bool(int(r[19]) & 2) == few for r in plan["records"])  # the flag under which remainders are multiplied
