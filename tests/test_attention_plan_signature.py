"""A launch takes a plan only if both divide the work in the same way: everything the division and the launch's grid are
computed from is in the signature that every record carries (CPU: the host planner)."""
import numpy as np
import pytest

import paper_2404_15778_amd as bass
from test_attention_plan import parse_plan


def signature(waves=0, flags=0, B=2, kmax=4, Hq=8, Hkv=2, D=128, Lcap=512, dtype="bf16"):
    d = bass.make_desc(B, kmax, Hq, Hkv, D, Lcap, dtype, 1.0)
    bass.bass_set_attention_waves(waves)
    try:
        plan, _ = bass.bass_attention_plan_host(d, [100] * B, [kmax] * B, flags, 0)
    finally:
        bass.bass_set_attention_waves(0)
    got = {int(r[18]) for r in parse_plan(plan, B, Hkv)["records"]}
    assert len(got) == 1 and 0 not in got
    return got.pop()


@pytest.mark.parametrize("dtype,Hq", [("bf16", 2), ("bf16", 8), ("bf16", 16), ("int8kv", 8), ("int8kv", 16), ("fp32", 8)])
def test_same_shape_and_setting_give_the_same_signature(dtype, Hq):
    for waves in (0, 128, 768, 1024):
        assert signature(waves, Hq=Hq, dtype=dtype) == signature(waves, Hq=Hq, dtype=dtype)


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
def test_default_and_its_explicit_count_differ(dtype):
    # 768 wavefronts either way with one query tile, but only the default divides short lists over fewer shares
    assert signature(0, dtype=dtype) != signature(768, dtype=dtype)


@pytest.mark.parametrize("dtype", ["bf16", "int8kv"])
@pytest.mark.parametrize("waves", [128, 512, 1024, 8192])
def test_one_and_several_query_tiles_differ(dtype, waves):
    # 16 and 32 query rows per kv head: with INT8 caches both plans have `waves` records, but the launch for more than 16 rows
    # has a workgroup for every second one only
    assert signature(waves, Hq=8, dtype=dtype) != signature(waves, Hq=16, dtype=dtype)


def test_parts_of_the_shape_and_the_append_flag_differ():
    base = signature()
    others = [signature(B=3), signature(kmax=3), signature(Hq=4, Hkv=1), signature(Lcap=544), signature(256), signature(flags=bass.PLAN_APPEND)]
    assert len({base, *others}) == 1 + len(others)


def test_signatures_of_a_sweep_of_settings_are_distinct():
    counts = np.arange(64, 1024, 32)
    assert len({signature(int(w)) for w in counts}) == len(counts)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,plan_waves,plan_Hq,waves,Hq", [("bf16", 0, 2, 768, 2), ("int8kv", 768, 2, 0, 2), ("int8kv", 1024, 8, 1024, 16)])
def test_launch_refuses_the_other_division(dtype, plan_waves, plan_Hq, waves, Hq):
    import torch
    dev, B, kmax, Hkv, D, Lcap = "cuda:0", 2, 4, 2, 128, 512
    make = lambda h: bass.make_desc(B, kmax, h, Hkv, D, Lcap, dtype, 1.0)  # noqa: E731
    d = make(Hq)
    lens = [torch.tensor(x, dtype=torch.int32, device=dev) for x in ([300, 100], [4, 2])]
    cache = [torch.zeros(bass.bass_kv_cache_bytes(d), dtype=torch.uint8, device=dev) for _ in range(2)]
    Q = torch.zeros((B, kmax, Hq, D), dtype=torch.bfloat16, device=dev)
    O, status = torch.full((B, kmax, Hq, D), 7.0, device=dev), torch.zeros(1, dtype=torch.int32, device=dev)
    plan, ws = bass.alloc_plan(d, dev), bass.alloc_workspace(d, dev)
    try:
        bass.bass_set_attention_waves(plan_waves)
        bass.bass_attention_plan(make(plan_Hq), *lens, 0, 0, plan, status)
        bass.bass_set_attention_waves(waves)
        bass.bass_verify_attention_planned(d, Q, None, None, *cache, plan, O, None, ws, status)
    finally:
        bass.bass_set_attention_waves(0)
    assert status.item() == bass.STATUS_PLAN_MISMATCH and (O == 7.0).all()
