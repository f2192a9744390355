"""The split of caches without 4-bit tiers: one sequence, or sequences of unequal length, are cut for two workgroups per CU (512),
several of equal length for three (test_abi.py holds their plans); the plan follows when lengths become unequal."""
import numpy as np
import pytest

from paper_2604_19769_amd import binding as B
from test_abi import plan_cache


@pytest.mark.parametrize("heads", [(32, 8), (16, 4), (6, 1)])
@pytest.mark.parametrize("tiers", [[("f16", "f16", 128, 0)], [("bf16", "bf16", 128, 255), ("i8", "i8", 128, 0)]])
def test_one_sequence_takes_one_round_of_two_per_cu(heads, tiers):
    n = 512 // heads[1] * 1024                      # as many items of 1024 tokens of the long tier as one round has
    c = plan_cache(1, *heads, [t[:3] + (t[3] or n,) for t in tiers])
    h = B.ttkv_create()
    try:
        parts = B.ttkv_count_parts(h, c) - (len(tiers) - 1)
        assert 0.95 * 512 <= parts * heads[1] <= 512, parts
    finally:
        B.ttkv_destroy(h)


def test_unequal_lengths_change_the_plan_and_back():
    c = plan_cache(4, 32, 8, [("f16", "f16", 128, 255), ("i8", "i8", 128, 65536)])
    h = B.ttkv_create()
    try:
        assert B.ttkv_count_parts(h, c) == 1 + 24
        lens = c._keep[5]
        lens[1] = 65536 - 128
        assert B.ttkv_count_parts(h, c) <= 1 + 17
        lens[1] = 65536
        assert B.ttkv_count_parts(h, c) == 1 + 24
        many = np.arange(4) * 8192 + 128               # ragged: items of 256 to 8192 tokens cover every sequence
        lens[:] = many
        assert 1 + int(many.max()) // 8192 <= B.ttkv_count_parts(h, c) <= 1 + -(-int(many.max()) // 256)
    finally:
        B.ttkv_destroy(h)


@pytest.mark.parametrize("heads,tiers,parts", [
    ((8, 2), [("f16", "f16", 64, 507), ("i8", "i8", 64, 3584)], 4 + 28),             # 64 workgroups: items of 128 tokens
    ((32, 8), [("f16", "f16", 128, 4096)], 32),                                      # 256: one per CU, the most
    ((32, 8), [("f16", "f16", 128, 4097)], 17),                                      # 33 items would be 264
    ((8, 2), [("f16", "f16", 128, 300), ("i4", "i4", 128, 1024)], 3 + 4),            # int4 keys: 256 tokens are a batch per wave
    ((4, 4), [("f16", "f16", 128, 512)], 2),                                         # the vector kernel
])
def test_launches_that_leave_cus_idle_are_cut_finer(heads, tiers, parts):
    c = plan_cache(1, *heads, tiers)
    h = B.ttkv_create()
    try:
        assert B.ttkv_count_parts(h, c) == parts
        B.ttkv_set_split(h, 1 << 20)
        assert B.ttkv_count_parts(h, c) == sum(-(-t[3] // 256) for t in tiers)
    finally:
        B.ttkv_destroy(h)
