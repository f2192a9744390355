"""The eviction cascade in one call against its boundaries one after the other: the same bytes, sums and positions, whether the
boundaries go in one launch, wait for each other (a block that only just arrived moves on) or move several blocks."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd.cache import TierConfig, TieredCache

pytestmark = pytest.mark.gpu

F16, BF16, I8, I4 = ("f16", "f16"), ("bf16", "bf16"), ("i8", "i8"), ("i4", "i4")
# tiers: formats, block tokens, capacity; held: tokens of every sequence in each tier
CASES = {
    "independent": ([(F16, 128, 512), (I8, 128, 1024), (I4, 256, 10**9)], [[512, 500, 520], [1000, 1024, 900], [640, 128, 384]], True),
    "dependent": ([(F16, 256, 256), (I8, 128, 128), (I4, 128, 10**9)], [[256, 300, 10], [0, 64, 0], [0, 128, 384]], True),
    "several_blocks": ([(F16, 64, 256), (I8, 64, 256), (("i8", "i4"), 128, 10**9)], [[450, 256, 100], [255, 320, 64], [64, 0, 128]], False),
    "four_tiers": ([(BF16, 64, 128), (BF16, 128, 256), (I8, 64, 192), (I4, 64, 10**9)],
                   [[128, 130, 128], [256, 320, 192], [192, 128, 190], [64, 0, 320]], True),
    "no_sums_anywhere": ([(F16, 64, 128), (I8, 64, 128), (("i8", "i4c"), 128, 10**9)], [[130, 128, 64], [96, 100, 127], [96, 0, 32]], False),
    "grouped_keys": ([(F16, 128, 256), (I8, 128, 256), (("i4t", "i4"), 128, 10**9)], [[256, 300, 256], [256, 256, 128], [128, 0, 256]], True),
    "first_only": ([(F16, 64, 128), (I8, 64, 1024), (I4, 64, 10**9)], [[128, 0, 191], [64, 0, 100], [0, 0, 64]], True),
    "skipping_one": ([(F16, 64, 128), (I8, 64, 4096), (I8, 64, 128), (I4, 128, 10**9)],
                     [[128, 0, 191], [64, 0, 100], [128, 160, 0], [0, 0, 64]], False),
}


def filled(tiers, held, summary, paged, heads):
    dt = torch.bfloat16 if tiers[0][0] == BF16 else torch.float16
    cfg = [TierConfig(f[0], f[1], cap, bt, max(held[t]) // bt + 12, "device", 5 + t if paged else None, summary and t == len(tiers) - 1)
           for t, (f, bt, cap) in enumerate(tiers)]
    c = TieredCache(3, *heads, cfg)
    for t in range(len(tiers)):
        c.start[t][:] = [(3 + 5 * b) % cfg[t].ring_blocks * cfg[t].block_tokens for b in range(3)]
    g = torch.Generator(device="cuda:0").manual_seed(77)
    for t in range(len(tiers) - 1, -1, -1):
        for b, n in enumerate(held[t]):
            if n:
                k, v = (torch.randn(heads[1], n, 128, generator=g, device="cuda:0").to(dt) for _ in range(2))
                c.append(t, k, v, seq=b, through_tiers=True)
    return c


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_one_call_and_boundary_by_boundary(name, paged):
    tiers, held, summary = CASES[name]
    heads = (4, 2)
    one, many = (filled(tiers, held, summary, paged, heads) for _ in range(2))
    try:
        k0 = one.stats()["kernels"]
        one.demote()
        s = torch.cuda.current_stream().cuda_stream
        for t in range(len(tiers) - 1):
            B.ttkv_tier_demote(many.h, many.c, t, 0, None, 0, s, s)
        torch.cuda.synchronize()
        a, b = one.stats(), many.stats()
        assert a["demotions"] == b["demotions"] > 0 and a["kernels"] <= b["kernels"]
        if name in ("independent", "no_sums_anywhere", "skipping_one"):
            assert a["kernels"] - k0 == 1, a
        for t in range(len(tiers)):
            assert np.array_equal(one.start[t], many.start[t]) and np.array_equal(one.len[t], many.len[t]), t
            assert torch.equal(one.pool[t], many.pool[t]), t
        if summary:
            assert torch.equal(one.ksum, many.ksum) and torch.equal(one.kmu.view(torch.int16), many.kmu.view(torch.int16))
    finally:
        one.close()
        many.close()


def test_a_refused_boundary_ends_the_cascade():
    """The third tier's ring has no room: the first boundary has moved its block, the second none."""
    c = filled([(F16, 64, 128), (I8, 64, 128), (I4, 64, 10**9)], [[128] * 3, [128] * 3, [64] * 3], False, False, (4, 2))
    try:
        c.len[2][1] = c.cfg[2].ring_blocks * 64
        with pytest.raises(B.TTKVError) as e:
            c.demote()
        assert e.value.status == B.ERR_CAPACITY
        torch.cuda.synchronize()
        assert [int(x) for x in c.len[0]] == [64] * 3 and [int(x) for x in c.len[1]] == [192] * 3 and int(c.len[2][0]) == 64
    finally:
        c.close()


@pytest.mark.parametrize("tokens", [64, 192])      # one unit of 64 rows, and three: workgroups of two units, one of them alone
@pytest.mark.parametrize("last", [("i4", "i4"), ("i8", "i4c")])
def test_units_side_by_side(tokens, last):
    """Blocks whose 64-row units do not pair up, rows that start inside a unit, sums beside conversions without them."""
    tiers = [(F16, tokens, tokens), (I8, tokens, 2 * tokens), (last, 64, 10**9)]
    held = [[tokens, tokens + 1, tokens], [tokens, 2 * tokens - 1, 2 * tokens + 32], [32, 64, 96]]
    one, many = (filled(tiers, held, True, False, (6, 3)) for _ in range(2))
    try:
        one.demote()
        s = torch.cuda.current_stream().cuda_stream
        for t in range(2):
            B.ttkv_tier_demote(many.h, many.c, t, 0, None, 0, s, s)
        torch.cuda.synchronize()
        assert one.stats()["demotions"] == many.stats()["demotions"] >= 6
        for t in range(3):
            assert np.array_equal(one.len[t], many.len[t]) and torch.equal(one.pool[t], many.pool[t]), t
        assert torch.equal(one.ksum, many.ksum) and torch.equal(one.kmu.view(torch.int16), many.kmu.view(torch.int16))
    finally:
        one.close()
        many.close()
