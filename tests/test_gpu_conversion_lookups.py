"""Conversions find entry, KV head, ring block and row without divisions: block sizes that are no powers of two (the last
tier's are: its means are products with a rounded 1 / block), odd numbers of sequences and KV heads, rings that wrap, paged or
not, against the oracle (codes and sums bit for bit)."""
import numpy as np
import pytest

from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("paged", [None, 4])
@pytest.mark.parametrize("sizes", [(64, 192, 256), (192, 64, 1024), (320, 448, 128)])
@pytest.mark.parametrize("last", [("i4", "i4"), ("i8", "i4"), ("i4t", "i4")])
def test_blocks_of_any_size(sizes, last, paged):
    if last[0] == "i4t" and (sizes[1] % 128 or sizes[2] % 128):
        sizes = (128, 384, 256)
    a, b, c = sizes
    tiers = [dict(k_fmt="f16", v_fmt="f16", capacity=2 * a, block_tokens=a, ring_blocks=4, paged_seed=paged),
             dict(k_fmt="i8", v_fmt="i8", capacity=2 * b, block_tokens=b, ring_blocks=3 + 2 * a // b + 2, paged_seed=paged),
             dict(k_fmt=last[0], v_fmt=last[1], capacity=10**9, block_tokens=c, ring_blocks=9, paged_seed=paged, summary=True)]
    p = Pair(3, 6, 3, tiers, "f16")
    try:
        for s in range(3):
            p.load(s, *synth.kv(500 + s, 3, 2 * a - 1 + b + 128 * (s + 1), "f16"))
        g = synth.rng(9)
        for _ in range(a + 2):   # a block of every sequence moves down, and the next one soon after
            args = [synth.normal(g, (3, 6, 128), "f16")] + [synth.normal(g, (3, 3, 128), "f16") for _ in range(2)]
            p.ora.step(*args)
            p.gpu.step(dev(args[0], "f16"), dev(args[1][:, :, None, :], "f16"), dev(args[2][:, :, None, :], "f16"))
        p.assert_state_equal()
        for s in range(3):
            for blk, mu in p.ora.summaries(s).items():
                assert np.array_equal(p.gpu.dump_summary(2, s, blk), mu), (s, blk)
    finally:
        p.close()
