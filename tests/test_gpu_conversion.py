"""Row conversion at the edges of its units (64 rows of one destination block; a whole block where key sums are kept):
rows that start and end inside a unit, sources that straddle two blocks, sums continued over several arrivals, groups of
32 and 128 tokens, and groups whose scale is zero, subnormal or far from their values.  Codes, scales, zeros and mean
keys bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, dev

pytestmark = pytest.mark.gpu


def awkward(x, dtype):
    """Rows and groups with zero, constant, tiny and offset values among ordinary ones."""
    x = x.copy()
    x[:, 3::17] = 0.0
    x[:, 5::19] = 2.5
    x[:, 7::23] *= 1e-6
    x[:, 11::29] = x[:, 11::29] * 0.01 + 40.0
    x[:, 13::31, 64:] = -0.0
    return synth.round_to(x, dtype)


def check(p):
    p.assert_state_equal()
    last = len(p.tiers) - 1
    if p.tiers[last].get("summary"):
        for b in range(p.B):
            for blk, mu in p.ora.summaries(b).items():
                assert np.array_equal(p.gpu.dump_summary(last, b, blk), mu), (b, blk)


CASES = {
    # last tier's blocks larger than, smaller than and not a multiple of what arrives; odd lengths everywhere
    "summary_512": ("f16", [("f16", "f16", 256, 64, 6), ("i8", "i8", 448, 192, 5), ("i4", "i4", 10**9, 512, 8)], True, False),
    "summary_small_blocks": ("bf16", [("bf16", "bf16", 384, 192, 4), ("i4", "i4", 640, 320, 5), ("i8", "i8", 10**9, 64, 60)], True, True),
    "summary_fp": ("f16", [("i8", "i8", 256, 128, 4), ("i4", "i4", 10**9, 1024, 4)], True, False),
    "four_tiers": ("bf16", [("bf16", "bf16", 192, 64, 5), ("i8", "i4", 320, 192, 4), ("i4", "i4", 256, 128, 6), ("i8", "i8", 10**9, 448, 9)], False, True),
    "channel_major": ("f16", [("f16", "f16", 256, 128, 4), ("i8", "i8", 384, 64, 10), ("i4", "i4c", 10**9, 256, 16)], True, True),
    "over_tokens": ("bf16", [("bf16", "bf16", 256, 128, 4), ("i8", "i8", 384, 128, 6), ("i4t", "i4", 10**9, 256, 14)], True, False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_units_and_sums(name):
    dtype, tiers, summary, paged = CASES[name]
    spec = [dict(k_fmt=k, v_fmt=v, capacity=c, block_tokens=bt, ring_blocks=r, paged_seed=5 + i if paged else None,
                 summary=summary and i == len(tiers) - 1) for i, (k, v, c, bt, r) in enumerate(tiers)]
    whole = 128 if name == "over_tokens" else 32 if name == "channel_major" else 1   # the last tier takes whole groups
    p = Pair(3, 6, 3, spec, dtype)
    try:
        # the tiers above the last one are full but for one token: what is left over is the last tier's length
        above = spec[0]["capacity"] - 1 + sum(t["capacity"] for t in spec[1:-1])
        for b, n in enumerate((1, 333, 1217)):
            n = -(-n // whole) * whole + above
            k, v = synth.kv(900 + b, 3, n, dtype)
            p.load(b, awkward(k, dtype), awkward(v, dtype))
        check(p)
        g = synth.rng(17)
        bt = spec[0]["block_tokens"]
        for s in range(2 * bt + 3):          # every sequence evicts at least twice; partly filled blocks continue
            r = [synth.normal(g, (3, h, 128), dtype) for h in (6, 3, 3)]
            p.step(*r)
            if s in (0, 1, bt, bt + 1):
                check(p)
        check(p)
    finally:
        p.close()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 200])
def test_fp32_source(n):
    """fp32 rows appended in two calls, the second one starting inside a unit."""
    spec = [dict(k_fmt="i8", v_fmt="i4", capacity=10**9, block_tokens=128, ring_blocks=6, summary=True)]
    p = Pair(1, 2, 2, spec, "f16")
    try:
        k, v = (np.float32(1.0) * x for x in synth.kv(77, 2, n + 77, "f16"))
        k, v = (k * np.float32(1.2345678)).astype(np.float32), (v * np.float32(0.7654321)).astype(np.float32)
        for lo, hi in ((0, 77), (77, 77 + n)):
            p.ora.append(0, 0, k[:, lo:hi], v[:, lo:hi], lo)
            p.gpu.append(0, *(torch.from_numpy(np.ascontiguousarray(x[:, lo:hi])).cuda() for x in (k, v)), seq=0)
        check(p)
    finally:
        p.close()


@pytest.mark.parametrize("name", ["rows", "channel_major", "over_tokens", "summary"])
def test_zero_points_beyond_half_precision(name):
    """Minima outside fp16's range (bf16 values may lie there): a zero point of minus infinity puts every element of the
    group at the top code, one of plus infinity at code 0, whatever the scale; ordinary rows beside them."""
    g = synth.rng(31)
    k, v = synth.kv(78, 2, 256, "bf16")
    ramp = g.random((2, 256, 128)).astype(np.float32)
    for x in (k, v):
        x[:, 1::5] = -1e5 + 4e4 * ramp[:, 1::5]          # finite scale, zero point -inf
        x[:, 2::7] = 1e5 + 4e4 * ramp[:, 2::7]           # zero point +inf
        x[:, 3::11] = -1e5                               # and a scale of zero
        x[:, 4::13] = 3e6 * (ramp[:, 4::13] - 0.5)       # scale infinite as well
    if name == "over_tokens":
        k[:, :128] = -1e5 + 4e4 * ramp[:, :128]
        k[:, 128:, ::2] = 1e5
    spec = {"rows": ("i4", "i4"), "channel_major": ("i8", "i4c"), "over_tokens": ("i4t", "i4"), "summary": ("i4", "i4")}[name]
    tiers = [dict(k_fmt="bf16", v_fmt="bf16", capacity=128, block_tokens=128, ring_blocks=3),
             dict(k_fmt=spec[0], v_fmt=spec[1], capacity=10**9, block_tokens=128, ring_blocks=4, summary=name == "summary")]
    p = Pair(1, 4, 2, tiers, "bf16")
    try:
        for x in (k, v):
            x[...] = synth.round_to(x, "bf16")
        p.ora.append(1, 0, k, v, 0)
        p.gpu.append(1, dev(k, "bf16"), dev(v, "bf16"), seq=0)
        p.assert_state_equal()
    finally:
        p.close()
