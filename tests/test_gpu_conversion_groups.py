"""Conversion of groups on either side of the ordinary case (no NaN, a scale that is a normal fp16 number, a zero point
near the minimum) and of key sums in launches of many blocks: the two-step quotients against the division, emulated in
fp32, and codes, scales, zeros and mean keys bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import synth
from ttkv_testlib import Pair

F, L = np.float32, np.longdouble


def test_codes_of_eleven_bit_values_need_no_exact_quotient():
    """rint(y / s) = RN(RN(y r + 1536) + (1.5 2^23 - 1536)) - 1.5 2^23 with r = RN(1 / s), for every mantissa of s and of y
    and every ratio of powers of two that leaves |y / s| below 127.5: all ties and all neighbours of ties."""
    s = (np.arange(1024, dtype=np.uint16) + np.uint16(0x3C00)).view(np.float16).astype(F)
    y0 = s.copy()
    r = (F(1.0) / s).astype(F)
    for e in range(-14, 8):
        y = np.ldexp(y0, e).astype(F)[:, None]
        # y has 11 and r 24 significant bits: exact in 64-bit floats, one rounding to fp32 after the sum (which is exact too)
        q = (y.astype(np.float64) * r.astype(np.float64)[None] + 1536.0).astype(F)
        n = (q + F(12582912.0 - 1536.0)).astype(F) - F(12582912.0)
        exact = (y / s[None]).astype(F)
        live = exact < 127.5
        assert np.array_equal(n[live], np.rint(exact)[live]), e


def test_quotient_in_two_steps_is_correctly_rounded():
    """q = y r + RN(y r'), r = RN(1 / s), r' = RN(RN(1 - s r) r), equals RN(y / s): half-integers and their neighbours and any
    y, for fp16 mantissas of s.  (Products of 24-bit numbers are exact in 64-bit mantissas, and their sum with a term 2^-24 as
    large loses nothing that could matter: the quotient lies 2^-12 ulp from a midpoint or further.)"""
    g = np.random.default_rng(1976960)
    s = np.repeat((np.arange(1024, dtype=np.uint16) + np.uint16(0x3400)).view(np.float16).astype(F), 4000)
    r = (F(1.0) / s).astype(F)
    rest = ((1 - s.astype(L) * r.astype(L)).astype(F) * r).astype(F)
    ties = ((g.integers(0, 16, s.size) + 0.5) * s * (1 + g.integers(-3, 4, s.size) * F(2.0 ** -23))).astype(F)
    for y in (ties, (g.standard_normal(s.size) * 2.0 ** g.integers(-8, 9, s.size)).astype(F)):
        q = (y.astype(L) * r.astype(L) + (y * rest).astype(F).astype(L)).astype(F)
        assert np.array_equal(q, (y / s).astype(F))


def groups(x, dtype):
    """Rows whose scale is zero, subnormal, barely normal or infinite, whose minimum is far from its fp16 zero point, and
    ordinary ones beside them in the same wave."""
    x = x.copy()
    x[:, 1::7] = 0.0
    x[:, 2::11] *= 2e-6                                  # subnormal scales of both formats
    x[:, 3::13] *= 127 * 2.0 ** -14 / 4.0                 # around the smallest normal scale
    x[:, 4::17, 32:64] = 0.0                              # one group of a row
    x[:, 5::19] = x[:, 5::19] * 0.01 + 300.0              # zero point up to several scales off the minimum (bf16, int4 of int8)
    x[:, 6::23, 64:] = np.where(x[:, 6::23, 64:] > 0, 60000.0, -60000.0)   # about the largest span
    return synth.round_to(x, dtype)


CASES = {   # tiers above the last hold 511 tokens; the rest lands in blocks of the last one, 8 heads x many blocks or few
    "i4_via_i8": ("f16", [("f16", "f16", 256, 64, 6), ("i8", "i8", 256, 128, 4), ("i4", "i4", 10**9, 64, 132)]),
    "i8_via_i4": ("bf16", [("bf16", "bf16", 256, 64, 6), ("i4", "i4", 256, 128, 4), ("i8", "i8", 10**9, 64, 132)]),
    "i4": ("bf16", [("bf16", "bf16", 512, 64, 10), ("i4", "i4", 10**9, 64, 132)]),
    "i8": ("f16", [("f16", "f16", 512, 64, 10), ("i8", "i8", 10**9, 64, 132)]),
    "fp": ("f16", [("f16", "f16", 512, 64, 10), ("f16", "f16", 10**9, 64, 132)]),
}


@pytest.mark.gpu
@pytest.mark.parametrize("blocks", [3, 129])             # 24 and 1032 blocks of keys in the launch: 512 and 256 threads
@pytest.mark.parametrize("name", list(CASES))
def test_groups_and_sums(name, blocks):
    dtype, tiers = CASES[name]
    spec = [dict(k_fmt=k, v_fmt=v, capacity=c, block_tokens=bt, ring_blocks=r, summary=i == len(tiers) - 1)
            for i, (k, v, c, bt, r) in enumerate(tiers)]
    p = Pair(1, 8, 8, spec, dtype)
    try:
        n = 511 + 64 * (blocks - 1) + 37
        k, v = synth.kv(1976961, 8, n, dtype)
        p.load(0, groups(k, dtype), groups(v, dtype))
        p.assert_state_equal()
        for blk, mu in p.ora.summaries(0).items():
            assert np.array_equal(p.gpu.dump_summary(len(tiers) - 1, 0, blk), mu), blk
    finally:
        p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("summary", [False, True])
@pytest.mark.parametrize("bad", [np.nan, -np.nan, np.inf])
def test_groups_with_nan_beside_others(bad, summary):
    """A NaN does not count for its group's range, takes the lowest code and leaves every other byte alone, in waves with
    zero, tiny and ordinary groups; an infinity makes the scale of its own group infinite and changes no other group."""
    spec = [dict(k_fmt="i8", v_fmt="i4", capacity=10**9, block_tokens=64, ring_blocks=8, summary=summary)]
    k, v = synth.kv(1976962, 2, 300, "f16")
    k, v = groups(k, "f16"), groups(v, "f16")
    at = np.zeros((300, 128), bool)
    at[3::16, 7] = at[9::16, 70] = at[10::16, 100] = at[14::64, 33] = True
    dump = []
    for x in (0, bad):
        p = Pair(1, 2, 2, spec, "f16")
        try:
            kv = []
            for t in (k, v):
                t = t.copy()
                t[:, at] = x if x else np.roll(t, 1, axis=2)[:, at]    # a neighbour in the same group: the range as without it
                kv.append(torch.from_numpy(t).cuda().half().contiguous())
            p.gpu.append(0, *kv, seq=0)
            dump.append(p.gpu.dump_tier(0, 0))
        finally:
            p.close()
    without, got = dump
    nib = lambda d: np.stack([d & 15, d >> 4], -1).reshape(2, 300, 128)
    codes = [(without["k"], got["k"], 32, 0x81), (nib(without["v"]), nib(got["v"]), 64, 0)]
    for (a, b, g, low), name in zip(codes, "kv"):
        own = at.reshape(300, 128 // g, g)
        other = ~(np.broadcast_to(own.any(-1, keepdims=True), own.shape).reshape(300, 128) if np.isinf(bad) else at)
        assert np.array_equal(a[:, other], b[:, other]), name
        ma, mb = (d[name + "_meta"].view(np.uint16).reshape(2, 300, 128 // g, -1) for d in (without, got))
        if np.isinf(bad):
            hit = own.any(-1)
            assert np.array_equal(ma[:, ~hit], mb[:, ~hit]), name
            assert np.all(mb[:, hit][..., 0] == 0x7c00), name
        else:
            zero = (ma[..., 0] == 0)[..., None].repeat(g, -1).reshape(2, 300, 128)[:, at]   # a scale of zero: code 0 whatever the value
            assert np.array_equal(ma, mb), name
            assert np.array_equal(b[:, at][~zero], np.full((~zero).sum(), low, b.dtype)), name
