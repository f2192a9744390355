"""Conversion of groups on either side of the ordinary case (no NaN, a scale that is a normal fp16 number, a zero point
near the minimum) and of key sums in launches of many blocks: the two-step quotients against the division, emulated in
fp32, and codes, scales, zeros and mean keys bit for bit against the oracle."""
import numpy as np
import pytest

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
