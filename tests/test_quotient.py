"""The conversion kernels' quotient at the codes (Sec. 4.2's quantizers are fixed as one IEEE division per element followed
by round-to-nearest-even and a clamp): q = x r, t = q + (x - q s) r in fused steps, clamped, then rounded by adding
1.5 x 2^23.  Emulated here in fp32 with numpy against the plain division, on scales of every fp16 magnitude (subnormal
and largest included) and quotients placed on, next to and between the half-integers, far outside the code range too:
after the clamp the two must agree everywhere.  (The GPU tests compare the kernels' codes with the oracle's.)"""
import numpy as np
import pytest

F, L = np.float32, np.longdouble


def codes(x, s, lo, hi):
    """(the kernels' codes, the recipe's)"""
    x, s = x.astype(F), s.astype(F)
    r = (F(1.0) / s).astype(F)
    q = (x * r).astype(F)
    e = (x.astype(L) - q.astype(L) * s.astype(L)).astype(F)
    t = (e.astype(L) * r.astype(L) + q.astype(L)).astype(F)
    got = ((np.clip(t, F(lo), F(hi)) + F(12582912.0)).astype(F) - F(12582912.0)).astype(F)
    return got, np.clip(np.rint((x / s).astype(F)), lo, hi)


@pytest.mark.parametrize("lo,hi", [(-127, 127), (0, 15)])
def test_reciprocal_quotient_equals_the_division_after_the_clamp(lo, hi):
    g = np.random.default_rng(1976900 + hi)
    n = 2_000_000
    s = g.integers(1, 0x7BFF, n).astype(np.uint16).view(np.float16).astype(F)              # every positive finite half
    k = g.integers(-300, 300, n).astype(F)
    frac = np.where(g.random(n) < 0.5, 0.5, g.random(n)).astype(F)                          # half of them exact ties
    jitter = (1 + g.integers(-4, 5, n) * F(2.0 ** -23)).astype(F)                           # and a few ulps around them
    got, want = codes((k + frac) * s * jitter, s, lo, hi)
    assert np.array_equal(got, want)
    x = g.standard_normal((200_000, 32)).astype(np.float16).astype(F)
    sc = (np.abs(x).max(1, keepdims=True) / F(127)).astype(np.float16).astype(F)
    got, want = codes(x.ravel(), np.repeat(sc, 32, 1).ravel(), lo, hi)
    assert np.array_equal(got, want)
