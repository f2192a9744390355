"""The conversion kernels' shortcuts against the recipes they stand for (Sec. 4.2: one IEEE operation per step), emulated
in fp32 with numpy: the division by the constants 15 and 127, and by a group's fp16 scale, in three operations each.  (The GPU tests compare the kernels' codes and
key sums with the oracle's.)"""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

F = np.float32


@pytest.mark.parametrize("D", [15, 127])
def test_constant_division_is_correctly_rounded(D):
    """y = d * (1 / D), corrected by one residual: equal to d / D for every fp32 mantissa (scaling by powers of two
    changes nothing while no step leaves the normal range).  The fused steps are evaluated in extended precision: the
    residual has at most a few bits, so they are exact there before their one rounding."""
    c = F(1.0) / F(D)
    for e in (0, 7):
        d = (np.arange(1 << 23, dtype=np.uint32) | np.uint32((127 + e) << 23)).view(F)
        y = d * c
        res = (d.astype(np.longdouble) - np.longdouble(D) * y.astype(np.longdouble)).astype(F)
        q = (y.astype(np.longdouble) + res.astype(np.longdouble) * np.longdouble(c)).astype(F)
        assert np.array_equal(q, d / F(D))


def group_reciprocal(s, g):
    """1 / s from an approximation one unit in the last place off either way, corrected by one step."""
    r0 = (F(1.0) / s).astype(F)
    r0 = np.nextafter(r0, np.where(g.random(r0.shape) < 0.5, F(0), F(np.inf)).astype(F)).astype(F)
    e = (1 - s.astype(np.longdouble) * r0.astype(np.longdouble)).astype(F)
    return (e.astype(np.longdouble) * r0.astype(np.longdouble) + r0.astype(np.longdouble)).astype(F)


@pytest.mark.parametrize("kind", ["ties", "any"])
def test_quotient_by_a_half_precision_scale_is_correctly_rounded(kind):
    """q = y r, q + (y - q s) r in fused steps (Markstein's correction) equals y / s, for 2000 values of y with every
    fp16 mantissa of s, half-integers and their neighbours included; test_quotient_exhaustively takes every pair of
    mantissas, test_quotient.py scales of every magnitude and both code ranges."""
    g = np.random.default_rng(1976950)
    s = np.repeat((np.arange(1024, dtype=np.uint16) + np.uint16(0x3400)).view(np.float16).astype(F), 2000)
    r = group_reciprocal(s, g)
    assert np.array_equal(r, F(1.0) / s)
    if kind == "ties":
        y = ((g.integers(-130, 130, s.size) + 0.5) * s).astype(F)
        y = (y * (1 + g.integers(-3, 4, s.size) * F(2.0 ** -23))).astype(F)
    else:
        y = (g.standard_normal(s.size) * 2.0 ** g.integers(-8, 9, s.size)).astype(F)
    q = (y * r).astype(F)
    e = (y.astype(np.longdouble) - q.astype(np.longdouble) * s.astype(np.longdouble)).astype(F)
    t = (e.astype(np.longdouble) * r.astype(np.longdouble) + q.astype(np.longdouble)).astype(F)
    assert np.array_equal(t, (y / s).astype(F))
    c = np.clip(t, F(-127), F(127))
    assert np.array_equal(((c + F(12582912.0)).astype(F) - F(12582912.0)).astype(F), np.rint(c))


def test_quotient_exhaustively(tmp_path):
    """Every fp16 mantissa of s with every fp32 mantissa of y: 2^33 pairs, in C (exhaustive_quotient.c)."""
    if not {"fma", "avx2"} <= set(open("/proc/cpuinfo").read().split()):
        pytest.skip("needs a processor with fused multiply-add and 256-bit vectors")
    so = str(tmp_path / "exhaustive_quotient.so")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "exhaustive_quotient.c")
    subprocess.run(["gcc", "-O3", "-mfma", "-mavx2", "-ffp-contract=off", "-shared", "-fPIC", "-o", so, src], check=True)
    L = C.CDLL(so)
    L.check_scales.restype = C.c_longlong
    assert L.check_scales(0, 1024) == 0
