"""A decode call allocates host memory only when its plan is larger than any before it.  Counted in a child process in
which operator new is this test's own: two identical attention calls (recorded by ttkv_staged_schedule, so without a
GPU), the second one with no allocation."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COUNTER = r"""
#include <cstdlib>
#include <new>
static long count;
extern "C" long allocations() { return count; }
void *operator new(size_t n) { ++count; return std::malloc(n); }
void *operator new[](size_t n) { ++count; return std::malloc(n); }
void *operator new(size_t n, const std::nothrow_t &) noexcept { ++count; return std::malloc(n); }
void *operator new[](size_t n, const std::nothrow_t &) noexcept { ++count; return std::malloc(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }
"""

CHILD = r"""
import ctypes as C, sys
sys.path[:0] = [sys.argv[1], sys.argv[1] + "/tests"]
counter = C.CDLL(sys.argv[2], mode=C.RTLD_GLOBAL)
counter.allocations.restype = C.c_long
from paper_2604_19769_amd import binding as B
from test_abi import plan_cache
h = B.ttkv_create()
assert counter.allocations() > 0                      # the counter sees the library
for batch, Hq, Hkv, tiers in ((4, 32, 8, [("f16", "f16", 128, 2013), ("i8", "i8", 128, 8192), ("i4", "i4", 128, 30720)]),
                              (3, 8, 8, [("f16", "f16", 128, 2013), ("i4", "i4", 128, 30720)])):
    c = plan_cache(batch, Hq, Hkv, tiers)
    n = C.c_int32()
    call = lambda: B.lib().ttkv_staged_schedule(h, C.byref(c), None, None, 0, 0, 1, None, 0, C.byref(n))
    assert call() == B.OK and n.value > 0
    before = counter.allocations()
    assert call() == B.OK
    print(counter.allocations() - before)
"""


def test_an_identical_second_call_allocates_nothing(tmp_path):
    src, so = tmp_path / "counter.cpp", tmp_path / "counter.so"
    src.write_text(COUNTER)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(so)], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, LD_PRELOAD=" ".join(x for x in (str(so), os.environ.get("LD_PRELOAD", "")) if x)))
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["0", "0"], r.stdout
