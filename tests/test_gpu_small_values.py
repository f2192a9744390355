"""Grouped-query attention over quantized values far from 1 beside a peaked softmax: the weights that carry the values'
scales to the matrix cores are 16-bit numbers, so the product of a small weight with a small scale must keep its bits.
One work item of several thousand tokens whose first token scores 5 to 7 above the rest (an attention sink), so that
the others' weights are 1e-3 to 1e-6 of the largest and yet a few per cent of the sum together; the values have a mean,
so what they contribute does not average out.  The oracle's bounds are the suite's own (2e-3 of the largest output)."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, assert_close, dev

pytestmark = pytest.mark.gpu

FORMATS = [("i8", "i8"), ("i8", "i4"), ("i4", "i4"), ("i8", "i4c"), ("i4", "i4c")]


def sink_case(kfmt, vfmt, Hq, Hkv, values, n=4096, mem="device", above=7.0, seed=0):
    """values(g, n) -> [Hkv][n][128] of the older tier.  One item over all n tokens, then the fp16 window."""
    g = synth.rng(synth.SEED_BASE + 700 + seed)
    tiers = [dict(k_fmt="f16", v_fmt="f16", capacity=64, block_tokens=64, ring_blocks=3),
             dict(k_fmt=kfmt, v_fmt=vfmt, capacity=10**9, block_tokens=256, ring_blocks=n // 256 + 2, mem=mem)]
    p = Pair(1, Hq, Hkv, tiers, "f16", host_append_direct=True)
    try:
        B.ttkv_set_split(p.gpu.h, 1)
        k, _ = synth.kv(synth.SEED_BASE + 701 + seed, Hkv, n + 63, "f16")
        u = synth.normal(g, (Hkv, 128), "f16")
        q = np.repeat(u, Hq // Hkv, axis=0) + 0.3 * g.standard_normal((Hq, 128), dtype=np.float32)
        q = synth.round_to(q[None], "f16")
        others = np.einsum("hd,hnd->hn", u, k).max(1) / np.sqrt(128.0)
        k[:, 0] = synth.round_to(u * ((others + above) * np.sqrt(128.0) / (u * u).sum(1))[:, None], "f16")
        v = np.zeros((Hkv, n + 63, 128), np.float32)
        v[:, :n] = values(g, n)
        v[:, n:] = v[:, n - 63:n]
        p.load(0, k, synth.round_to(v, "f16"))
        p.assert_state_equal()
        assert B.ttkv_count_parts(p.gpu.h, p.gpu.c) == 1 + (n + (8191 if mem == "device" else 2047)) // (8192 if mem == "device" else 2048)
        out, lse = p.gpu.decode(dev(q, "f16"))
        torch.cuda.synchronize()
        ro, rl = p.ora.attend(q)
        assert_close(out.cpu().numpy(), ro, "out")
        assert_close(lse.cpu().numpy(), rl, "lse")
        assert p.gpu.stats()["mfma_launches"] > 0
    finally:
        p.close()


@pytest.mark.parametrize("std", [1.0, 0.1, 0.02, 0.005])
@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
def test_small_values_beside_a_sink(kfmt, vfmt, std):
    sink_case(kfmt, vfmt, 8, 2, lambda g, n: std * (1.0 + g.standard_normal((2, n, 128), dtype=np.float32)))


@pytest.mark.parametrize("Hq,n,above", [(4, 8192, 7.0), (32, 3072, 5.0), (34, 4096, 6.0)])
@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
def test_small_values_by_heads_and_length(kfmt, vfmt, Hq, n, above):
    sink_case(kfmt, vfmt, Hq, 2, lambda g, n: 0.02 * (1.0 + g.standard_normal((2, n, 128), dtype=np.float32)), n, above=above, seed=Hq)


@pytest.mark.parametrize("kfmt,vfmt", [("i8", "i8"), ("i4", "i4c")])
def test_small_values_in_a_host_tier(kfmt, vfmt):
    sink_case(kfmt, vfmt, 8, 2, lambda g, n: 0.01 * (1.0 + g.standard_normal((2, n, 128), dtype=np.float32)), 2048, "host", seed=90)


@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
@pytest.mark.parametrize("order", ["growing", "falling", "zeros first", "large"])
def test_value_scales_that_change_within_the_item(kfmt, vfmt, order):
    """Magnitudes from 0.004 to 4 along the sequence either way, rows of zeros (scale 0) before the first other one, and
    values near the largest fp16 number (scales of several thousand)."""
    def values(g, n):
        x = 1.0 + g.standard_normal((2, n, 128), dtype=np.float32)
        step = np.arange(n, dtype=np.float32)[None, :, None] * 8 // n
        if order == "large":
            return np.clip(x * 12000.0, -65000, 65000)
        if order == "zeros first":
            x[:, :n // 2] = 0.0
            x[:, ::5] = 0.0
            return 0.004 * x
        return 0.004 * x * np.exp2(1.4 * (step if order == "growing" else 7 - step))
    sink_case(kfmt, vfmt, 8, 2, values, seed=50, above=3.0)
