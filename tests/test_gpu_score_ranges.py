"""Grouped-query attention over quantized tiers at the ends of the score range that the entry points accept: scores so large
that the weights of their heads carry no power of two, and heads whose queries differ by a factor of millions."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, assert_close, dev

pytestmark = pytest.mark.gpu

FORMATS = [("i8", "i8"), ("i8", "i4"), ("i4", "i4"), ("i8", "i4c"), ("i4", "i4c")]


def run(kfmt, vfmt, q, k, v, mem, scale=None):
    """One KV head, the last 63 tokens of k and v in an fp16 window, the others in one work item of a quantized tier."""
    n = k.shape[1]
    tiers = [dict(k_fmt="f16", v_fmt="f16", capacity=64, block_tokens=64, ring_blocks=3),
             dict(k_fmt=kfmt, v_fmt=vfmt, capacity=10**9, block_tokens=128, ring_blocks=n // 128 + 2, mem=mem)]
    p = Pair(1, q.shape[1], 1, tiers, "f16", host_append_direct=True)
    try:
        B.ttkv_set_split(p.gpu.h, 1)
        if scale is not None:
            p.gpu.c.softmax_scale = p.ora.scale = scale
        p.load(0, k, v)
        out, lse = p.gpu.decode(dev(q, "f16"))
        torch.cuda.synchronize()
        assert p.gpu.stats()["mfma_launches"] > 0
        ro, rl = p.ora.attend(q)
        return out.cpu().numpy().astype(np.float64)[0], lse.cpu().numpy()[0], ro[0], rl[0]
    finally:
        p.close()


@pytest.mark.parametrize("mem", ["device", "host"])
@pytest.mark.parametrize("ordinary", [0, 1])
@pytest.mark.parametrize("G", [2, 4, 8, 16])
@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
def test_scores_of_millions_beside_the_largest_values(kfmt, vfmt, G, ordinary, mem):
    """Scores of 2.9e6 (a reference beyond 2^22 in powers of two), a few tokens up to 2.7 above the ones their wave meets
    first, and values that span the whole fp16 range (int4 scales of 8736): a weight of 2^3.8 times such a scale is beyond
    fp16.  All tokens have the same value, so the result does not depend on how fp32 rounds scores of this size.
    ordinary: every second head has queries around 1 instead."""
    n = 640
    g = synth.rng(synth.SEED_BASE + 900 + G)
    q = np.zeros((1, G, 128), np.float32)
    q[..., :64], q[..., 64] = 512.0, 1.0
    if ordinary:
        q[:, 1::2] = synth.round_to(1e-3 * g.standard_normal((1, G // 2, 128)).astype(np.float32), "f16")
    k = np.zeros((1, n + 63, 128), np.float32)
    k[:, :n, :64], k[:, :n, 65] = 1010.0, 30.0
    for t, x in ((133, 16.0), (261, 30.0), (300, 30.0), (450, 24.0), (639, 30.0)):
        k[:, t, 64] = x
    v = np.zeros((1, n + 63, 128), np.float32)
    v[:, :n] = np.where(np.arange(128) % 3 == 0, 65504.0, -65504.0)
    v[:, n:] = v[:, :1]
    out, lse, ro, rl = run(kfmt, vfmt, q, k, v, mem)
    assert_close(out, ro, "out")
    assert_close(lse, rl, "lse")
    # exact codes, weights of 22 bits, sums of n terms in fp32: a few units of 2^-22; the window's value rows differ from the
    # dequantized ones only for the heads that see it
    assert np.linalg.norm(out - ro) <= 1e-5 * np.linalg.norm(ro)


@pytest.mark.parametrize("mem", ["device", "host"])
@pytest.mark.parametrize("G", [2, 4, 8, 16])
@pytest.mark.parametrize("kfmt,vfmt", [f for f in FORMATS if f[0] == "i4"])
def test_small_queries_beside_large_ones(kfmt, vfmt, G, mem):
    """A head with queries of 5000 does not take bits from the heads beside it: theirs are some 2.5e-4 here (fp16's smallest
    normal number is 6e-5) over keys up to 60000, scores around 10.  An error of up to 2^-21 in every second query element (what
    is left of one as a sixteenth of it, an fp16 subnormal) moves these scores by 7e-3."""
    n = 1088
    g = synth.rng(synth.SEED_BASE + 950 + G)
    k = synth.round_to(g.uniform(-60000.0, 60000.0, (1, n + 63, 128)).astype(np.float32), "f16")
    v = synth.normal(g, (1, n + 63, 128), "f16")
    q = synth.round_to(2.5e-4 * g.standard_normal((1, G, 128)).astype(np.float32), "f16")
    q[:, :, 0] = synth.round_to(np.array([0.002], np.float32), "f16")[0]
    k[:, n:] = 0.0
    k[:, n:, 0] = -60000.0                     # the window, whose weights are rounded to 16 bits: e^-40 of the others
    q[:, G // 2] = 0.0
    q[:, G // 2, 7] = 5000.0
    out, lse, ro, rl = run(kfmt, vfmt, q, k, v, mem)
    small = np.arange(G) != G // 2
    assert np.all(np.isfinite(out))
    assert_close(out[small], ro[small], "out")
    # codes are exact, products summed in fp32: 2^-21 of a score's terms (some 100 together) at the most, i.e. 5e-5 of a weight
    assert np.linalg.norm(out[small] - ro[small]) <= 2e-4 * np.linalg.norm(ro[small])
    assert np.abs(lse[small] - rl[small]).max() <= 2e-4


@pytest.mark.parametrize("scale", [1e-30, 1e30, 1e37])
@pytest.mark.parametrize("G", [4, 16])
@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
def test_zero_scores_at_any_scale(kfmt, vfmt, G, scale):
    """Keys of zero have scores of zero whatever the softmax scale: the result is the mean of the values."""
    n = 416
    g = synth.rng(synth.SEED_BASE + 990)
    k, v = np.zeros((1, n + 63, 128), np.float32), synth.normal(g, (1, n + 63, 128), "f16")
    q = synth.normal(g, (1, G, 128), "f16")
    out, lse, ro, rl = run(kfmt, vfmt, q, k, v, "device", np.float32(scale))
    assert_close(out, ro, "out")
    assert np.abs(lse - np.log(n + 63)).max() <= 1e-5
