"""Grouped-query attention over quantized tiers at the ends of the score range that the entry points accept: scores so large
that the weights of their heads carry no power of two."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, assert_close, dev

pytestmark = pytest.mark.gpu

FORMATS = [("i8", "i8"), ("i8", "i4"), ("i4", "i4"), ("i8", "i4c"), ("i4", "i4c")]


def run(kfmt, vfmt, q, k, v, mem):
    """One KV head, the last 63 tokens of k and v in an fp16 window, the others in one work item of a quantized tier."""
    n = k.shape[1]
    tiers = [dict(k_fmt="f16", v_fmt="f16", capacity=64, block_tokens=64, ring_blocks=3),
             dict(k_fmt=kfmt, v_fmt=vfmt, capacity=10**9, block_tokens=128, ring_blocks=n // 128 + 2, mem=mem)]
    p = Pair(1, q.shape[1], 1, tiers, "f16", host_append_direct=True)
    try:
        B.ttkv_set_split(p.gpu.h, 1)
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
