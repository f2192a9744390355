"""fp16 and bf16 tiers under grouped queries: the softmax weights meet the values with 22 bits (fp16 and remainder, times
2^14), also where most of them are far below the largest, and for heads whose scores are beyond 2^22 in powers of two, whose
weights carry no power of two.  Against float64: the weights' 2^-22, exact products, fp32 sums of up to 5000 terms and the
merge stay below 5e-6 of the result (2-norm; measured 5e-7); with weights rounded to 16 bits once 3e-5 to 1e-4."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, assert_close, dev

pytestmark = pytest.mark.gpu


def run(dtype, q, k, v, split, mem="device", scale=None):
    n = k.shape[1]
    p = Pair(1, q.shape[1], k.shape[0], [dict(k_fmt=dtype, v_fmt=dtype, capacity=10**9, block_tokens=64, ring_blocks=n // 64 + 2, mem=mem)],
             dtype, host_append_direct=True)
    try:
        B.ttkv_set_split(p.gpu.h, split)
        if scale is not None:
            p.gpu.c.softmax_scale = p.ora.scale = scale
        p.load(0, k, v)
        out, lse = p.gpu.decode(dev(q, dtype))
        torch.cuda.synchronize()
        assert p.gpu.stats()["mfma_launches"] > 0
        return out.cpu().numpy().astype(np.float64)[0], lse.cpu().numpy().astype(np.float64)[0], p.ora.attend(q)
    finally:
        p.close()


@pytest.mark.parametrize("G", [2, 5, 16])
@pytest.mark.parametrize("n", [1, 33, 700, 5000])
@pytest.mark.parametrize("dtype,mem", [("f16", "device"), ("bf16", "device"), ("f16", "host")])
@pytest.mark.parametrize("peaked", [False, True])
def test_weights_keep_22_bits(dtype, mem, n, G, peaked):
    seed = synth.SEED_BASE + 1000 + G + n
    k, v = synth.kv(seed, 2, n, dtype)
    q = synth.normal(synth.rng(seed), (1, 2 * G, 128), dtype)
    if peaked:      # one token 8 above the rest, in the middle: the others together weigh about as much
        k[:, n // 2] = synth.round_to(8.0 * np.sqrt(128.0) * q[0].reshape(2, G, 128)[:, 0] / 128.0, dtype)
    out, lse, _ = run(dtype, q, k, v, 1 if peaked else 0, mem)
    s = np.einsum("hgd,htd->hgt", q[0].reshape(2, G, 128).astype(np.float64), k.astype(np.float64)) / np.sqrt(128.0)
    w = np.exp(s - s.max(-1, keepdims=True))
    want = (np.einsum("hgt,htd->hgd", w, v.astype(np.float64)) / w.sum(-1, keepdims=True)).reshape(2 * G, 128)
    err = np.linalg.norm(out - want, axis=1) / np.linalg.norm(want, axis=1)
    assert err.max() <= 5e-6, err.max()
    assert np.abs(lse - (s.max(-1) + np.log(w.sum(-1))).reshape(-1)).max() <= 1e-5


@pytest.mark.parametrize("G", [2, 16])
def test_scores_beyond_four_million(G):
    """Scores of 2.9e6 beside ordinary heads; all tokens have one value, so the rounding of such scores does not show."""
    n = 640
    q = np.zeros((1, G, 128), np.float32)
    q[..., :64], q[..., 64] = 512.0, 1.0
    q[:, 1::2] = synth.round_to(1e-3 * synth.rng(7).standard_normal((1, G // 2, 128)).astype(np.float32), "f16")
    k = np.zeros((1, n, 128), np.float32)
    k[..., :64] = 1010.0
    for t, x in ((133, 16.0), (261, 30.0), (639, 30.0)):
        k[:, t, 64] = x
    v = np.broadcast_to(np.where(np.arange(128) % 3 == 0, 65504.0, -65504.0).astype(np.float32), (1, n, 128)).copy()
    out, lse, (ro, rl) = run("f16", q, k, v, 1)
    assert_close(out, ro[0], "out")
    assert_close(lse, rl[0], "lse")
    assert np.linalg.norm(out - ro[0]) <= 1e-5 * np.linalg.norm(ro[0])


@pytest.mark.parametrize("scale", [1e-30, 1e37])
def test_zero_scores_at_any_scale(scale):
    v = synth.normal(synth.rng(8), (1, 416, 128), "f16")
    q = synth.normal(synth.rng(9), (1, 4, 128), "f16")
    out, lse, (ro, _) = run("f16", q, np.zeros((1, 416, 128), np.float32), v, 0, scale=np.float32(scale))
    assert_close(out, ro[0], "out")
    assert np.abs(lse - np.log(416)).max() <= 1e-5
