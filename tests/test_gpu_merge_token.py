"""The merge with the step's new token: parts below and above a lane's one and the first batches of 64 and 256, numbers of query heads
that are and are not powers of two, and queries, keys and values that start at any even address."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, assert_close, dev

pytestmark = pytest.mark.gpu


def shifted(t):
    """The same values two bytes behind a 16-byte boundary."""
    buf = torch.zeros(t.numel() + 8, dtype=t.dtype, device=t.device)
    buf[1:1 + t.numel()] = t.reshape(-1)
    return buf[1:1 + t.numel()].view(t.shape)


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (3, 3), (6, 2), (14, 2), (40, 2)])
@pytest.mark.parametrize("tokens", [1, 2047, 9000, 20000, 66000])      # 1, 8, 36, 80 and 258 parts (256 tokens each)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_new_token_joins_any_number_of_parts(Hq, Hkv, tokens, dtype):
    p = Pair(2, Hq, Hkv, [dict(k_fmt=dtype, v_fmt=dtype, capacity=10**9, block_tokens=64, ring_blocks=tokens // 64 + 2)], dtype)
    try:
        B.ttkv_set_split(p.gpu.h, 1 << 16)
        seed = synth.SEED_BASE + 900 + Hq + tokens
        for b in range(2):
            p.load(b, *synth.kv(seed * 3 + b, Hkv, max(1, tokens - 700 * b), dtype))
        g = synth.rng(seed)
        q = synth.normal(g, (2, Hq, 128), dtype)
        kn, vn = synth.normal(g, (2, Hkv, 128), dtype), synth.normal(g, (2, Hkv, 128), dtype)
        kn[1] = synth.round_to(3.0 * q[1].reshape(Hkv, Hq // Hkv, 128).mean(1), dtype)   # a token that carries weight
        ro, rl = p.ora.step(q, kn, vn)[:2]
        out, lse = p.gpu.step(shifted(dev(q, dtype)), shifted(dev(kn[:, :, None, :], dtype)), shifted(dev(vn[:, :, None, :], dtype)))
        torch.cuda.synchronize()
        assert_close(out.cpu().numpy(), ro, "out")
        assert_close(lse.cpu().numpy(), rl, "lse")
        p.assert_state_equal()
    finally:
        p.close()
