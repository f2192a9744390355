"""Attention over selected blocks of rings that have moved on: the newest block anywhere in the ring, ids on both sides of the
wrap, the newest block chosen or not, partly filled or not; both attention kernels, paged or not; against the blocks'
decompressed tokens attended in float64."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd.cache import TierConfig, TieredCache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads", [(4, 4), (8, 2), (40, 2)])
@pytest.mark.parametrize("paged", [None, 3])
@pytest.mark.parametrize("ring,first,tokens", [(9, 0, 9 * 64), (9, 5, 9 * 64), (9, 40, 7 * 64 + 13), (9, 44, 64 * 8 + 1), (5, 24, 3 * 64)])
def test_ids_across_the_wrap(heads, paged, ring, first, tokens):
    Hq, Hkv = heads
    g = torch.Generator(device="cuda:0").manual_seed(ring + first)
    c = TieredCache(1, Hq, Hkv, [TierConfig("f16", "f16", 10**9, 64, 2), TierConfig("f16", "f16", 10**9, 64, ring, paged_seed=paged, summary=True)])
    try:
        c.start[1][:] = first * 64
        k, v = (torch.randn(Hkv, tokens, 128, generator=g, device="cuda:0").half() for _ in range(2))
        c.append(1, k, v, seq=0)
        n = (tokens + 63) // 64
        q = torch.randn(1, Hq, 128, generator=g, device="cuda:0").half()
        kn, vn = (torch.randn(1, Hkv, 1, 128, generator=g, device="cuda:0").half() for _ in range(2))
        for keep in sorted({1, n // 2, n - 1, n}):
            c.start[0][:], c.len[0][:] = 0, 0
            out, lse = c.step(q, kn, vn, select_k=keep)
            torch.cuda.synchronize()
            ids = c.sel_blocks[0, :int(c.sel_count[0])].numpy() - first
            assert len(ids) == keep and ids.min() >= 0 and ids.max() < n
            tok = np.concatenate([np.arange(i * 64, min(i * 64 + 64, tokens)) for i in ids])
            kk = torch.cat([k[:, tok], kn[0]], 1).double().repeat_interleave(Hq // Hkv, 0)
            vv = torch.cat([v[:, tok], vn[0]], 1).double().repeat_interleave(Hq // Hkv, 0)
            s = (q[0].double()[:, None, :] * kk).sum(-1) / np.sqrt(128.0)
            want = (torch.softmax(s, -1)[..., None] * vv).sum(1)
            # exact fp16 operands, weights of 22 bits or fp32, sums in fp32: a few 1e-7 (a wrong block shows as 1e-1)
            assert float((out[0].double() - want).norm() / want.norm()) <= 1e-5
            assert float((lse[0].double() - torch.logsumexp(s, -1)).abs().max()) <= 1e-5
    finally:
        c.close()
