"""Block selection over numbers of live blocks at the edges of the two ranking kernels (up to 256 blocks ranks are counted, beyond
it a radix select) and the two forms of the scoring launch (up to 1024 blocks of all sequences together, and more), of waves and of four; ties, NaN and both zeros; numbers of query heads that are no powers of two.  Scores,
and so the selection, are defined bit for bit; the ids reach the caller's memory whether it is page-locked or not."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd.cache import TierConfig, TieredCache

pytestmark = pytest.mark.gpu


def phi(q, mean, G):
    """Per head a chain of fused multiply-adds over the channels in ascending order, then the heads in ascending order: in
    float64 with one rounding per step (a product of two halves is exact in 32 bits, so the step rounds once)."""
    s = np.zeros((mean.shape[0], q.shape[0]), np.float32)
    m = np.repeat(mean, G, axis=1).astype(np.float64)
    for d in range(128):
        s = (s.astype(np.float64) + q[None, :, d].astype(np.float64) * m[:, :, d]).astype(np.float32)
    out = np.zeros(mean.shape[0], np.float32)
    for h in range(q.shape[0]):
        out = out + s[:, h]
    return out


@pytest.mark.parametrize("n", [1, 3, 4, 63, 64, 65, 127, 255, 256, 257, 512, 513, 700, 1024])
@pytest.mark.parametrize("heads", [(8, 2), (14, 2), (5, 5), (72, 8)])
@pytest.mark.parametrize("kind", ["ordinary", "ties", "special"])
def test_ids_at_every_number_of_blocks(n, heads, kind):
    Hq, Hkv = heads
    g = np.random.default_rng(n + Hq)
    mean = g.standard_normal((2 * n, Hkv, 128)).astype(np.float16)
    if kind == "ties":
        mean = mean[g.integers(0, max(1, n // 5), 2 * n)]
    if kind == "special":
        mean[::3] = 0.0
        mean[1::7] = -0.0
        mean[2::5, 0, 5] = np.nan
        mean[4::11, 0, 9] = np.inf
    q = g.standard_normal((2, Hq, 128)).astype(np.float16)
    c = TieredCache(2, Hq, Hkv, [TierConfig("f16", "f16", 10**9, 64, 2), TierConfig("i8", "i8", 10**9, 64, n, paged_seed=3, summary=True)])
    try:
        lens = [64 * n, max(1, 64 * n - 64 * (n // 3) - 5)]
        c.len[1][:] = lens
        c.start[1][:] = [64 * 5 * n, 64 * (n - 1)]                     # rings that have moved on
        c.kmu.view(2 * n, Hkv, 128).copy_(torch.from_numpy(mean).cuda())
        for k in sorted({1, max(1, n // 2), n, n + 3}):
            blocks, count = c.select(torch.from_numpy(q).cuda(), k)
            for b in range(2):
                first, end = int(c.start[1][b]) // 64, (int(c.start[1][b]) + lens[b] + 63) // 64
                with np.errstate(all="ignore"):
                    s = phi(q[b], mean[[c.table[1][b][i % n] for i in range(first, end)]], Hq // Hkv)
                s[np.isnan(s)] = -np.inf
                s[s == 0] = 0.0
                want = np.sort(np.argsort(-s, kind="stable")[:k]) + first
                assert int(count[b]) == len(want)
                assert np.array_equal(blocks[b, :len(want)].numpy(), want), (k, b)
    finally:
        c.close()


@pytest.mark.parametrize("pinned", [True, False])
@pytest.mark.parametrize("heads", [(8, 2), (4, 4), (40, 2)])      # matrix cores, vector kernel, blocks of heads
@pytest.mark.parametrize("lens", [(128 * 9, 128 * 4), (128 * 9, 0)])
def test_ids_reach_the_callers_memory(heads, lens, pinned):
    g = torch.Generator(device="cuda:0").manual_seed(5)
    c = TieredCache(2, *heads, [TierConfig("f16", "f16", 10**9, 64, 8), TierConfig("i8", "i8", 10**9, 128, 10, summary=True)])
    try:
        for b in range(2):
            for t, n in ((1, lens[b]), (0, 70)):
                if n:
                    k, v = (torch.randn(heads[1], n, 128, generator=g, device="cuda:0").half() for _ in range(2))
                    c.append(t, k, v, seq=b)
        q = torch.randn(2, heads[0], 128, generator=g, device="cuda:0").half()
        kn, vn = (torch.randn(2, heads[1], 1, 128, generator=g, device="cuda:0").half() for _ in range(2))
        k = 6
        blocks, count = c.select(q, k)
        want = [blocks[b, :int(count[b])].tolist() for b in range(2)]
        assert [len(w) for w in want] == [min(k, n // 128) for n in lens]
        c.sel_blocks = torch.full((2, k), -7, dtype=torch.int32, pin_memory=pinned)
        c.sel_count = torch.full((2,), -7, dtype=torch.int32, pin_memory=pinned)
        for _ in range(3):
            c.step(q, kn, vn, select_k=k)
            torch.cuda.synchronize()
            assert [c.sel_blocks[b, :int(c.sel_count[b])].tolist() for b in range(2)] == want
    finally:
        c.close()
