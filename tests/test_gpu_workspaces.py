"""Calls whose split-K plan needs more parts than a bound of the caller's allows.  The caches are empty rows (zeros):
what is tested is that the calls are taken, and what they return."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd.cache import TierConfig, TieredCache

pytestmark = pytest.mark.gpu


def zeros_cache(batch, Hq, Hkv, tiers, summary):
    """tiers: (k_fmt, v_fmt, block tokens, tokens held)."""
    cfg = [TierConfig(k, v, 10**9, bt, n // bt + 3, summary=summary and t == len(tiers) - 1) for t, (k, v, bt, n) in enumerate(tiers)]
    c = TieredCache(batch, Hq, Hkv, cfg)
    for t, (_, _, _, n) in enumerate(tiers):
        c.len[t][:] = n
    return c


@pytest.mark.parametrize("batch,Hq,Hkv,k,tiers", [
    (3, 8, 2, 1, [("f16", "f16", 128, 1341), ("i8", "i8", 128, 35438), ("i8", "i4", 128, 640)]),
    (4, 28, 4, 1, [("f16", "f16", 128, 171), ("i8", "i8", 128, 35902), ("i4", "i4", 64, 1536)]),
    (1, 16, 16, 5, [("f16", "f16", 128, 77), ("i8", "i8", 128, 49982), ("i4", "i4", 128, 3072)]),
])
def test_a_selection_that_cuts_the_other_tiers_finer(batch, Hq, Hkv, k, tiers):
    """With few blocks of the last tier selected there are fewer bytes in all, so the other tiers are cut into more items
    than a dense pass uses: the step takes the workspace it needs."""
    c = zeros_cache(batch, Hq, Hkv, tiers, True)
    try:
        z = torch.zeros(batch, Hkv, 1, 128, dtype=torch.float16, device="cuda:0")
        q = torch.ones(batch, Hq, 128, dtype=torch.float16, device="cuda:0")
        for s in range(2):
            out, lse = c.step(q, z, z, select_k=k)
            torch.cuda.synchronize()
            attended = tiers[0][3] + s + tiers[1][3] + k * tiers[2][2] + 1
            assert torch.all(out == 0)
            assert torch.allclose(lse, torch.full_like(lse, float(np.log(attended))), atol=1e-4)
        c.step(q, z, z)        # and a dense step with the same workspace
        torch.cuda.synchronize()
    finally:
        c.close()


@pytest.mark.parametrize("batch,Hq,Hkv,tiers", [
    (53, 64, 2, [("f16", "f16", 128, 1), ("i8", "i8", 128, 6879)]),
    (26, 64, 2, [("f16", "f16", 128, 1593), ("i4", "i4", 128, 24623)]),
])
def test_noalloc_takes_a_coarser_split_where_the_default_one_does_not_fit(batch, Hq, Hkv, tiers):
    """The default split's partials exceed the library's array (16 MiB); the same result as with a workspace, up to the
    rounding of another split: fp16 weights, 2^-11 of the values."""
    c = zeros_cache(batch, Hq, Hkv, tiers, False)
    try:
        g = torch.Generator(device="cuda:0")
        g.manual_seed(5)
        for t, (_, _, bt, n) in enumerate(tiers):
            c.len[t][:] = 0
            k, v = (torch.randn(batch, Hkv, n, 128, generator=g, device="cuda:0").half() for _ in range(2))
            c.append(t, k, v)
        parts = B.ttkv_count_parts(c.h, c.c)
        assert batch * Hq * parts * 520 > B.TTKV_NOALLOC_SCRATCH_BYTES
        q = torch.randn(batch, Hq, 128, generator=g, device="cuda:0").half()
        ref, ref_lse = (x.clone() for x in c.decode(q))
        out, lse = torch.full_like(ref, 7.0), torch.full_like(ref_lse, 7.0)
        B.ttkv_decode_attn_noalloc(c.h, c.c, q, B.F16, out, lse, None, None, 0, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert float((out - ref).abs().max()) <= 2e-3 * float(ref.abs().max())
        assert torch.allclose(lse, ref_lse, atol=1e-4)
        assert B.ttkv_count_parts(c.h, c.c) == parts       # the default stays the default
    finally:
        c.close()
