"""The first step on a cache of exactly as many tokens as a launch of 256 workgroups takes in items of 128: the cache with the
step's token has about half the parts, and the workspace covers both."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from test_gpu_workspaces import zeros_cache

pytestmark = pytest.mark.gpu

F, I8 = ("f16", "f16", 128), ("i8", "i8", 128)


@pytest.mark.parametrize("one_call", [True, False])
@pytest.mark.parametrize("batch,Hq,Hkv,tiers", [
    (1, 8, 2, [F + (16384,)]), (1, 16, 4, [F + (8192,)]), (1, 64, 4, [F + (8192,)]), (1, 8, 1, [F + (32768,)]),
    (2, 8, 2, [F + (8192,)]), (1, 8, 2, [F + (512,), I8 + (15872,)]), (1, 8, 2, [F + (16383,)]),
])
def test_a_step_at_the_longest_cache_of_short_items(batch, Hq, Hkv, tiers, one_call):
    """Empty rows (zeros): every token weighs the same."""
    c = zeros_cache(batch, Hq, Hkv, tiers, False)
    c.one_call_step = one_call
    try:
        z = torch.zeros(batch, Hkv, 1, 128, dtype=torch.float16, device="cuda:0")
        q = torch.ones(batch, Hq, 128, dtype=torch.float16, device="cuda:0")
        tokens = sum(t[3] for t in tiers)
        for s in range(3):
            out, lse = c.step(q, z, z)
            torch.cuda.synchronize()
            assert torch.all(out == 0)
            assert torch.allclose(lse, torch.full_like(lse, float(np.log(tokens + s + 1))), atol=1e-4)
    finally:
        c.close()


def test_the_same_result_in_a_workspace_for_the_longer_cache():
    """A caller's workspace with room for the parts of one token more: the 256-token items it holds give the result of the
    128-token ones up to the rounding of sums of 16384 terms in fp32."""
    c = zeros_cache(1, 8, 2, [F + (16384,)], False)
    try:
        g = torch.Generator(device="cuda:0").manual_seed(11)
        c.len[0][:] = 0
        k, v = (torch.randn(1, 2, 16384, 128, generator=g, device="cuda:0").half() for _ in range(2))
        c.append(0, k, v)
        q = torch.randn(1, 8, 128, generator=g, device="cuda:0").half()
        ref, ref_lse = (x.clone() for x in c.decode(q))
        assert B.ttkv_count_parts(c.h, c.c) == 128
        c.len[0] += 1
        parts = B.ttkv_count_parts(c.h, c.c)
        c.len[0] -= 1
        assert parts == 65
        need = B.ttkv_workspace_bytes(c.c, parts, 0)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
        out, lse = torch.full_like(ref, 7.0), torch.full_like(ref_lse, 7.0)
        s = torch.cuda.current_stream().cuda_stream
        B.ttkv_decode_attn(c.h, c.c, q, B.F16, out, lse, None, None, 0, ws, need, 0, s, s)
        torch.cuda.synchronize()
        assert float((out - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
        assert torch.allclose(lse, ref_lse, atol=1e-5)
    finally:
        c.close()


def test_a_selection_of_few_blocks_keeps_short_items():
    """A workspace made for a dense step of 256-token items holds the 128-token ones of a selection."""
    c = zeros_cache(1, 8, 2, [F + (300,), I8 + (65536,)], True)
    try:
        z = torch.zeros(1, 2, 1, 128, dtype=torch.float16, device="cuda:0")
        q = torch.ones(1, 8, 128, dtype=torch.float16, device="cuda:0")
        c.step(q, z, z)
        out, lse = c.step(q, z, z, select_k=100)
        torch.cuda.synchronize()
        assert c.ws_parts >= 3 + 100
        assert torch.all(out == 0)
        assert torch.allclose(lse, torch.full_like(lse, float(np.log(300 + 2 + 100 * 128))), atol=1e-4)
    finally:
        c.close()
