"""The matrix-core kernel's quantized path places the heads of 1, 2 or 4 tiles in the 16 rows of a score product (16, 8 or 4
places), works in batches of 32 (int8 keys) or 64 tokens (int4), and lets the items of a run take turns at its batches:
numbers of heads around each boundary, lengths around a batch and a turn, few and many items.  The weights meet the values
with 22 bits and codes enter exactly: with the window's weights out of the way every sequence of every case below comes
within 5e-6 of the oracle (2-norm), most of it the scores' own sums in fp32.  Bound 2e-5.  Without the remainders of the weights
(rounded to 16 bits once) the sequences of 31 tokens and more are off by 1.1e-4 to 2.3e-4, so a lost or misplaced remainder shows."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from paper_2604_19769_amd import synth
from ttkv_testlib import Pair, assert_close, dev

pytestmark = pytest.mark.gpu

FORMATS = [("i8", "i8"), ("i8", "i4"), ("i4", "i4"), ("i8", "i4c"), ("i4", "i4c")]


def check(kfmt, vfmt, Hq, Hkv, lens, split, scale_q=1.0, softmax=None, mem="device", dtype="f16", paged=None):
    tiers = [dict(k_fmt=dtype, v_fmt=dtype, capacity=64, block_tokens=64, ring_blocks=3),
             dict(k_fmt=kfmt, v_fmt=vfmt, capacity=10**9, block_tokens=128, ring_blocks=max(lens) // 128 + 2, mem=mem, paged_seed=paged)]
    p = Pair(len(lens), Hq, Hkv, tiers, dtype, host_append_direct=True)
    try:
        B.ttkv_set_split(p.gpu.h, split)
        seed = synth.SEED_BASE + 800 + Hq * 7 + sum(lens)
        for b, n in enumerate(lens):
            k, v = synth.kv(seed * 3 + b, Hkv, n + 63, dtype)
            k[:, n:, 0] = -200.0          # the window's weights (rounded to 16 bits) are e^-70 of the others: what is
            p.load(b, synth.round_to(k / scale_q, dtype), v)     # compared comes from the quantized tier alone
        q = synth.normal(synth.rng(seed), (len(lens), Hq, 128), dtype)
        q[..., 0] = 4.0
        q = synth.round_to(q * scale_q, dtype)
        out, lse = p.gpu.decode(dev(q, dtype))
        torch.cuda.synchronize()
        ro, rl = p.ora.attend(q)
        got = out.cpu().numpy().astype(np.float64)
        assert_close(got, ro, "out")
        assert_close(lse.cpu().numpy(), rl, "lse")
        err = np.linalg.norm(got - ro, axis=(1, 2)) / np.linalg.norm(ro, axis=(1, 2))
        assert err.max() <= 2e-5, err
        assert p.gpu.stats()["mfma_launches"] > 0
    finally:
        p.close()


@pytest.mark.parametrize("G", [2, 3, 4, 5, 8, 9, 16, 17, 20])
@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
def test_heads_around_the_places(kfmt, vfmt, G):
    check(kfmt, vfmt, 2 * G, 2, [1536, 416], 0)


@pytest.mark.parametrize("G", [4, 8, 16])
@pytest.mark.parametrize("split", [1, 7, 4096])
@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
def test_lengths_around_a_batch(kfmt, vfmt, split, G):
    """Whole 32-token groups where the values are stored in them, odd lengths elsewhere; items from one per run (at most
    8192 tokens) to one per 256 tokens."""
    lens = [32, 64, 96, 288, 1120] if vfmt == "i4c" else [1, 31, 33, 63, 65, 127, 257, 1089]
    check(kfmt, vfmt, G, 1, lens, split, paged=3 if split == 7 else None)


@pytest.mark.parametrize("kfmt,vfmt", FORMATS)
def test_large_queries_and_bf16(kfmt, vfmt):
    """Queries up to 2e4 (int4 keys carry a factor 16 on them unless that leaves fp16's range), and bf16 ones."""
    check(kfmt, vfmt, 8, 2, [992], 0, scale_q=4096.0)
    check(kfmt, vfmt, 8, 2, [992], 0, dtype="bf16")
    check(kfmt, vfmt, 8, 2, [992], 0, mem="host")
