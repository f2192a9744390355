"""Launches whose run table is nearly or more than full (208 runs): 64 sequences in two, three and four tiers."""
import pytest

from paper_2604_19769_amd import synth
from test_gpu_parity import run_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,n_tiers", [(4, 2, 2), (4, 2, 3), (2, 2, 3), (4, 2, 4)])
def test_maximum_batch_in_several_tiers(Hq, Hkv, n_tiers):
    tiers = [dict(k_fmt="f16", v_fmt="f16", capacity=128, block_tokens=64, ring_blocks=4),
             dict(k_fmt="i8", v_fmt="i8", capacity=128, block_tokens=64, ring_blocks=4),
             dict(k_fmt="i8", v_fmt="i4", capacity=128, block_tokens=128, ring_blocks=4, paged_seed=3),
             dict(k_fmt="i4", v_fmt="i4", capacity=10**9, block_tokens=64, ring_blocks=12)][:n_tiers]
    tiers[-1] = dict(tiers[-1], capacity=10**9, ring_blocks=12)
    st = run_config(64, Hq, Hkv, tiers, "f16", None, 2, synth.SEED_BASE + 61, lens=[520 + 3 * b for b in range(64)], want_stats=True)
    if Hq > Hkv:   # two steps, one launch each while 208 runs hold them; the first eviction empties the third of four tiers
        assert st["mfma_launches"] == (2 if n_tiers <= 3 else 2 + 1), st
