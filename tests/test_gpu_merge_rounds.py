"""The merge over more parts than its first loads ask for: both widths on either side of the lines between them (192 parts, 256 rows), and
rows that have fewer parts than the launch was told, down to none."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B
from test_gpu_workspaces import zeros_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [7, 300])
@pytest.mark.parametrize("n_parts", [65, 128, 129, 191, 192, 193, 513])
def test_rows_of_unequal_parts_against_float64(n_parts, rows):
    """Tolerance as for equal rows (test_gpu_merge_widths): 1e-5 covers the sums of n products below 4 whose weights sum to one,
    and the exponentials."""
    g = np.random.default_rng(n_parts + rows)
    m = g.standard_normal((rows, n_parts)).astype(np.float32) * 3
    l = (g.random((rows, n_parts)) + 0.5).astype(np.float32)
    acc = g.standard_normal((rows, n_parts, 128)).astype(np.float32) * l[..., None]
    cnt = g.integers(0, n_parts + 1, rows).astype(np.int32)
    cnt[:7] = (n_parts, 0, 1, 64, 65, n_parts - 1, min(n_parts, 128))
    beyond = np.arange(n_parts) >= cnt[:, None]
    acc[beyond] = np.nan                       # never part of a sum
    m[beyond] = 1e30
    tm, tl, ta, tc = (torch.from_numpy(x).cuda() for x in (m, l, acc, cnt))
    out = torch.full((rows, 128), 7.0, device="cuda:0")
    lse = torch.full((rows,), 7.0, device="cuda:0")
    h = B.ttkv_create()
    try:
        B.ttkv_merge_partials(h, tm, tl, ta, n_parts, n_parts, tc, rows, out, lse, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        B.ttkv_destroy(h)
    w = np.where(beyond, 0.0, np.exp(np.where(beyond, 0.0, m.astype(np.float64))))
    den = (w * l).sum(1)
    want = np.einsum("rp,rpd->rd", w, np.where(beyond[..., None], 0.0, acc)) / np.where(den > 0, den, 1.0)[:, None]
    assert np.max(np.abs(out.cpu().numpy() - want)) <= 1e-5
    got = lse.cpu().numpy()
    assert np.all(np.isneginf(got[cnt == 0]))
    assert np.max(np.abs(got[cnt > 0] - np.log(den[cnt > 0]))) <= 1e-5


def test_a_token_joins_many_parts_of_many_rows():
    """320 rows of 79 parts take 256 threads each: the same step as with 16 parts a row, up to the rounding of
    sums of 20000 terms in fp32 (the weights are exact to 22 bits), and the same row stored."""
    c = zeros_cache(8, 40, 2, [("f16", "f16", 128, 20000)], False)
    try:
        g = torch.Generator(device="cuda:0").manual_seed(21)
        c.len[0][:] = 0
        k, v = (torch.randn(8, 2, 20000, 128, generator=g, device="cuda:0").half() for _ in range(2))
        c.append(0, k, v)
        q = torch.randn(8, 40, 128, generator=g, device="cuda:0").half()
        kn, vn = (torch.randn(8, 2, 1, 128, generator=g, device="cuda:0").half() for _ in range(2))
        B.ttkv_set_split(c.h, 256)
        ref, ref_lse = (x.clone() for x in c.decode(q, new=(kn, vn)))
        row = c.dump_tier(0, 5)
        assert B.ttkv_count_parts(c.h, c.c) <= 32          # 128 threads a row
        c.len[0] -= 1
        B.ttkv_set_split(c.h, 1 << 16)
        assert B.ttkv_count_parts(c.h, c.c) == 79
        c._parts_age = None
        out, lse = c.decode(q, new=(kn, vn))
        torch.cuda.synchronize()
        assert float((out - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
        assert torch.allclose(lse, ref_lse, atol=1e-5)
        again = c.dump_tier(0, 5)
        assert np.array_equal(row["k"], again["k"]) and np.array_equal(row["v"], again["v"])
    finally:
        c.close()
