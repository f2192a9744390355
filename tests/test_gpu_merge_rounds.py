"""The merge over more parts than its first loads ask for: both widths on either side of the lines between them (192 parts, 256 rows), and
rows that have fewer parts than the launch was told, down to none."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B

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
