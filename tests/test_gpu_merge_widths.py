"""The merge kernel's two widths and its batches of parts, and arrays that start at any float."""
import numpy as np
import pytest
import torch

from paper_2604_19769_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_parts", [1, 31, 32, 33, 64, 65, 255, 256, 257, 600])
@pytest.mark.parametrize("shift", [0, 1])
def test_merge_against_float64(n_parts, shift):
    """Tolerance: n fp32 products and sums of values below 4 on weights that sum to one: a few hundred ulp of 1 at most,
    and the exponentials' own error (2 ulp) -- 1e-5 covers both."""
    rows, stride = 3, n_parts + 2
    g = np.random.default_rng(n_parts)
    m = g.standard_normal((rows, stride)).astype(np.float32) * 3
    l = (g.random((rows, stride)) + 0.5).astype(np.float32)
    acc = g.standard_normal((rows, stride, 128)).astype(np.float32)
    if n_parts > 2:
        m[1, 1] = -np.inf                      # an empty part
    acc *= l[..., None]
    buf = torch.zeros(acc.size + 8, dtype=torch.float32, device="cuda:0")
    ta = buf[shift:shift + acc.size]
    ta.copy_(torch.from_numpy(acc.ravel()))
    tm, tl = (torch.from_numpy(x).cuda() for x in (m, l))
    out = torch.empty(rows, 128, device="cuda:0")
    lse = torch.empty(rows, device="cuda:0")
    h = B.ttkv_create()
    try:
        B.ttkv_merge_partials(h, tm, tl, ta, n_parts, stride, None, rows, out, lse, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        B.ttkv_destroy(h)
    m64, l64, a64 = (x[:, :n_parts].astype(np.float64) for x in (m, l, acc))
    M = m64.max(1, keepdims=True)
    w = np.exp(m64 - M)
    den = (w * l64).sum(1)
    want = (w[..., None] * a64).sum(1) / den[:, None]
    assert np.max(np.abs(out.cpu().numpy() - want)) <= 1e-5
    assert np.max(np.abs(lse.cpu().numpy() - (M[:, 0] + np.log(den)))) <= 1e-5
