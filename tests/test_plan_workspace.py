"""Items of 128 tokens (launches that leave CUs idle) are twice the partials of 256-token ones, and a cache one token longer
may be beyond them: they are taken only where the workspace holds their partials, so that a workspace sized for the longer
cache stays large enough.  Host arithmetic: the top-k step checks its plan against the workspace before anything else, and
here it is refused after that, for more live blocks than it ranks; nothing is enqueued."""
import ctypes as C

import numpy as np
import pytest

from paper_2604_19769_amd import binding as B
from test_abi import plan_cache


@pytest.mark.parametrize("heads,selected", [((8, 2), 200), ((16, 4), 100), ((64, 4), 100), ((8, 1), 400)])
def test_a_workspace_for_256_token_items_is_taken(heads, selected):
    """512 fp16 tokens and `selected` blocks of 64 int8 tokens: that many items of 128 tokens, at most 256 workgroups."""
    c = plan_cache(1, *heads, [("f16", "f16", 128, 512), ("i8", "i8", 64, 64 * 1500)])
    z = np.zeros(64, np.uint8)
    c.tier[1].k_sum = c.tier[1].k_summary = z.ctypes.data
    p, h = C.c_void_p(z.ctypes.data), B.ttkv_create()

    def step(parts):
        ws = parts * heads[0] * 130 * 4                  # at a 256-byte address: room for exactly so many parts per row
        return B.lib().ttkv_decode_step_topk(h, C.byref(c), p, B.F16, p, p, B.F16, p, None, selected, None, None, selected, p, 1 << 20,
                                             C.c_void_p(4096), ws, None)

    try:
        coarse = 512 // 256 + selected * 64 // 256
        assert (512 // 128 + selected * 64 // 128) * heads[1] <= 256
        for parts in (coarse, coarse + 16, 2 * coarse - 1, 2 * coarse):
            assert step(parts) == B.ERR_UNSUPPORTED, parts
        assert step(coarse - 1) == B.ERR_WORKSPACE       # and no smaller one
        B.ttkv_set_split(h, 1 << 20)                     # a split that was asked for stays as it is
        assert step(coarse) == B.ERR_UNSUPPORTED and step(coarse - 1) == B.ERR_WORKSPACE
    finally:
        B.ttkv_destroy(h)
