"""Which kernel a pack gets, seen through dit_attn_plan's block_m (128 or 256 query rows per item) on a 256-CU device."""
import numpy as np
import pytest

import paper_2604_04335_amd as da


@pytest.mark.parametrize("lens,heads,head_dim,block_m", [
    ([1280], 24, 64, 128),           # 240 items of 128 rows: each has a compute unit of its own
    ([1281], 24, 64, 256),           # 264 of them, 144 items of 256 rows in one round
    ([700] * 4, 12, 64, 256),
    ([410] * 8, 24, 64, 128),        # several rounds of short items
    ([2049] * 6, 24, 64, 256),       # 33 key tiles: long items
    ([2048] * 6, 24, 64, 128),       # 32
    ([4250, 410], 13, 64, 256),      # 247 items, one round
    ([2458, 410], 24, 128, 256),     # 288 items whose second round is made of short ones: no longer than the longest item
    ([2458, 2458], 14, 128, 128),    # 280 equal items: a second round that is nearly empty
    ([2458, 0], 24, 128, 256),
])
def test_kernel_choice(lens, heads, head_dim, block_m):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    assert da.dit_attn_plan(cu, heads, head_dim)[1] == block_m
