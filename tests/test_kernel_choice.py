"""Which kernel a pack gets, seen through dit_attn_plan's block_m (128 or 256 query rows per item) on a 256-CU device."""
import numpy as np
import pytest

import paper_2604_04335_amd as da


@pytest.mark.parametrize("lens,heads,head_dim,block_m", [
    ([1280], 24, 64, 128),           # 240 items of 128 rows: each has a compute unit of its own
    ([1281], 24, 64, 256),           # 264 of them, 144 items of 256 rows in one round
    ([700] * 4, 12, 64, 256),
    ([410] * 8, 24, 64, 128),        # 768 items of 128 rows, three per compute unit
    ([2049] * 6, 24, 64, 128),       # 33 key tiles
    ([4352] * 4, 24, 64, 128),
    ([6400], 24, 64, 128),           # 100 key tiles
    ([6401], 24, 64, 128),           # 101: 283 us, the ping-pong kernel 298
    ([1054] * 4, 24, 64, 256),       # 864 items of 128 rows: a second round of 96 of them
    ([300] * 10, 24, 64, 128),       # 720: one round
    ([410] * 8 + [250], 24, 64, 256),      # 816, 408 items of 256 rows
    ([400] * 9, 24, 64, 256),        # 432 items of 256 rows with 200 rows each on average
    ([399] * 9, 24, 64, 128),
    ([1024] * 16, 8, 64, 256),       # 1024 items of 128 rows, 512 of 256: two full rounds
    ([1024] * 16 + [30], 8, 64, 128),      # 520: a third round
    ([1088] * 4, 24, 64, 256),       # 17 key tiles, 864 items of 128 rows
    ([1089] * 4, 24, 64, 128),       # 18
    ([1536] * 3, 24, 64, 128),       # 24: 55 us, the ping-pong kernel 57
    ([1537] * 3, 24, 64, 128),       # 25
    ([2458] * 4, 24, 64, 128),       # 960 items of 256 rows, a fourth round three quarters full: 164 us, 174
    ([2458] * 3 + [2304], 24, 64, 128),    # 936
    ([4096] * 8, 8, 64, 128),        # 1024, four full rounds: 278 us, 284
    ([4096] * 8 + [30], 8, 64, 128),       # 1032
    ([4250, 410], 13, 64, 256),      # 247 items, one round
    ([2458, 410], 24, 128, 256),     # 288 items whose second round is made of short ones: no longer than the longest item
    ([2458, 2458], 14, 128, 128),    # 280 equal items: a second round that is nearly empty
    ([2458, 0], 24, 128, 256),
])
def test_kernel_choice(lens, heads, head_dim, block_m):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    assert da.dit_attn_plan(cu, heads, head_dim)[1] == block_m


@pytest.mark.gpu
@pytest.mark.parametrize("n_keys,kernel", [(64, "PINGPONG"), (128, "PINGPONG"), (129, "128"), (320, "128"), (512, "128")])
def test_cross_choice_at_head_dim_64(n_keys, kernel):
    """One and two key tiles run the ping-pong kernel, more the 128-row kernel; either gives the bits of the other."""
    import torch
    print(f"cross choice: {n_keys} keys", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n_keys)
    q, k, v = (torch.randn((n, 24, 64), device="cuda", generator=gen).to(torch.bfloat16) for n in (5000, 2 * n_keys, 2 * n_keys))
    ctx, stream = da.dit_attn_create(0), torch.cuda.current_stream().cuda_stream
    try:
        outs = []
        for forced in (da.KERNEL_AUTO, da.KERNEL_128, da.KERNEL_PINGPONG):
            da.dit_attn_set_kernel(ctx, forced)
            outs.append(torch.full_like(q, float("nan")))
            da.dit_attn_cross_varlen_fwd(ctx, q, k, v, [0, 2600, 5000], [0, n_keys, 2 * n_keys], 24, 64, 0.125, outs[-1], None, stream)
            if forced == da.KERNEL_AUTO and torch.cuda.get_device_properties(0).multi_processor_count == 256:
                assert da.dit_attn_last_launch_kernel(ctx) == getattr(da, "KERNEL_" + kernel)
        torch.cuda.synchronize()
        assert not bool(outs[0].isnan().any())
        assert all(torch.equal(outs[0].view(torch.int16), o.view(torch.int16)) for o in outs[1:])
    finally:
        da.dit_attn_destroy(ctx)


@pytest.mark.parametrize("lens,heads,head_dim,block_m", [
    ([1280], 24, 128, 128),          # 240 items of 128 rows: each has a compute unit of its own
    ([1281], 24, 128, 256),          # 264 items of 128 rows
    ([2048], 15, 128, 128),
    ([2048], 16, 128, 128),          # 256 of them, each with a compute unit of its own: 36 us, the ping-pong kernel 44
    ([2048], 17, 128, 256),
    ([2100], 15, 128, 128),          # 255, although 135 items of 256 rows are more than half of the compute units
    ([200] * 16, 8, 128, 128),       # 256 ragged ones
    ([3600], 24, 128, 128),          # 360: a second round 41 % full
    ([3841], 23, 128, 128),          # 368, 44 %: 161 us, the ping-pong kernel 178
    ([4096], 24, 128, 128),          # 384: half full
    ([4097], 23, 128, 256),          # 391
    ([1152] * 4, 19, 128, 256),      # 380 items of 18 key tiles
    ([1153] * 4, 19, 128, 128),      # 19
    ([1152] * 4, 14, 128, 128),      # 504 items of 128 rows: one round of two on every compute unit
    ([700] * 10, 12, 128, 128),      # 360 of 11 key tiles: at most three sevenths
    ([700] * 10, 13, 128, 256),      # 390
    ([705] * 10, 12, 128, 256),      # 12
    ([6000], 24, 128, 128),          # 576 equal items: a third round a quarter full
    ([6000], 25, 128, 128),          # 600: 413 us, the ping-pong kernel 431
    ([4096], 40, 128, 128),          # 640: half full
    ([4097], 38, 128, 256),          # 646
    ([6000, 3000], 17, 128, 256),    # 612 items of two lengths: the short ones fill the round
    ([8128], 24, 64, 128),           # 127 key tiles: 395 us, the ping-pong kernel 416
    ([8129], 24, 64, 128),           # 128
])
def test_kernel_choice_of_fuller_rounds(lens, heads, head_dim, block_m):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    assert da.dit_attn_plan(cu, heads, head_dim)[1] == block_m


@pytest.mark.gpu
@pytest.mark.parametrize("n_keys,kernel", [(64, "128"), (448, "128"), (704, "128"), (705, "PINGPONG")])
def test_cross_choice_at_head_dim_128(n_keys, kernel):
    """Up to eleven key tiles run the 128-row kernel, more the ping-pong kernel; either gives the bits of the other."""
    import torch
    print(f"cross choice: {n_keys} keys", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n_keys)
    q, k, v = (torch.randn((n, 24, 128), device="cuda", generator=gen).to(torch.bfloat16) for n in (5000, 2 * n_keys, 2 * n_keys))
    ctx, stream = da.dit_attn_create(0), torch.cuda.current_stream().cuda_stream
    try:
        outs = []
        for forced in (da.KERNEL_AUTO, da.KERNEL_128, da.KERNEL_PINGPONG):
            da.dit_attn_set_kernel(ctx, forced)
            outs.append(torch.full_like(q, float("nan")))
            da.dit_attn_cross_varlen_fwd(ctx, q, k, v, [0, 2600, 5000], [0, n_keys, 2 * n_keys], 24, 128, 0.09, outs[-1], None, stream)
            if forced == da.KERNEL_AUTO and torch.cuda.get_device_properties(0).multi_processor_count == 256:
                assert da.dit_attn_last_launch_kernel(ctx) == getattr(da, "KERNEL_" + kernel)
        torch.cuda.synchronize()
        assert not bool(outs[0].isnan().any())
        assert all(torch.equal(outs[0].view(torch.int16), o.view(torch.int16)) for o in outs[1:])
    finally:
        da.dit_attn_destroy(ctx)
