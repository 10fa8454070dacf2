"""The 128-row kernel's tile loop at every number of key tiles where its parts meet (first step, main loop, last steps, both
ring depths), against the ping-pong kernel bit for bit and against attention in float64."""
import pytest
import torch

import paper_2604_04335_amd as da

pytestmark = pytest.mark.gpu

# 128 rows (one workgroup on its compute unit: the deep ring from 16 tiles on at head dimension 128) against 1 to 23 tiles,
# whole and ragged, and around 12 and 19 tiles on a chip that is more than half full (loads at the start of a step).
TILES = [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 18, 19, 20, 21, 22, 23]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("ragged", [0, 1, 63])
@pytest.mark.parametrize("heads", [1, 130])
def test_numbers_of_key_tiles(head_dim, ragged, heads):
    ctx, stream = da.dit_attn_create(0), torch.cuda.current_stream().cuda_stream
    try:
        for tiles in TILES if heads == 1 else [11, 12, 13, 18, 19, 20, 21, 30]:
            n_keys = 64 * tiles - ragged
            print(f"D={head_dim} heads={heads} keys={n_keys}", flush=True)
            gen = torch.Generator(device="cuda").manual_seed(n_keys)
            q = torch.randn((128, heads, head_dim), device="cuda", generator=gen).to(torch.bfloat16)
            k, v = (torch.randn((n_keys, heads, head_dim), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
            outs, lses = [], []
            for kernel in (da.KERNEL_128, da.KERNEL_PINGPONG):
                da.dit_attn_set_kernel(ctx, kernel)
                outs.append(torch.full_like(q, float("nan")))
                lses.append(torch.full((128, heads), float("nan"), device="cuda"))
                da.dit_attn_cross_varlen_fwd(ctx, q, k, v, [0, 128], [0, n_keys], heads, head_dim, head_dim ** -0.5, outs[-1], lses[-1], stream)
            torch.cuda.synchronize()
            assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16)) and torch.equal(lses[0], lses[1])
            s = torch.stack([q[:, h].double() @ k[:, h].double().t().contiguous() for h in range(heads)]) * head_dim ** -0.5
            ref = torch.stack([torch.softmax(s[h], -1) @ v[:, h].double() for h in range(heads)], 1)
            # the parity bar of the benchmark definition (rounding of P and of the output to bf16: about 2e-3)
            assert float((outs[0].double() - ref).norm() / ref.norm()) <= 1e-2
    finally:
        da.dit_attn_destroy(ctx)
