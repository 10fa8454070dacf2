"""Work distribution at the edge of one round: packs with one item fewer than, as many as, and one or more items than there
are resident workgroups, several launches in a row (each leaves the work counter as the next one needs it), both kernels."""
import os
import sys

import pytest
import torch

import paper_2604_04335_amd as da

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
def test_items_around_one_round(head_dim):
    ctx = da.dit_attn_create(0)
    try:
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        stream = torch.cuda.current_stream().cuda_stream
        for slots, kernel, bm in ((cus, da.KERNEL_PINGPONG, 256), (2 * cus, da.KERNEL_128, 128), (3 * cus, da.KERNEL_128, 128)):
            for items in (slots - 1, slots, slots + 1, 2 * slots + 1):
                # one head, `items` sequences of a ragged tile each: every sequence is one work item of either kernel
                n_keys = bm - 59
                cu = [i * n_keys for i in range(items + 1)]
                gen = torch.Generator(device="cuda").manual_seed(items)
                q, k, v = (torch.randn((cu[-1], 1, head_dim), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
                # the same rows as a batch of one-sequence problems in fp32
                s = torch.bmm(q.float().view(items, n_keys, head_dim), k.float().view(items, n_keys, head_dim).transpose(1, 2).contiguous())
                ref = torch.bmm(torch.softmax(s * head_dim ** -0.5, -1), v.float().view(items, n_keys, head_dim)).view_as(q)
                print(f"D={head_dim} kernel={kernel} items={items}", flush=True)
                da.dit_attn_set_kernel(ctx, kernel)
                outs = [torch.full_like(q, float("nan")) for _ in range(3)]
                for out in outs:
                    da.dit_attn_varlen_fwd(ctx, q, k, v, cu, 1, head_dim, head_dim ** -0.5, out, stream)
                torch.cuda.synchronize()
                # the parity bar of the benchmark definition (rounding of P and of the output to bf16: about 2e-3)
                assert float((outs[0].float() - ref).norm() / ref.norm()) <= 1e-2
                assert all(torch.equal(outs[0].view(torch.int16), o.view(torch.int16)) for o in outs[1:])
    finally:
        da.dit_attn_destroy(ctx)
