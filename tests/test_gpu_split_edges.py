"""Split keys where the choice of kernel and of the number of chunks changes: 31 and 32 key tiles, a pack whose chunks fill
the compute units exactly and one that no longer splits, both head dimensions, ragged lengths."""
import pytest
import torch

import paper_2604_04335_amd as da

pytestmark = pytest.mark.gpu


def _exact(q, k, v, cu, scale):
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
    for a, b in zip(cu[:-1], cu[1:]):
        for h in range(q.shape[1]):
            kt, vh = k[a:b, h].double().t().contiguous(), v[a:b, h].double()
            for r in range(a, b, 4096):
                e = min(b, r + 4096)
                s = (q[r:e, h].double() @ kt) * scale
                lse[r:e, h] = torch.logsumexp(s, 1)
                out[r:e, h] = torch.exp(s - lse[r:e, h, None]) @ vh
    return out, lse


@pytest.mark.parametrize("lens,H,D,max_splits,split", [
    ([4951], 3, 128, 8, True),         # 60 items of 256 rows: four chunks, ping-pong kernel
    ([1984], 3, 128, 8, True),         # 31 key tiles: three chunks, 128-row kernel
    ([1985], 3, 64, 8, True),          # 32 key tiles: four chunks, ping-pong kernel, the last of them one key longer
    ([8192, 8129], 2, 64, 2, True),    # 128 items of 256 rows: two chunks fill 256 compute units
    ([8193, 8192], 2, 128, 8, False),  # 130 items: no split
    ([1535], 2, 128, 8, True),         # 24 tiles: three chunks of eight
    ([1472], 2, 128, 2, False),        # 23 tiles: two chunks take eleven tiles off an item, too few
])
def test_split_choice(lens, H, D, max_splits, split):
    print(f"split edges: lens={lens} H={H} D={D} max_splits={max_splits}", flush=True)
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    gen = torch.Generator(device="cuda").manual_seed(sum(lens))
    q, k, v = (torch.randn((cu[-1], H, D), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
    scale, stream = D ** -0.5, torch.cuda.current_stream().cuda_stream
    ctx = da.dit_attn_create(0)
    try:
        base, out = torch.empty_like(q), torch.full_like(q, float("nan"))
        lse = torch.full((cu[-1], H), float("nan"), device="cuda")
        da.dit_attn_varlen_fwd(ctx, q, k, v, cu, H, D, scale, base, stream)
        da.dit_attn_set_split_kv(ctx, max_splits)
        da.dit_attn_varlen_fwd_lse(ctx, q, k, v, cu, H, D, scale, out, lse, stream)
        torch.cuda.synchronize()
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert torch.equal(base.view(torch.int16), out.view(torch.int16)) != split
        ref, ref_lse = _exact(q, k, v, cu, scale)
        # the parity bar of the benchmark definition, and the log-sum-exp's ln(1 + 2^-8) of the rounded probabilities
        assert float((out.double() - ref).norm() / ref.norm()) <= 1e-2 and float((out.double() - ref).abs().max()) <= 2e-2
        assert float((lse.double() - ref_lse).abs().max()) <= 4e-3
    finally:
        da.dit_attn_destroy(ctx)
