"""Split keys where the choice of kernel and of the number of chunks changes: 63 and 64, 127 and 128 key tiles, packs whose
chunks fill the compute units exactly and ones that no longer split, the fewest tiles that a split has to take off an item, a
short last chunk; both head dimensions, ragged lengths.  The number of chunks and the kernel are checked, and two calls' bits."""
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


@pytest.mark.parametrize("lens,H,D,max_splits,chunks,kernel", [
    ([4951], 3, 128, 8, 4, da.KERNEL_PINGPONG),         # 60 items of 256 rows: four chunks in one round
    ([1984], 3, 128, 8, 3, da.KERNEL_128),              # 31 key tiles
    ([1985], 3, 64, 8, 4, da.KERNEL_128),               # 32 key tiles, the last chunk 63 keys shorter than the others
    ([4032], 3, 128, 8, 2, da.KERNEL_128),              # 63 tiles, 96 items of 128 rows: two chunks in one round
    ([4033], 3, 128, 8, 5, da.KERNEL_PINGPONG),         # 64 tiles, 48 items of 256 rows
    ([2048], 8, 64, 8, 2, da.KERNEL_128),               # 128 items of 128 rows, two for every compute unit
    ([2049], 8, 64, 8, 1, None),                        # 136: no room for another round of them
    ([8192, 8129], 2, 64, 2, 2, da.KERNEL_PINGPONG),    # 256 of them, 128 tiles: two chunks fill 256 compute units
    ([8128, 8127], 2, 64, 8, 1, None),                  # 127 tiles
    ([8193, 8192], 2, 128, 8, 1, None),                 # 130 items of 256 rows: no split
    ([1535], 2, 128, 8, 3, da.KERNEL_128),              # 24 tiles: three chunks of eight
    ([1472], 2, 128, 2, 1, None),                       # 23 tiles: two chunks take eleven tiles off an item, too few
    ([1536], 5, 128, 2, 2, da.KERNEL_128),              # 24: twelve
    ([1536], 5, 64, 2, 1, None),                        # which are too few at head dimension 64
    ([1601], 5, 64, 2, 2, da.KERNEL_128),               # 26: thirteen
    ([2112], 14, 64, 8, 1, None),
    ([2176], 14, 64, 8, 1, None),                       # 238 items of 128 rows: 23.3 us, two chunks of 256-row items 27.8
    ([2304], 14, 128, 8, 1, None),                      # 39.5 us and 46.4
    ([4160, 4480], 1, 128, 8, 7, da.KERNEL_PINGPONG),   # 35 items; 65 tiles in seven chunks: 10 each, the last 5
])
def test_split_choice(lens, H, D, max_splits, chunks, kernel):
    print(f"split edges: lens={lens} H={H} D={D} max_splits={max_splits}", flush=True)
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    gen = torch.Generator(device="cuda").manual_seed(sum(lens))
    q, k, v = (torch.randn((cu[-1], H, D), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
    scale, stream = D ** -0.5, torch.cuda.current_stream().cuda_stream
    ctx = da.dit_attn_create(0)
    try:
        def run(limit):
            out, lse = torch.full_like(q, float("nan")), torch.full((cu[-1], H), float("nan"), device="cuda")
            da.dit_attn_set_split_kv(ctx, limit)
            da.dit_attn_varlen_fwd_lse(ctx, q, k, v, cu, H, D, scale, out, lse, stream)
            return out, lse

        out, lse = run(max_splits)
        used = da.dit_attn_last_launch_kernel(ctx)
        again, same, base = run(max_splits)[0], run(chunks)[0], run(1)[0]
        fewer = run(chunks - 1)[0] if chunks > 1 else None
        torch.cuda.synchronize()
        bits = lambda x: x.view(torch.int16)
        assert torch.equal(bits(out), bits(again))
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            # The bits depend on the number of chunks alone: as many as this limit allows, more than one less would.
            assert torch.equal(bits(out), bits(same)) and torch.equal(bits(out), bits(base)) == (chunks == 1)
            assert fewer is None or not torch.equal(bits(out), bits(fewer))
            assert kernel is None or used == kernel
        ref, ref_lse = _exact(q, k, v, cu, scale)
        # the parity bar of the benchmark definition, and the log-sum-exp's ln(1 + 2^-8) of the rounded probabilities
        assert float((out.double() - ref).norm() / ref.norm()) <= 1e-2 and float((out.double() - ref).abs().max()) <= 2e-2
        assert float((lse.double() - ref_lse).abs().max()) <= 4e-3
    finally:
        da.dit_attn_destroy(ctx)
