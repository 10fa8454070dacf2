"""The merge kernel at the edges of its chunks per thread and of the lines from which the parts are read with streaming
loads and the output is written with streaming stores."""
import pytest
import torch

import paper_2604_04335_amd as da

pytestmark = pytest.mark.gpu


def _parts(n_parts, T, H, D, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    o = [torch.randn((T, H, D), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(n_parts)]
    lse = [8.0 + torch.randn((T, H), device="cuda", generator=gen) for _ in range(n_parts)]
    lse[0][::3] = float("-inf")
    return o, lse


def _merge(o, lse):
    T, H, D = o[0].shape
    ctx = da.dit_attn_create(0)
    try:
        buf = torch.full((T * H * D + 128,), 0x7FC1, dtype=torch.int16, device="cuda")
        out, l = buf[64:-64].view(torch.bfloat16).view(T, H, D), torch.full((T, H), float("nan"), device="cuda")
        da.dit_attn_merge(ctx, o, lse, T, H, D, out, l, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert bool((buf[:64] == 0x7FC1).all()) and bool((buf[-64:] == 0x7FC1).all())
        return out, l
    finally:
        da.dit_attn_destroy(ctx)


@pytest.mark.parametrize("D,T,H", [(64, 1, 1), (64, 63, 1), (64, 65, 1), (128, 31, 1), (128, 33, 1), (128, 64, 1), (128, 21, 3)])
@pytest.mark.parametrize("n_parts", [2, 4, 8])
def test_chunks_per_thread(n_parts, D, T, H):
    """Eight chunks in all up to a few workgroups and a remainder of one row."""
    print(f"merge edges: parts={n_parts} T={T} H={H} D={D}", flush=True)
    o, lse = _parts(n_parts, T, H, D, 7 * T + D)
    out, l = _merge(o, lse)
    total = torch.logsumexp(torch.stack(lse).double(), 0)
    ref = sum(torch.exp(x.double() - total)[..., None] * y.double() for x, y in zip(lse, o))
    # the output's rounding to bf16 (2^-9 relative to the element) and fp32 arithmetic far below it
    assert bool(((out.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5).all())
    assert float((l.double() - total).abs().max()) <= 1e-5


@pytest.mark.parametrize("n_parts,line", [(2, "loads"), (4, "loads"), (8, "loads"), (2, "stores"), (4, "stores"), (5, "stores"), (6, "stores")])
def test_either_side_of_the_streaming_lines(n_parts, line):
    """96 MiB of parts and output; 400 MiB of parts and 80 MiB of output: the last row count below and the first above give the
    same bits on the rows they share (and 24 heads leave a remainder of the chunks per thread on one side of each line)."""
    H, D = 24, 128
    T = -(-(96 << 20) // ((n_parts + 1) * H * D * 2)) if line == "loads" else -(-(400 << 20) // (min(n_parts, 5) * H * D * 2))
    print(f"merge streaming {line}: parts={n_parts} T={T}", flush=True)
    o, lse = _parts(n_parts, T, H, D, n_parts)
    above, l_above = _merge(o, lse)
    below, l_below = _merge([x[:T - 1] for x in o], [x[:T - 1] for x in lse])
    assert torch.equal(above[:T - 1].view(torch.int16), below.view(torch.int16)) and torch.equal(l_above[:T - 1], l_below)
    rows = torch.arange(T - 700, T, device="cuda")
    total = torch.logsumexp(torch.stack([x[rows] for x in lse]).double(), 0)
    ref = sum(torch.exp(x[rows].double() - total)[..., None] * y[rows].double() for x, y in zip(lse, o))
    # the output's rounding to bf16 and fp32 arithmetic, as above
    assert bool(((above[rows].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5).all())
    assert float((l_above[rows].double() - total).abs().max()) <= 1e-5


@pytest.mark.parametrize("n_parts,D,T", [(1, 128, 33), (2, 64, 65), (4, 128, 21), (8, 128, 257), (3, 128, 5000), (4, 128, 17500)])
def test_output_over_a_part(n_parts, D, T):
    """The output may be the memory of any part: the bits of a merge into memory of its own, in each form of the kernel."""
    H = 24
    print(f"merge in place: parts={n_parts} T={T} D={D}", flush=True)
    o, lse = _parts(n_parts, T, H, D, T)
    ref, l_ref = _merge(o, lse)
    ctx = da.dit_attn_create(0)
    try:
        for i in sorted({0, n_parts - 1}):
            mine, l = [x.clone() if j == i else x for j, x in enumerate(o)], torch.full((T, H), float("nan"), device="cuda")
            da.dit_attn_merge(ctx, mine, lse, T, H, D, mine[i], l, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert torch.equal(mine[i].view(torch.int16), ref.view(torch.int16)) and torch.equal(l, l_ref)
    finally:
        da.dit_attn_destroy(ctx)
