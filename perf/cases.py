"""The attention work that a serving loop hands to this library, as cases that can be timed and compared.

A case is a dict of plain values: the operation, the sequence lengths as text ("4352*4 20506" is four sequences of
4352 tokens and one of 20506), heads, head dimension and the options of the call.  `prepare` makes what the loop holds
before the call (tensors on the GPU, the context), `run` is the call as the loop makes it, `work` the bytes and
operations that the operation cannot do without.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2604_04335_amd as da


def _lens(text: str) -> list:
    """"4352*4 20506" -> [4352, 4352, 4352, 4352, 20506]."""
    out = []
    for part in text.split():
        length, _, times = part.partition("*")
        out += [int(length)] * int(times or 1)
    return out


def _text(lens) -> str:
    return " ".join(str(n) for n in lens)


def listed() -> list:
    return [
        # One low-resolution image (256 latent + 154 text tokens): the smallest denoising step that is served, where the
        # launch and the length of one work item count.
        dict(name="image_small", op="self", entry="plain", q_lens="410", heads=24, head_dim=64, splits=1, head_scale=False),
        # The benchmark's tiny image step.
        dict(name="tiny_image", op="self", entry="plain", q_lens="1024", heads=8, head_dim=64, splits=1, head_scale=False),
        # One low-resolution video step (1344 latent + 226 text tokens) through the entry point that allocates nothing, as a
        # loop calls it that may not call hipMalloc when a pack is new.
        dict(name="video_small", op="self", entry="noalloc", q_lens="1570", heads=24, head_dim=128, splits=1, head_scale=False),
        # One GPU's three of 24 heads of a medium video (4725 latent + 226 text tokens, head split over eight GPUs), with
        # the split of the keys switched on for latency.
        dict(name="shard_split_kv", op="self", entry="plain", q_lens="4951", heads=3, head_dim=128, splits=8, head_scale=False),
        # Dynamic batch of images of several resolutions at head dimension 64, ragged lengths.
        dict(name="image_batch_d64", op="self", entry="plain", q_lens="2458*2 1054*3 410 4250*2", heads=24, head_dim=64,
             splits=1, head_scale=True),
        # The benchmark's batch of four 1024x1024 images, per-head value scale.
        dict(name="t2i_batch", op="self", entry="plain", q_lens="4352*4", heads=24, head_dim=128, splits=1, head_scale=True),
        # The benchmark's headline: images batched with a video, in its shuffled order.
        dict(name="mixed_varlen", op="self", entry="plain", q_lens="4352*2 1280 20506 4352*2 1280 4352*2", heads=24,
             head_dim=128, splits=1, head_scale=False),
        # The benchmark's sequence-parallel shard: 10 of 40 heads over a long video.  The largest call.
        dict(name="sp_shard", op="self", entry="plain", q_lens="76112", heads=10, head_dim=128, splits=1, head_scale=False),
        # Ring step of sequence parallelism: one GPU's quarter of that sequence against another GPU's quarter, with the
        # log-sum-exp that the merge needs.
        dict(name="ring_step", op="cross", entry="lse", q_lens="19028", k_lens="19028", heads=40, head_dim=128, splits=1,
             head_scale=False),
        # Cross-attention of image and video latents against 512 text keys each.
        dict(name="cross_text", op="cross", entry="plain", q_lens="4352*6 20506", k_lens="512*7", heads=24, head_dim=128,
             splits=1, head_scale=False),
        # Merge of the four partial results of a ring over the rows of mixed_varlen.
        dict(name="merge_parts", op="merge", parts=4, rows=49178, heads=24, head_dim=128),
        # Both layout changes around the head-split all-to-all of a quarter of the long video.
        dict(name="sp_exchange", op="exchange", rows=19028, heads=40, head_dim=128, degree=4),
    ]


MAX_FLOPS = 2.9e13  # under the largest listed case (sp_shard, 2.966e13)


def _log_int(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    """One more case: any of the operations, sizes over the range of the listed ones."""
    while True:
        kind = rng.choice(["image", "image", "video", "mixed", "shard", "shard", "cross", "cross", "ring", "merge", "exchange"])
        case = _draw_kind(rng, kind)
        if work(case)["flops"] <= MAX_FLOPS:
            return case


def _draw_kind(rng, kind: str) -> dict:
    image = lambda: _log_int(rng, 256, 4096) + rng.choice([0, 64, 154, 256])  # latent tokens and text tokens
    video = lambda lo=1344, hi=20280: _log_int(rng, lo, hi) + rng.choice([0, 226])
    base = dict(op="self", entry="plain", splits=1, head_scale=rng.random() < 0.3)
    if kind == "image":
        lens = [image() for _ in range(rng.randint(1, 8))] if rng.random() < 0.5 else [image()] * rng.randint(1, 8)
        return dict(base, q_lens=_text(lens), heads=rng.choice([8, 12, 24]), head_dim=rng.choice([64, 128]),
                    entry=rng.choice(["plain", "plain", "noalloc"]))
    if kind == "video":
        return dict(base, q_lens=_text([video()]), heads=24, head_dim=128, entry=rng.choice(["plain", "plain", "noalloc"]))
    if kind == "mixed":
        lens = [image() for _ in range(rng.randint(1, 8))] + [video()]
        rng.shuffle(lens)
        return dict(base, q_lens=_text(lens), heads=24, head_dim=128)
    if kind == "shard":  # a head split over 2, 4 or 8 GPUs
        return dict(base, q_lens=_text([video(1344, 75600)]), heads=rng.choice([3, 5, 6, 10, 12, 20]), head_dim=128,
                    splits=rng.choice([1, 8]), entry=rng.choice(["plain", "lse"]))
    if kind == "cross":
        lens = [rng.choice([image, video])() for _ in range(rng.randint(1, 7))]
        keys = [rng.randint(64, 512) for _ in lens] if rng.random() < 0.5 else [rng.choice([77, 226, 512])] * len(lens)
        return dict(base, op="cross", q_lens=_text(lens), k_lens=_text(keys), heads=24, head_dim=rng.choice([64, 128, 128]))
    if kind == "ring":
        n = _log_int(rng, 1024, 19028)
        return dict(base, op="cross", q_lens=_text([n]), k_lens=_text([max(1, n - rng.choice([0, 1, 77]))]),
                    heads=rng.choice([10, 24, 40]), head_dim=128, entry="lse")
    if kind == "merge":
        return dict(op="merge", parts=rng.randint(2, 8), rows=_log_int(rng, 256, 32768), heads=rng.choice([8, 10, 24]),
                    head_dim=rng.choice([64, 128]))
    degree = rng.choice([2, 4, 8])
    return dict(op="exchange", rows=_log_int(rng, 256, 19028), heads=rng.choice([24, 40]), head_dim=rng.choice([64, 128]),
                degree=degree)


@functools.lru_cache(maxsize=None)
def _context(max_splits: int) -> int:
    """The context a program creates once and keeps (one per setting of the split)."""
    ctx = da.dit_attn_create(torch.cuda.current_device())
    da.dit_attn_set_split_kv(ctx, max_splits)
    return ctx


def _cu(lens) -> np.ndarray:
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


def _inputs(case: dict, seed: int) -> dict:
    """The tensors that a call reads, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    H, D = case["heads"], case["head_dim"]

    def noise(*shape, scale=None):
        x = torch.randn(shape, device="cuda", generator=gen)
        return (x if scale is None else x * scale).to(torch.bfloat16)

    if case["op"] == "merge":
        T, P = case["rows"], case["parts"]
        # log-sum-exp of a few thousand keys each: a common level of its own per part and row noise around it
        return dict(o_parts=[noise(T, H, D) for _ in range(P)],
                    lse_parts=[8.0 + torch.randn((T, H), device="cuda", generator=gen) for _ in range(P)])
    if case["op"] == "exchange":
        n, p = case["rows"], case["degree"]
        return dict(x=noise(n, H, D), received=noise(p, n, H // p, D))
    q_lens = _lens(case["q_lens"])
    k_lens = _lens(case["k_lens"]) if case["op"] == "cross" else q_lens
    # N(0, 1), or with a factor of 0.5 to 2 per head, which makes the logits of some heads peaky
    scale = 0.5 + 1.5 * torch.rand((H, 1), device="cuda", generator=gen) if case["head_scale"] else None
    q = noise(sum(q_lens), H, D, scale=scale)
    k, v = (noise(sum(k_lens), H, D, scale=scale) for _ in range(2))
    return dict(q=q, k=k, v=v, cu_q=_cu(q_lens), cu_k=_cu(k_lens), scale=1.0 / math.sqrt(D))


def prepare(case: dict, seed: int) -> dict:
    st = dict(case, stream=torch.cuda.current_stream().cuda_stream, ctx=_context(case.get("splits", 1)))
    st.update(_inputs(case, seed))
    H = case["heads"]
    if case["op"] == "merge":
        st["out"], st["lse"] = torch.empty_like(st["o_parts"][0]), torch.empty_like(st["lse_parts"][0])
    elif case["op"] == "exchange":
        st["send"], st["y"] = torch.empty_like(st["received"]), torch.empty_like(st["x"])
    else:
        st["out"] = torch.empty_like(st["q"])
        st["lse"] = torch.empty((st["q"].shape[0], H), device="cuda") if case["entry"] == "lse" else None
    return st


def run(st: dict):
    ctx, H, D, stream = st["ctx"], st["heads"], st["head_dim"], st["stream"]
    if st["op"] == "merge":
        da.dit_attn_merge(ctx, st["o_parts"], st["lse_parts"], st["rows"], H, D, st["out"], st["lse"], stream)
        return st["out"], st["lse"]
    if st["op"] == "exchange":
        da.dit_attn_sp_pack_heads(ctx, st["x"], st["send"], st["rows"], H, D, st["degree"], stream)
        da.dit_attn_sp_unpack_heads(ctx, st["received"], st["y"], st["rows"], H, D, st["degree"], stream)
        return st["send"], st["y"]
    q, k, v, out = st["q"], st["k"], st["v"], st["out"]
    if st["op"] == "cross":
        da.dit_attn_cross_varlen_fwd(ctx, q, k, v, st["cu_q"], st["cu_k"], H, D, st["scale"], out, st["lse"], stream)
    elif st["entry"] == "lse":
        da.dit_attn_varlen_fwd_lse(ctx, q, k, v, st["cu_q"], H, D, st["scale"], out, st["lse"], stream)
    elif st["entry"] == "noalloc":
        da.dit_attn_varlen_fwd_noalloc(ctx, q, k, v, st["cu_q"], H, D, st["scale"], out, stream)
    else:
        da.dit_attn_varlen_fwd(ctx, q, k, v, st["cu_q"], H, D, st["scale"], out, stream)
    return out if st["lse"] is None else (out, st["lse"])


def exact(case: dict, seed: int):
    """What `run` returns, in 64 bits from the definitions."""
    x = _inputs(case, seed)
    if case["op"] == "exchange":
        n, H, D, p = case["rows"], case["heads"], case["head_dim"], case["degree"]
        return (x["x"].view(n, p, H // p, D).transpose(0, 1).contiguous(),
                x["received"].transpose(0, 1).reshape(n, H, D))
    if case["op"] == "merge":
        lse = torch.stack(x["lse_parts"]).double()
        total = torch.logsumexp(lse, 0)
        out = torch.zeros(x["o_parts"][0].shape, dtype=torch.float64, device="cuda")
        for o, l in zip(x["o_parts"], lse):
            out += torch.exp(l - total)[..., None] * o
        return out, total
    q, k, v, cu_q, cu_k = x["q"], x["k"], x["v"], x["cu_q"], x["cu_k"]
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
    for q0, q1, k0, k1 in zip(cu_q[:-1], cu_q[1:], cu_k[:-1], cu_k[1:]):
        step = max(1, int(2.5e8 // (k1 - k0)))  # rows at a time: two gigabytes of scores
        for h in range(case["heads"]):
            kt, vh = k[k0:k1, h].double().t().contiguous(), v[k0:k1, h].double()
            for r0 in range(q0, q1, step):
                r1 = min(q1, r0 + step)
                s = (q[r0:r1, h].double() @ kt).mul_(x["scale"])
                m = s.amax(1, keepdim=True)
                s = s.sub_(m).exp_()
                total = s.sum(1, keepdim=True)
                out[r0:r1, h] = (s @ vh) / total
                lse[r0:r1, h] = (m + total.log())[:, 0]
    return (out, lse) if case["entry"] == "lse" else out


def work(case: dict) -> dict:
    H, D = case["heads"], case["head_dim"]
    if case["op"] == "merge":
        n = case["rows"] * H
        return {"bytes": (case["parts"] + 1) * n * (2 * D + 4), "flops": 2 * case["parts"] * n * D}
    if case["op"] == "exchange":
        return {"bytes": 4 * case["rows"] * H * D * 2, "flops": 0}
    q_lens = _lens(case["q_lens"])
    k_lens = _lens(case["k_lens"]) if case["op"] == "cross" else q_lens
    rows = sum(q_lens)
    # Q, O, K and V once, the log-sum-exp where it is asked for; two contractions, a multiply-add counts as two
    nbytes = 2 * H * D * 2 * (rows + sum(k_lens)) + (4 * rows * H if case["entry"] == "lse" else 0)
    return {"bytes": nbytes, "flops": 4 * H * D * sum(a * b for a, b in zip(q_lens, k_lens))}


def tolerance(case: dict):
    """Against the exact result.  Measured in 64-bit arithmetic on rows of every listed case: attention outputs are off by
    1.9e-3 to 2.35e-3 in the 2-norm (1.66e-3 of it the bf16 output, the rest the bf16 probabilities) and at most by 0.032
    of the root mean square in one element (the bf16 step of the largest outputs); merged outputs by 1.66e-3 (the bf16
    output alone).  Stated here is four times that; the layout changes move bytes."""
    if case["op"] == "exchange":
        return "exact"
    if case["op"] == "merge":
        return {"rel": 6.6e-3}
    return {"rel": 9e-3, "max": 0.13}
