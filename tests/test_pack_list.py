"""The work-list as a formula (pack_list_build / pack_list_item) against the list that plan_build_cross writes, item for
item, compiled for the host: ties, empty sequences, ragged and whole lengths, either item height, the limits."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_04335_amd", "csrc")

PROGRAM = r"""
#include "plan.h"
#include <cstdio>
#include <cstring>
#include <random>
using namespace dit;
static WorkItem item(const PackList& l, uint32_t idx, int heads, int bm) {
  int j = 0;
  while (j + 1 < l.n && l.seq[j + 1].first <= idx) ++j;
  return pack_list_item(l.seq[j], idx, static_cast<uint32_t>(heads), bm);
}
int main() {
  std::mt19937 rng(7);
  auto pick = [&](int lo, int hi) { return lo + static_cast<int>(rng() % static_cast<unsigned>(hi - lo + 1)); };
  long built = 0, refused = 0;
  for (int trial = 0; trial < 20000; ++trial) {
    const int n = pick(1, trial % 2 ? 6 : 20), heads = pick(1, 3) == 1 ? pick(1, 200) : pick(1, 40);
    const bool cross = pick(0, 2) == 0;
    std::vector<int32_t> cq(1, 0), ck(1, 0);
    for (int i = 0; i < n; ++i) {
      const int kind = pick(0, 5);
      const int len = kind == 0 ? 0 : kind == 1 ? 256 * pick(1, 6) : kind == 2 ? 410 : kind == 3 ? pick(1, 9000) : pick(1, 700);
      cq.push_back(cq.back() + len);
      ck.push_back(ck.back() + (cross ? pick(0, 3) * pick(0, 300) : len));
    }
    for (int bm : {128, 256}) {
      std::vector<WorkItem> items;
      plan_build_cross(cq.data(), ck.data(), n, heads, bm, items);
      PackList list;
      int live = 0;
      for (int i = 0; i < n; ++i) live += cq[i + 1] > cq[i] && ck[i + 1] > ck[i];
      const bool ok = pack_list_build(cq.data(), ck.data(), n, heads, bm, list);
      const bool want = live > 0 && live <= kPackListSeqs && items.size() <= kPackListItems;
      if (ok != want || (list.n != 0) != ok) { std::printf("trial %d: accepted %d, expected %d\n", trial, ok, want); return 1; }
      if (!ok) { ++refused; continue; }
      ++built;
      for (uint32_t i = 0; i < items.size(); ++i) {
        const WorkItem it = item(list, i, heads, bm);
        if (std::memcmp(&it, &items[i], sizeof(it)) != 0) { std::printf("trial %d item %u differs\n", trial, i); return 1; }
      }
    }
  }
  // the largest quotients: one head, as many whole tiles as the formula takes, and one more
  for (int tiles : {16383, 16384, 16385}) {
    const int32_t cu[2] = {0, 128 * tiles};
    std::vector<WorkItem> items;
    plan_build(cu, 1, 1, 128, items);
    PackList list;
    if (pack_list_build(cu, cu, 1, 1, 128, list) != (tiles <= 16384)) return 1;
    for (uint32_t i = 0; list.n && i < items.size(); ++i) {
      const WorkItem it = item(list, i, 1, 128);
      if (std::memcmp(&it, &items[i], sizeof(it)) != 0) return 1;
    }
  }
  std::printf("built %ld refused %ld\n", built, refused);
  return built > 1000 && refused > 1000 ? 0 : 1;
}
"""


LIST_PROGRAM = r"""
#include "plan.h"
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <random>
using namespace dit;
int main() {
  std::mt19937 rng(11);
  auto pick = [&](int lo, int hi) { return lo + static_cast<int>(rng() % static_cast<unsigned>(hi - lo + 1)); };
  std::vector<WorkItem> items;
  for (int trial = 0; trial < 20000; ++trial) {
    const int n = pick(0, 12), heads = pick(1, 30), splits = pick(0, 1) ? 1 : pick(2, 15), bm = pick(0, 1) ? 128 : 256;
    std::vector<int32_t> cq(1, 0), ck(1, 0);
    for (int i = 0; i < n; ++i) {
      cq.push_back(cq.back() + pick(0, 3) * pick(0, 400));
      ck.push_back(ck.back() + pick(0, 3) * pick(0, 1500));
    }
    // as the list is defined: most keys first, heads, whole query tiles, the ragged tiles behind them, chunks of whole key tiles
    std::vector<int> order;
    for (int i = 0; i < n; ++i) order.push_back(i);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return ck[a + 1] - ck[a] > ck[b + 1] - ck[b]; });
    std::vector<WorkItem> want;
    for (int s : order)
      for (int ragged = 0; ragged < 2; ++ragged)
        for (int h = 0; h < heads; ++h)
          for (int m = cq[s]; m < cq[s + 1]; m += bm) {
            const int rows = std::min(bm, cq[s + 1] - m), keys = ck[s + 1] - ck[s], chunk = ((keys + 63) / 64 + splits - 1) / splits * 64;
            if ((rows < bm) != (ragged == 1)) continue;
            for (int part = 0; part * chunk < keys; ++part)
              want.push_back(WorkItem{m, ck[s] + part * chunk, std::min(chunk, keys - part * chunk), (part << 28) | (rows << 16) | h});
          }
    if (trial % 3 == 0) items.assign(7, WorkItem{1, 2, 3, 4});  // what an earlier call left does not matter
    plan_build_cross(cq.data(), ck.data(), n, heads, bm, items, splits);
    if (items.size() != want.size() || (!want.empty() && std::memcmp(items.data(), want.data(), want.size() * sizeof(WorkItem)) != 0)) {
      std::printf("trial %d: %zu records, expected %zu\n", trial, items.size(), want.size());
      return 1;
    }
  }
  return 0;
}
"""


def _run(program, tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(program)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), os.path.join(CSRC, "plan.cpp"), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout


def test_formula_equals_list(tmp_path):
    _run(PROGRAM, tmp_path)


def test_list_as_defined(tmp_path):
    """plan_build_cross, record for record, against a plain statement of its order: any number of chunks, empty sequences on
    either side, a list object used before."""
    _run(LIST_PROGRAM, tmp_path)


@pytest.mark.gpu
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lens", [[257], [64, 300], [0, 130, 5, 130, 0, 1000, 129], [65 + 7 * i for i in range(16)], [33] * 16 + [0], [40] * 17])
def test_no_allocation_one_round(head_dim, lens):
    """One round of items through the entry point that allocates nothing (up to 16 sequences: no list; 17: the list kernel)
    gives the bits of the ordinary call, also replayed from a graph that was captured without a call before it."""
    import numpy as np
    import torch

    import paper_2604_04335_amd as da

    print(f"no-allocation, one round: D={head_dim} lens={lens}", flush=True)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(len(lens))
    q, k, v = (torch.randn((int(cu[-1]), 5, head_dim), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
    ctx = da.dit_attn_create(0)
    try:
        out, ref = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            da.dit_attn_varlen_fwd_noalloc(ctx, q, k, v, cu, 5, head_dim, 0.1, out, torch.cuda.current_stream().cuda_stream)
        for _ in range(3):
            da.dit_attn_varlen_fwd(ctx, q, k, v, cu, 5, head_dim, 0.1, ref, torch.cuda.current_stream().cuda_stream)
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
        out.fill_(float("nan"))
        da.dit_attn_varlen_fwd_noalloc(ctx, q, k, v, cu, 5, head_dim, 0.1, out, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
    finally:
        da.dit_attn_destroy(ctx)


@pytest.mark.gpu
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lens,heads,kernel", [
    ([1570], 24, "PINGPONG"),                       # the choice at either head dimension too
    ([1, 700, 0, 64, 410, 130], 7, "PINGPONG"),
    ([65 + 70 * i for i in range(16)], 3, "PINGPONG"),
    ([4096], 16, "PINGPONG"),                       # 256 items: one for every compute unit
    ([4352], 15, "PINGPONG"),                       # 255, 68 key tiles
    ([1024], 24, "128"),                            # 192 items of 16 key tiles
    ([1024], 8, "128"),                             # 64
    ([1570, 3, 64, 1215], 5, "128"),
])
def test_no_allocation_one_round_of_either_kernel(head_dim, lens, heads, kernel):
    """Every form of both kernels that takes its items from the formula gives the bits of the ordinary call."""
    import numpy as np
    import torch

    import paper_2604_04335_amd as da

    print(f"no-allocation, {kernel}: D={head_dim} heads={heads} lens={lens}", flush=True)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(len(lens))
    q, k, v = (torch.randn((int(cu[-1]), heads, head_dim), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
    stream = torch.cuda.current_stream().cuda_stream
    ctx = da.dit_attn_create(0)
    try:
        da.dit_attn_set_kernel(ctx, getattr(da, "KERNEL_" + kernel))
        out, again, ref = (torch.full_like(q, float("nan")) for _ in range(3))
        da.dit_attn_varlen_fwd(ctx, q, k, v, cu, heads, head_dim, -0.1, ref, stream)
        da.dit_attn_varlen_fwd_noalloc(ctx, q, k, v, cu, heads, head_dim, -0.1, out, stream)
        da.dit_attn_varlen_fwd_noalloc(ctx, q, k, v, cu, heads, head_dim, -0.1, again, stream)
        torch.cuda.synchronize()
        assert da.dit_attn_last_launch_kernel(ctx) == getattr(da, "KERNEL_" + kernel)
        assert not bool(ref.isnan().any())
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)) and torch.equal(again.view(torch.int16), ref.view(torch.int16))
    finally:
        da.dit_attn_destroy(ctx)
