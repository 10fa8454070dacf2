// Single-GPU halves of the head-split sequence-parallel all-to-all (paper Section 4.3 elastic sequence parallelism,
// Section 5 unified sequence parallelism): pure index maps over 16-byte chunks, HBM bound.
//     pack    [n, H, D] -> [p, n, H/p, D]     send[g, r, h, :] = x[r, g*H/p + h, :]
//     unpack  [p, n, H/p, D] -> [n, H, D]     y[r, g*H/p + h, :] = recv[g, r, h, :]
// Both sides of a group are walked with one index e = row * group_chunks + chunk: on the side [p, n, H/p, D] a group is
// contiguous, on the side [n, H, D] its rows are H*D*2 bytes apart.  One thread per 16 bytes and one group per blockIdx.y,
// so that an index costs one 32-bit division (64-bit ones, three a chunk, held the loop at a third fewer bytes in
// flight).
// Traffic: every byte read once and written once; bound by HBM, above 256 MB in total, or by the memory-side cache.  Pack
// and unpack of [19028, 40, 128], p = 4, MI355X: 153 -> 128 us (6.1 TB/s; torch's copy of the same bytes 5.2).  Two to
// eight chunks per thread were no faster at any size (8: half the rate).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sp_layout.h"
#include "store_through.h"

namespace dit {

// Index: uint32_t, or uint64_t for a group of 2^32 chunks and more.
// group_chunks: 16-byte chunks of one (row, head group) = (H/p) * D * 2 / 16;  group_total = n_rows * group_chunks.
// STREAM_IN: the source is read with streaming loads.  STREAM_OUT: the destination is written with streaming stores.
template <bool PACK, bool STREAM_IN, bool STREAM_OUT, class Index>
__global__ void __launch_bounds__(256) sp_layout_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, Index group_total,
                                                        uint32_t p, uint32_t group_chunks) {
  const uint32_t g = blockIdx.y;
  const uint64_t step = (uint64_t)gridDim.x * 256;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < group_total; i += step) {
    const Index e = (Index)i;
    const uint64_t row = e / group_chunks;
    const uint64_t grouped = (uint64_t)g * group_total + e;              // [g][row][chunk]
    const uint64_t plain = e + (row * (p - 1) + g) * group_chunks;       // [row][g][chunk]
    const u32x4* from = src + (PACK ? plain : grouped);
    const u32x4 x = STREAM_IN ? __builtin_nontemporal_load(from) : *from;
    if constexpr (STREAM_OUT) __builtin_nontemporal_store(x, dst + (PACK ? grouped : plain));
    else store_through(dst + (PACK ? grouped : plain), x);
  }
}

template <bool PACK, bool STREAM_IN, bool STREAM_OUT>
static void launch(const void* src, void* dst, int64_t group_total, uint32_t p, uint32_t group_chunks, hipStream_t stream) {
  int64_t blocks = (group_total + 255) / 256;
  if (blocks > (1 << 23)) blocks = 1 << 23;  // 2^31 threads; the rest by the loop
  const dim3 grid((unsigned)blocks, p), block(256);
  if (group_total <= 0xFFFFFFFFll)
    hipLaunchKernelGGL((sp_layout_kernel<PACK, STREAM_IN, STREAM_OUT, uint32_t>), grid, block, 0, stream, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), (uint32_t)group_total, p, group_chunks);
  else
    hipLaunchKernelGGL((sp_layout_kernel<PACK, STREAM_IN, STREAM_OUT, uint64_t>), grid, block, 0, stream, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), (uint64_t)group_total, p, group_chunks);
}

// Tensors of kStreamInBytes and more are read with streaming loads, which keep the source from pushing the destination out of
// the memory-side cache before its reader comes; from kStreamOutBytes on, where it does not stay there anyway, the destination
// is written with streaming stores instead.  Us of a pack of [n, 40, 128], ordinary / streaming loads with stores written
// through, streaming loads and stores, MI355X:
//            three pairs of buffers    many               and a copy of the result   and a reader of 64 workgroups
//    15 MB    5.5 /  5.7 /  6.4       8.0 /  6.5 /  6.9    13.0 / 12.1 / 14.5          24 /  24 /  37
//    25 MB    8.2 /  8.7 /  9.8      11.4 / 10.4 / 10.5    18.8 / 17.9 / 21.6          38 /  38 /  59
//    41 MB   12.4 / 13.4 / 14.5      16.7 / 15.0 / 15.2    27.6 / 26.6 / 31.7          57 /  58 /  92
//    61 MB   22.2 / 19.0 / 21.0      23.2 / 20.9 / 21.6    39.8 / 37.9 / 44.8          83 /  83 / 135
//   123 MB   43.7 / 38.8 / 40.2      43.7 / 38.8 / 40.1   103   / 82.5 / 84           206 / 160 / 264
//   195 MB   70   / 60   / 62        70   / 60   / 62     143   / 133  / 137          433 / 354 / 428
// A pack and an unpack in turn on three sets of buffers, ordinary / streaming loads: 15 MB 11.4 / 12.7, 20 MB 14.0 / 16.2 (on
// six sets 15.1 / 13.3 and 19.0 / 16.4);  written through / with streaming stores, streaming loads: 82 MB 57 / 58, 123 MB 82 /
// 84, 159 MB 108 / 108, 174 MB 118 / 115, 195 MB 134 / 128.  Below 12 MB all are alike (3.6 to 4.4 us a call).
constexpr int64_t kStreamInBytes = 24ll << 20;
constexpr int64_t kStreamOutBytes = 160ll << 20;

hipError_t sp_layout_launch(bool pack, const void* src, void* dst, int64_t n_rows, int n_heads, int head_dim, int sp_degree,
                            hipStream_t stream) {
  const uint32_t group_chunks = (uint32_t)(n_heads / sp_degree) * (uint32_t)head_dim * 2 / 16;
  const int64_t group_total = n_rows * group_chunks;
  if (group_total == 0) return hipSuccess;
  const int64_t bytes = group_total * sp_degree * 16;
  auto run = bytes < kStreamInBytes    ? (pack ? launch<true, false, false> : launch<false, false, false>)
             : bytes < kStreamOutBytes ? (pack ? launch<true, true, false> : launch<false, true, false>)
                                       : (pack ? launch<true, true, true> : launch<false, true, true>);
  run(src, dst, group_total, (uint32_t)sp_degree, group_chunks, stream);
  return hipGetLastError();
}

}  // namespace dit
