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

namespace dit {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// Index: uint32_t, or uint64_t for a group of 2^32 chunks and more.
// group_chunks: 16-byte chunks of one (row, head group) = (H/p) * D * 2 / 16;  group_total = n_rows * group_chunks.
// STREAM_IN, STREAM_OUT: the source is read, the destination is written past the caches.
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
    u32x4* to = dst + (PACK ? grouped : plain);
    const u32x4 x = STREAM_IN ? __builtin_nontemporal_load(from) : *from;
    if constexpr (STREAM_OUT) __builtin_nontemporal_store(x, to);
    else *to = x;
  }
}

template <bool PACK, bool STREAM_IN, bool STREAM_OUT>
static void launch(const void* src, void* dst, int64_t group_total, uint32_t p, uint32_t group_chunks, hipStream_t stream) {
  int64_t blocks = (group_total + 255) / 256;
  // Ordinary accesses run better from 4096 workgroups that loop than from one workgroup per 256 chunks ([2000, 40, 128] on
  // changing buffers 10.0 / 10.5 us, [4000, 40, 128] 16.7 / 17.6); streaming loads the other way round ([12000, 40, 128]
  // 45 / 43 us, [15500, 40, 128] 60 / 55), and streaming stores do not care.
  const int64_t cap = STREAM_IN ? 1 << 23 : p < 4096 ? 4096 / p : 1;  // 1 << 23: 2^31 threads
  if (blocks > cap) blocks = cap;
  const dim3 grid((unsigned)blocks, p), block(256);
  if (group_total <= 0xFFFFFFFFll)
    hipLaunchKernelGGL((sp_layout_kernel<PACK, STREAM_IN, STREAM_OUT, uint32_t>), grid, block, 0, stream, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), (uint32_t)group_total, p, group_chunks);
  else
    hipLaunchKernelGGL((sp_layout_kernel<PACK, STREAM_IN, STREAM_OUT, uint64_t>), grid, block, 0, stream, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), (uint64_t)group_total, p, group_chunks);
}

// By the size of the tensor: ordinary accesses; from kStreamInBytes on streaming loads, which keep the source from pushing
// the destination out of the 256 MB memory-side cache before its reader comes; from kStreamOutBytes on, where it does
// not stay there anyway, streaming stores too.  What counts is the pair of the call and the kernel that reads its destination
// next: a full-speed copy, or 64 workgroups that wait for each line, as a collective does.
// Us of a pack of [n, 40, 128] on changing buffers with the 64-workgroup reader / with a copy / alone, MI355X:
//              ordinary            streaming loads     streaming stores    both
//     20 MB    32 /  16.2 / 10.0       /  15.7 /  8.8   49 /  18.4 /  9.1        /  18.3 /  8.7
//     61 MB    85 /  40.8 / 24.1    86 /  41.3 / 23.9  136 /  45.1 / 22.4   136 /  44.9 / 21.6
//     82 MB   132 /  61.4 / 31.9   119 /  54.2 / 30.3  177 /  58.2 / 29.1   177 /  57.9 / 27.7
//    123 MB   187 / 104   / 46.7   163 /  86   / 43.1  269 /  92   / 41.8   262 /  84   / 40.2
//    159 MB   335 / 127   / 60.4   250 / 113   / 54.7  344 / 117   / 53.8   345 / 113   / 51.2
//    195 MB   442 / 147   / 73.9   363 / 141   / 66.4  424 / 142   / 64.6   427 / 137   / 61.9
// (Small tensors that are packed again and again in the same two buffers want ordinary loads: 20 MB 6.4 / 7.7, 41 MB
// 12.5 / 14.6, 82 MB 24.2 / 26.9.)
constexpr int64_t kStreamInBytes = 75ll << 20;
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
