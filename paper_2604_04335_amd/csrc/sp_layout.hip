// Single-GPU halves of the head-split sequence-parallel all-to-all (paper Section 4.3 elastic sequence parallelism,
// Section 5 unified sequence parallelism): pure index maps over 16-byte chunks, HBM bound.
//     pack    [n, H, D] -> [p, n, H/p, D]     send[g, r, h, :] = x[r, g*H/p + h, :]
//     unpack  [p, n, H/p, D] -> [n, H, D]     y[r, g*H/p + h, :] = recv[g, r, h, :]
// Both sides of a group are walked with one index e = row * group_chunks + chunk: on the side [p, n, H/p, D] a group is
// contiguous, on the side [n, H, D] its rows are H*D*2 bytes apart.  One thread per 16 bytes and one group per blockIdx.y,
// so that an index costs one 32-bit division (64-bit ones, three a chunk, held the loop at a third fewer bytes in
// flight); the rows leave as streaming stores, which do not evict from the memory-side cache what is still to be read.
// Traffic: every byte read once and written once; bound by HBM, above 256 MB in total, or by that cache.  Pack and
// unpack of [19028, 40, 128], p = 4, MI355X: 153 -> 128 us (6.1 TB/s; torch's copy of the same bytes 5.2); [8000, 40, 128]:
// 64 us without streaming stores, 48 us with them, 57 us with streaming loads too.  Two to eight chunks per thread
// were no faster at any size (8: half the rate).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sp_layout.h"

namespace dit {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// Index: uint32_t, or uint64_t for a group of 2^32 chunks and more.
// group_chunks: 16-byte chunks of one (row, head group) = (H/p) * D * 2 / 16;  group_total = n_rows * group_chunks.
template <bool PACK, bool STREAM, class Index>
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
    __builtin_nontemporal_store(STREAM ? __builtin_nontemporal_load(from) : *from, dst + (PACK ? grouped : plain));
  }
}

template <bool PACK, bool STREAM>
static void launch(const void* src, void* dst, int64_t group_total, uint32_t p, uint32_t group_chunks, hipStream_t stream) {
  int64_t blocks = (group_total + 255) / 256;
  if (blocks > (1 << 23)) blocks = 1 << 23;  // 2^31 threads; the rest by the loop
  const dim3 grid((unsigned)blocks, p), block(256);
  if (group_total <= 0xFFFFFFFFll)
    hipLaunchKernelGGL((sp_layout_kernel<PACK, STREAM, uint32_t>), grid, block, 0, stream, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), (uint32_t)group_total, p, group_chunks);
  else
    hipLaunchKernelGGL((sp_layout_kernel<PACK, STREAM, uint64_t>), grid, block, 0, stream, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), (uint64_t)group_total, p, group_chunks);
}

// Tensors of this size and more are read with streaming loads: [19028, 40, 128] (195 MB) 131 -> 128 us a pair on the same
// buffers and 161 -> 143 us on new ones; [12000, 40, 128] (123 MB), whose bytes the 256 MB memory-side cache still
// holds from the program's last step, 69.5 us with ordinary loads and 80.7 us with streaming ones.
constexpr int64_t kStreamBytes = 160ll << 20;

hipError_t sp_layout_launch(bool pack, const void* src, void* dst, int64_t n_rows, int n_heads, int head_dim, int sp_degree,
                            hipStream_t stream) {
  const uint32_t group_chunks = (uint32_t)(n_heads / sp_degree) * (uint32_t)head_dim * 2 / 16;
  const int64_t group_total = n_rows * group_chunks;
  if (group_total == 0) return hipSuccess;
  const bool stream_loads = group_total * sp_degree * 16 >= kStreamBytes;
  auto run = pack ? (stream_loads ? launch<true, true> : launch<true, false>) : (stream_loads ? launch<false, true> : launch<false, false>);
  run(src, dst, group_total, (uint32_t)sp_degree, group_chunks, stream);
  return hipGetLastError();
}

}  // namespace dit
