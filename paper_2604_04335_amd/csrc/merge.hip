// Merge of partial attention results over disjoint key sets, and the fill of output rows that have no keys.
//
// (O_p, lse_p), p < P, are results of the same queries against disjoint key sets (sequence parallelism along the
// sequence, the ring half of the unified sequence parallelism of paper Section 5, hands every GPU one key block per
// step; split-KV does the same inside one GPU).  With lse = ln sum_p exp(lse_p):
//     O = sum_p exp(lse_p - lse) O_p.
// Elementwise and HBM bound: P * (T*H*D*2 + T*H*4) bytes in, T*H*D*2 + T*H*4 out; a thread works on 16-byte chunks.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "merge.h"
#include "store_through.h"

namespace dit {

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  f32x2 f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));  // round to nearest even
}

// U chunks per thread, 256 apart, all their loads issued before the first is used.  SHIFT: log2 of the chunks of a (row,
// head).  STREAM_IN: the parts are read with streaming loads.  STREAM_OUT: the output is written with streaming stores.
// Four bf16 parts on 49178 rows x 24 heads x 128 (1.5 GB in all), MI355X, us: one chunk per thread and ordinary accesses
// 274 (5.5 TB/s); streaming loads and stores 250, with four chunks per thread 245 (6.2 TB/s).
template <int P, bool F32, int U, int SHIFT, bool STREAM_IN, bool STREAM_OUT>
__global__ void __launch_bounds__(256) merge_kernel(MergeParams p) {
  static_assert(!F32 || U == 1, "fp32 parts: one chunk per thread");
  const int64_t e0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;  // 16-byte chunk of the output
  float l[U][P];
  u32x4 x[U][P];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int64_t e = e0 + j * 256;
    if (e >= p.n_chunks) continue;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      l[j][i] = p.lse[i][e >> SHIFT];
      if constexpr (!F32) {
        const u32x4* src = reinterpret_cast<const u32x4*>(p.o[i]) + e;
        x[j][i] = STREAM_IN ? __builtin_nontemporal_load(src) : *src;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int64_t e = e0 + j * 256;
    if (e >= p.n_chunks) break;
    const int64_t rh = e >> SHIFT;  // (row, head)
    float m = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < P; ++i) m = __builtin_fmaxf(m, l[j][i]);
    const float m_safe = m == -__builtin_inff() ? 0.f : m;
    float w[P], tot = 0.f;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      w[i] = __expf(l[j][i] - m_safe);  // exp(-inf) = 0: a part without keys has no weight
      tot += w[i];
    }
    const float inv = tot > 0.f ? 1.0f / tot : 0.f;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const float wi = w[i] * inv;
      float xv[8];
      if constexpr (F32) {
        typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
        const f32x4* src = reinterpret_cast<const f32x4*>(p.o[i]) + 2 * e;
        const f32x4 x0 = src[0], x1 = src[1];
        xv[0] = x0[0]; xv[1] = x0[1]; xv[2] = x0[2]; xv[3] = x0[3];
        xv[4] = x1[0]; xv[5] = x1[1]; xv[6] = x1[2]; xv[7] = x1[3];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          xv[2 * k] = bf16_lo(x[j][i][k]);
          xv[2 * k + 1] = bf16_hi(x[j][i][k]);
        }
      }
      // a weight of exactly 0 must also silence a non-finite value of a part that had no keys
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] += wi == 0.f ? 0.f : wi * xv[k];
    }
    u32x4 y;
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] = pack2(acc[2 * k], acc[2 * k + 1]);
    u32x4* dst = reinterpret_cast<u32x4*>(p.out) + e;
    if constexpr (STREAM_OUT) __builtin_nontemporal_store(y, dst);
    else store_through(dst, y);
    if (p.lse_out != nullptr && (e & ((1 << SHIFT) - 1)) == 0) p.lse_out[rh] = tot > 0.f ? m_safe + __logf(tot) : -__builtin_inff();
  }
}

// By the bytes of parts and output: ordinary loads and one chunk per thread (more workgroups); from kStreamInBytes on
// streaming loads, which keep the parts from pushing the output out of the 256 MB memory-side cache before its reader comes,
// two chunks per thread from three parts on; with kLargeBytes of parts and kStreamOutBytes of output, where the output does
// not stay there anyway, streaming stores and up to four chunks per thread.  What counts is the pair of the call and the kernel
// that reads the output next: a full-speed copy, or 64 workgroups that wait for each line, as a collective does.
// Us of a merge on changing buffers with the 64-workgroup reader / with a copy / alone, by bytes of the parts, MI355X:
//                          ordinary loads        streaming loads       and streaming stores
//   four parts   60 MB    33 /  21.0 /  15.8    32 /  19.4 /  13.9    45 /  22.0 /  14.5
//               100 MB    51 /  32   /  24.2    49 /  29.6 /  21.6    71 /  33.3 /  22.6
//               220 MB   114 /  74   /  52     100 /  60   /  44     146 /  67   /  46
//               400 MB   269 / 136   /  93     217 / 128   /  84     265 / 121   /  84
//               600 MB   417 / 198   / 140     311 / 193   / 129     402 / 182   / 123
//               1.2 GB   833 / 391   / 278     832 / 377   / 262     809 / 362   / 247
//   two parts   100 MB    77 /  42   /  28.1    76 /  40   /  24.1
//               300 MB   360 / 138   /  80     249 / 130   /  73     346 / 133   /  72
//               600 MB   719 / 269   / 155     721 / 260   / 146     706 / 257   / 142
//   eight parts  60 MB    25 /  18.5 /  15.4    23 /  17   /  13.7
//               300 MB   113 /  81   /  65      97 /  69   /  58     127 /  73   /  58
//               600 MB   256 / 161   / 131     192 / 140   / 110     250 / 143   / 114
//               780 MB                                    / 163                 / 151   (three sets: their outputs no longer fit)
// (Parts that all still lie in that cache want ordinary loads: three sets of four parts of 60 MB in turn 12.7 us and 14.1, the
// same 150 MB over and over 28.3 and 30.7;  all written just before the call, which then counts too, 100 MB 61 and 63, 150 MB
// 92 and 89.)
constexpr int64_t kStreamInBytes = 96ll << 20;    // of parts and output
constexpr int64_t kLargeBytes = 400ll << 20;      // of parts
constexpr int64_t kStreamOutBytes = 80ll << 20;   // of output

template <int P, bool F32, int U, int SHIFT, bool STREAM_IN, bool STREAM_OUT>
static hipError_t launch(const MergeParams& p, hipStream_t stream) {
  const int64_t blocks = (p.n_chunks + 256 * U - 1) / (256 * U);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL((merge_kernel<P, F32, U, SHIFT, STREAM_IN, STREAM_OUT>), dim3((unsigned)blocks), dim3(256), 0, stream, p);
  return hipGetLastError();
}

template <int P, int SHIFT>
static hipError_t launch_parts(const MergeParams& p, hipStream_t stream) {
  if (p.in_f32) return launch<P, true, 1, SHIFT, false, false>(p, stream);  // split keys: a few rows
  if ((P + 1) * p.n_chunks * 16 < kStreamInBytes) return launch<P, false, 1, SHIFT, false, false>(p, stream);
  if (P * p.n_chunks * 16 < kLargeBytes || p.n_chunks * 16 < kStreamOutBytes) return launch<P, false, P <= 2 ? 1 : 2, SHIFT, true, false>(p, stream);
  return launch<P, false, P <= 4 ? 4 : 2, SHIFT, true, true>(p, stream);  // 64 registers of loads in flight
}

template <int P>
static hipError_t launch_rows(const MergeParams& p, hipStream_t stream) {
  if (p.chunks_per_row == 8) return launch_parts<P, 3>(p, stream);
  if (p.chunks_per_row == 16) return launch_parts<P, 4>(p, stream);
  return hipErrorInvalidValue;
}

hipError_t merge_launch(const MergeParams& p, int n_parts, hipStream_t stream) {
  if (p.n_chunks == 0) return hipSuccess;
  switch (n_parts) {
    case 1: return launch_rows<1>(p, stream);
    case 2: return launch_rows<2>(p, stream);
    case 3: return launch_rows<3>(p, stream);
    case 4: return launch_rows<4>(p, stream);
    case 5: return launch_rows<5>(p, stream);
    case 6: return launch_rows<6>(p, stream);
    case 7: return launch_rows<7>(p, stream);
    case 8: return launch_rows<8>(p, stream);
    default: return hipErrorInvalidValue;
  }
}

// Rows [row0, row0 + n_rows) of out (n_rows * row_chunks 16-byte chunks) := 0 and of lse := -inf: query rows of a
// sequence that has no keys.  A kernel, not a memset, so that the call can be captured into a graph.
__global__ void __launch_bounds__(256) fill_rows_kernel(u32x4* out, float* lse, int64_t chunk0, int64_t n_chunks, int64_t lse0,
                                                         int64_t n_lse) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n_chunks) out[chunk0 + e] = u32x4{0u, 0u, 0u, 0u};
  if (lse != nullptr && e < n_lse) lse[lse0 + e] = -__builtin_inff();
}

__global__ void __launch_bounds__(256) fill_neg_inf_kernel(float* p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n) p[e] = -__builtin_inff();
}

hipError_t fill_neg_inf_launch(float* p, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fill_neg_inf_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

hipError_t fill_rows_launch(void* out, float* lse, int64_t row0, int64_t n_rows, int n_heads, int head_dim, hipStream_t stream) {
  if (n_rows <= 0) return hipSuccess;
  const int64_t row_chunks = (int64_t)n_heads * head_dim * 2 / 16;
  const int64_t n_chunks = n_rows * row_chunks, n_lse = n_rows * n_heads;
  const int64_t blocks = (n_chunks + 255) / 256;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fill_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, static_cast<u32x4*>(out), lse, row0 * row_chunks,
                     n_chunks, row0 * n_heads, n_lse);
  return hipGetLastError();
}

}  // namespace dit
