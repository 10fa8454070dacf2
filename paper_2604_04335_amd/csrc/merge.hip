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

namespace dit {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  f32x2 f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));  // round to nearest even
}

// U chunks per thread, 256 apart, all their loads issued before the first is used.  SHIFT: log2 of the chunks of a (row,
// head).  STREAM_IN, STREAM_OUT: the parts are read, the output is written past the caches.
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
    else *dst = y;
    if (p.lse_out != nullptr && (e & ((1 << SHIFT) - 1)) == 0) p.lse_out[rh] = tot > 0.f ? m_safe + __logf(tot) : -__builtin_inff();
  }
}

// Where parts and output together fit the 256 MB memory-side cache, whoever reads the output next finds it there, and it is
// written with ordinary stores, one chunk per thread (more workgroups).  Past that it would be evicted anyway and leaves as
// streaming stores, two chunks per thread from three parts on (two parts of 380 MB and the copy below: 173 us with one
// chunk per thread, 180 with two, 171 with ordinary stores).
// Us of a merge on changing buffers and a copy that reads its output, ordinary stores and one chunk / streaming ones and two
// (in brackets without the copy), by bytes of the parts, MI355X:
//   two parts   10 MB  7.0 / 7.8 (4.2 / 4.3)    60 MB 26.8 / 29.3 (17.9 / 17.4)   150 MB 69 / 70 (40 / 40)   250 MB 120 / 118 (67 / 65)
//   four parts  20 MB  9.0 / 10.2 (6.4 / 6.5)   60 MB 21.4 / 23.4 (16.1 / 15.9)   150 MB 47 / 49 (36 / 35)   250 MB  86 / 84 (59 / 56)
//   eight parts 20 MB  8.3 / 9.8 (6.0 / 7.1)    60 MB 18.4 / 19.3 (15.3 / 14.6)   150 MB 39 / 41 (34 / 32)   270 MB  72 / 71 (59 / 56)
constexpr int64_t kStreamOutBytes = 256ll << 20;  // of parts and output
// Parts of this many bytes and more in all are also read with streaming loads, up to four chunks per thread.  The same
// buffers over and over, ordinary loads / streaming ones: four parts of 147 MB 27.5 / 30, of 295 MB 56 / 61;  of 450 MB
// 100 / 92, of 600 MB 134 / 123, of 1.2 GB 266 / 245.  With the copy that reads the output, 600 MB 198 / 181, 1.2 GB 388 / 361.
constexpr int64_t kStreamInBytes = 400ll << 20;

template <int P, bool F32, int U, int SHIFT, bool STREAM_IN, bool STREAM_OUT>
static hipError_t launch(const MergeParams& p, hipStream_t stream) {
  const int64_t blocks = (p.n_chunks + 256 * U - 1) / (256 * U);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL((merge_kernel<P, F32, U, SHIFT, STREAM_IN, STREAM_OUT>), dim3((unsigned)blocks), dim3(256), 0, stream, p);
  return hipGetLastError();
}

template <int P, int SHIFT>
static hipError_t launch_parts(const MergeParams& p, hipStream_t stream) {
  if (p.in_f32) return launch<P, true, 1, SHIFT, false, false>(p, stream);  // split keys: a few rows, read next by the caller
  if ((P + 1) * p.n_chunks * 16 < kStreamOutBytes) return launch<P, false, 1, SHIFT, false, false>(p, stream);
  if (P * p.n_chunks * 16 < kStreamInBytes) return launch<P, false, P <= 2 ? 1 : 2, SHIFT, false, true>(p, stream);
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
