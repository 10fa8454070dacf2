// Launch interface between the C ABI and the gfx950 attention kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.h"

namespace dit {

struct AttnParams {
  const void* q;            // bf16 [Tq, H, D]
  const void* k;            // bf16 [Tk, H, D] (Tk = Tq and the same boundaries for self-attention)
  const void* v;
  void* out;                // bf16 [T, H, D]
  float* part_out;          // split-KV: fp32 [n_parts, Tq, H, D] workspace for normalised partial results, else nullptr;
                            // then out is not written and part_lse (fp32 [n_parts, Tq, H]) takes every part's lse
  float* part_lse;
  int64_t part_rows;        // Tq
  float* lse;               // fp32 [T, H] or nullptr: natural-log sum of exp(scale * score) of every (query row, head)
  const WorkItem* items;    // device work-list
  uint32_t* sync;           // device, 8 words (8-byte aligned): [0] items asked for so far, [1] unused, [2..3] shader
                            // cycles and [4..5] 100 MHz ticks workgroup 0 of the last launch ran for.  Word 0 is zero
                            // between launches: the last workgroup to ask clears it (so a launch can be replayed from
                            // a captured graph, and the host keeps no count).
  uint32_t n_items;
  int32_t n_heads;
  float c_log2;             // |scale| * log2(e), at least 1e-30: never zero, so that a masked score of -inf times it
                            // stays -inf (scale 0 then gives every live key the same weight, as it must)
  int32_t negate;           // 1 when scale < 0: the sign of Q is flipped on load
};

// The parameters of a launch with no more items than workgroups whose items are a formula (items and sync are not read).  A type and
// kernel instances of their own: with the list among the arguments of every launch the small packs of the ordinary entry
// points took 0.25 us longer (410 rows x 24 heads at head dimension 64, 7.8 -> 8.05).
struct AttnListParams : AttnParams {
  PackList list;
};

// Two kernels share the tile code.
//   kIndependent128: 4 wavefronts, 128 query rows per item, two (head dimension 64: three) unsynchronised workgroups per
//                    compute unit; a wavefront contracts the next tile's scores beside the softmax of this one.
//   kPingPong256:    8 wavefronts, 256 query rows per item, one workgroup per compute unit whose two wavefront
//                    groups alternate between the matrix and the vector phase of consecutive tiles.
enum class AttnKernel : int { kIndependent128 = 0, kPingPong256 = 1 };

// Which kernel a pack runs on a device with n_cus compute units (a pure function of the pack).
// cu_seqlens_k == nullptr: keys share the query boundaries.
AttnKernel attn_fwd_select(const int32_t* cu_seqlens, const int32_t* cu_seqlens_k, int32_t n_seqs, int32_t n_heads,
                           int head_dim, int n_cus);

// Query rows per work item and resident workgroups per compute unit of a kernel.
int attn_fwd_block_m(AttnKernel kernel);
int attn_fwd_wgs_per_cu(AttnKernel kernel, int head_dim);

// Load the code of every attention kernel on the current device and set its LDS limit (a launch would otherwise do both
// the first time, which allocates; dit_attn_create calls this so that no later launch has to).
hipError_t attn_fwd_prepare();

// Enqueue the forward kernel with persistent workgroups (at most attn_fwd_wgs_per_cu of them per compute unit) on a device
// with n_cus compute units.  max_keys: the most keys of any item.  list: nullptr, or the items in place of p.items.
hipError_t attn_fwd_launch(const AttnParams& p, const PackList* list, AttnKernel kernel, int head_dim, int n_cus, int32_t max_keys, hipStream_t stream);

}  // namespace dit

