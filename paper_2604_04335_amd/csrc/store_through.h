// A 16-byte store that is written through the L2 and stays in the 256 MB memory-side cache.
//
// An ordinary store leaves its line dirty in the L2 of its XCD; the end of the kernel waits for all of them (up to 32 MB) to be
// written back.  A streaming store avoids that wait but is not kept by the memory-side cache either, and a kernel that reads
// the result next goes to HBM for it: 64 workgroups that wait for each line took up to 1.6 times as long.  Device-scope
// stores have neither cost.  Pack of [6000, 40, 128] (61 MB) with streaming loads, MI355X, us alone / with such a reader /
// with a copy: ordinary 22.4 / 86 / 39.7, streaming 21.6 / 136 / 44.9, this 20.9 / 83 / 37.9;  [19028, 40, 128] 66.4 / 363 /
// 141, 62.2 / 425 / 137, 60.4 / 354 / 133.
//
// (Assembly, because only scalar types have a builtin with a scope.  The s_nop keeps the next instruction from overwriting
// the data registers too early, which the compiler takes care of only for stores that it emits itself.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dit {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

__device__ __forceinline__ void store_through(u32x4* p, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

}  // namespace dit
