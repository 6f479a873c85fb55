// Work items of the batch kernels (batch.hip, gather_wave.hip): the persistent
// kernels' counters and the decoding of an item.
#pragma once

#include "hcg_internal.h"

namespace hcg {

// ctl: [0..7] next item of each XCD's segment, [8] item count, [9] segment
// count.  The item space of a class is cut into eight contiguous segments,
// one per XCD (the hardware deals workgroups to the XCDs in turn, so
// workgroup b starts on XCD b % 8); a workgroup pops items from its own
// XCD's segment -- neighbouring tiles of one field, sharing candidate rows in
// that XCD's L2 -- and, once it is empty, from the others.
__device__ __forceinline__ uint32_t batch_seg_begin(uint32_t total, int x) {
  return (uint32_t)(((uint64_t)total * (uint32_t)x) / kBatchXcds);
}

// The next item of a persistent workgroup: thread 0 pops one from its
// XCD's segment, then from the others once it is empty (*k counts the
// segments it has found empty); 0xFFFFFFFF when every segment is empty.
// Called by every thread of the workgroup.
__device__ inline uint32_t batch_next_item(uint32_t* __restrict__ ctl, uint32_t total, int home,
                                           int* k, uint32_t* s_item) {
  if (threadIdx.x == 0) {
    uint32_t it = 0xFFFFFFFFu;
    while (*k < kBatchXcds) {
      const int x = (home + *k) % kBatchXcds;
      const uint32_t i = atomicAdd(&ctl[x], 1u);
      if (i < batch_seg_begin(total, x + 1)) { it = i; break; }
      ++*k;
    }
    *s_item = it;
  }
  __syncthreads();
  const uint32_t it = __builtin_amdgcn_readfirstlane(*s_item);
  __syncthreads();
  return it;
}

// The segment of item it: the last one whose base is <= it.
__device__ inline BatchSeg batch_seg_of(const BatchSeg* __restrict__ segs, uint32_t nseg,
                                        uint32_t it) {
  uint32_t lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (segs[mid].base <= it) lo = mid; else hi = mid - 1;
  }
  return segs[lo];
}

}  // namespace hcg
