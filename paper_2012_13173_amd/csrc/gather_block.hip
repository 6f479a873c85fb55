// Launches of the 16 x 16-cell matrix-core gather (gather_block.h) on one plan.
#include <cmath>

#include "batch_items.h"
#include "gather_block.h"

namespace hcg {

template <int kJ, bool kVec, bool kMask>
__global__ void __launch_bounds__(512, 2) k_gather_block(const GatherArgs a) {
  __shared__ BlockSmem<4> sm;
  // workgroups go to the eight XCDs in turn: each takes a contiguous eighth
  // of the blocks, neighbours on a row of the map behind one L2
  const int per_slab = a.tiles_per_xcd * 8;
  const int slab = blockIdx.x / per_slab;
  const int local = blockIdx.x - slab * per_slab;
  const int tile = (local & 7) * a.tiles_per_xcd + (local >> 3);
  if (tile >= a.ntiles) return;
  gather_block<4, 8, kJ, kVec, kMask>(a, tile, slab, sm);
}

// Rows of two channels to a load: even C, spectra aligned to 8 bytes.
bool block_rows2(const void* spec, int64_t C) { return C % 2 == 0 && (uintptr_t)spec % 8 == 0; }

void block_args(const hcg_plan_s* p, GatherArgs* a) {
  a->kern.kmaj = a->kern.wscale * (1.0 / 12.0);
  a->kern.kmin = a->kern.wscale * (1.0 / 90.0);
  a->ranges = p->branges;
  a->nranges = p->bnranges;
  a->maxr = p->bmaxr;
  a->ntx = p->bntx;
  a->ntiles = p->bntx * p->bnty;
  a->tiles_per_xcd = (a->ntiles + 7) / 8;
}

hcg_status launch_block(const hcg_plan_s* p, const float* spec, int64_t C, float* cube, float* wmap,
                        float* wcube, bool mask, hipStream_t stream) {
  GatherArgs a = plan_args(p);
  block_args(p, &a);
  a.spec = spec;
  a.C = C;
  a.cube = cube;
  a.wmap = wmap;
  a.wcube = wcube;
  const int64_t slab = mask ? kBlockSlabFlagged : kBlockSlab;
  const int64_t blocks = (C + slab - 1) / slab * a.tiles_per_xcd * 8;
  if (blocks > INT32_MAX) return fail(HCG_E_UNSUPPORTED, "hcg_grid: too many channels");
  const unsigned n = (unsigned)blocks;
  if (mask) k_gather_block<1, false, true><<<n, 512, 0, stream>>>(a);
  else if (block_rows2(spec, C)) k_gather_block<2, true, false><<<n, 512, 0, stream>>>(a);
  else k_gather_block<2, false, false><<<n, 512, 0, stream>>>(a);
  HCG_LAUNCH_CHECK("k_gather_block");
  return HCG_OK;
}

// ---------------------------------------------------------------------------
// Fields of a batch: a work item is a block of one channel slab.
// ---------------------------------------------------------------------------
template <bool kVec>
__global__ void __launch_bounds__(512, 2) k_block_items(const GatherArgs* __restrict__ fields,
                                                        const BatchSeg* __restrict__ segs,
                                                        uint32_t nseg) {
  __shared__ BlockSmem<4> sm;
  const uint32_t it = blockIdx.x;
  const BatchSeg sg = batch_seg_of(segs, nseg, it);
  const uint32_t local = it - sg.base;
  const GatherArgs& a = fields[sg.field];
  const uint32_t per_slab = (uint32_t)a.tiles_per_xcd * 8u;
  const uint32_t slab = local / per_slab, loc = local - slab * per_slab;
  const uint32_t tile = (loc & 7u) * (uint32_t)a.tiles_per_xcd + (loc >> 3);
  if (tile < (uint32_t)a.ntiles) gather_block<4, 8, 2, kVec, false>(a, (int)tile, (int)slab, sm);
}

template <bool kVec>
__global__ void __launch_bounds__(512, 2) k_block_batch(const GatherArgs* __restrict__ fields,
                                                        const BatchSeg* __restrict__ segs,
                                                        uint32_t* __restrict__ ctl) {
  __shared__ BlockSmem<4> sm;
  __shared__ uint32_t s_item;
  const uint32_t total = ctl[8], nseg = ctl[9];
  const int home = (int)(blockIdx.x % kBatchXcds);
  int k = 0;
  for (;;) {
    const uint32_t it = batch_next_item(ctl, total, home, &k, &s_item);
    if (it == 0xFFFFFFFFu) break;
    const BatchSeg sg = batch_seg_of(segs, nseg, it);
    const uint32_t local = it - sg.base, slab = local / sg.ntiles;
    gather_block<4, 8, 2, kVec, false>(fields[sg.field], (int)(local - slab * sg.ntiles),
                                       (int)slab, sm);
    __syncthreads();
  }
}

void launch_block_items(bool vec, bool items, uint32_t blocks, const GatherArgs* fields,
                        const BatchSeg* segs, uint32_t nseg, uint32_t* ctl, hipStream_t stream) {
  if (items) {
    if (vec) k_block_items<true><<<blocks, 512, 0, stream>>>(fields, segs, nseg);
    else k_block_items<false><<<blocks, 512, 0, stream>>>(fields, segs, nseg);
  } else {
    if (vec) k_block_batch<true><<<blocks, 512, 0, stream>>>(fields, segs, ctl);
    else k_block_batch<false><<<blocks, 512, 0, stream>>>(fields, segs, ctl);
  }
}

}  // namespace hcg
