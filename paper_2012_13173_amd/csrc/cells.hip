// Launches of the few-channel gather (FP32, C <= 8) on one plan: the kernels
// around cells_tile (cells_tile.h).
#include <cmath>

#include "cells_tile.h"

namespace hcg {

// ---------------------------------------------------------------------------
// Few channels (C <= 8): cells_tile (cells_tile.h) on one plan.  Workgroups
// of four waves on four sub-blocks of a tile, or of nk waves on one.  The
// blocks go to the XCDs in contiguous eighths, as in k_gather_mfma.
// ---------------------------------------------------------------------------
// Largest workgroup: sixteen waves where a wave's registers allow four per
// SIMD, else eight.
template <int kCM, bool kWide>
constexpr int kCellsThreads = kCM <= 2 && !kWide ? 1024 : 512;

template <int kCM, bool kMask, bool kWide, bool kGen>
__global__ void __launch_bounds__((kCellsThreads<kCM, kWide>)) k_gather_cells(const GatherArgs a, int subs, int nk) {
  extern __shared__ __align__(32) unsigned char s_dyn[];
  const int per_tile = CellsShape<kCM, kMask>::kSubs / subs;
  const int work = a.ntiles * per_tile;
  const int w = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (w >= work) return;
  const int tile = w / per_tile;
  cells_tile<kCM, kMask, kWide, kGen>(a, tile, (w - tile * per_tile) * subs, subs, nk, s_dyn);
}

// Waves per sub-block, by the number of sub-blocks: one from two waves per
// SIMD on, else four, and below a quarter of that as many as a workgroup
// takes (kMost), which also shortens the last round of workgroups (576
// sub-blocks of 10^7 samples on 90 x 90 cells: 629 us with eight waves each,
// 567 us with sixteen).
constexpr int64_t kCellsFewWaves = 8192;

template <int kCM, bool kMask, bool kWide, bool kGen>
static void launch_cells_kernel(const GatherArgs& a, hipStream_t stream) {
  using Sh = CellsShape<kCM, kMask>;
  const int64_t all = (int64_t)a.ntiles * Sh::kSubs;
  constexpr int kMost = kCellsThreads<kCM, kWide> / 64;
  const int nk = all >= kCellsFewWaves ? 1 : all >= kCellsFewWaves / 4 ? 4 : kMost;
  const int subs = nk == 1 ? 4 : 1;
  const int64_t work = all / subs;
  const size_t lds = cells_lds_size<Sh::kNC, Sh::kS, kGen>(subs * nk, subs, a.maxr);
  k_gather_cells<kCM, kMask, kWide, kGen>
      <<<(unsigned)((work + 7) / 8 * 8), 64 * subs * nk, lds, stream>>>(a, subs, nk);
}

template <bool kMask, bool kWide, bool kGen>
static void launch_cells_by_c(const GatherArgs& a, hipStream_t stream) {
  if (a.C == 1) launch_cells_kernel<1, kMask, kWide, kGen>(a, stream);
  else if (a.C == 2) launch_cells_kernel<2, kMask, kWide, kGen>(a, stream);
  else if (a.C <= 4) launch_cells_kernel<4, kMask, kWide, kGen>(a, stream);
  else launch_cells_kernel<8, kMask, kWide, kGen>(a, stream);
}

// Values in the plan's order: out[p][c] = spec[perm[p]][c].
__global__ void __launch_bounds__(256) k_sort_values(const float* __restrict__ spec,
                                                     const uint32_t* __restrict__ perm, int64_t n,
                                                     int C, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (C == 1) {
    if (i < n) out[i] = spec[perm[i]];
  } else if (i < n * C) {
    const int64_t p = i / C;
    out[i] = spec[(int64_t)perm[p] * C + (i - p * C)];
  }
}

// From this many samples on, the values are put into the plan's order first
// (scratch): every candidate's values are read by several sub-blocks, and
// through the permutation each such read is a line of its own.
constexpr int64_t kCellsSortFrom = 1 << 18;

hcg_status launch_cells(const hcg_plan_s* p, const float* spec, int C, float* cube, float* wmap,
                        float* wcube, bool mask, bool may_alloc, hipStream_t stream) {
  GatherArgs a = plan_args(p);
  a.spec = spec;
  float* sorted = nullptr;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (may_alloc && p->n >= kCellsSortFrom &&
      hipStreamIsCapturing(stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone) {
    hipMemPool_t pool = plan_pool();
    const size_t bytes = sizeof(float) * (size_t)p->n * C;
    if ((pool ? hipMallocFromPoolAsync((void**)&sorted, bytes, pool, stream)
              : hipMallocAsync((void**)&sorted, bytes, stream)) == hipSuccess) {
      k_sort_values<<<(unsigned)((p->n * C + 255) / 256), 256, 0, stream>>>(spec, p->perm, p->n, C,
                                                                           sorted);
      a.spec = sorted;
      a.perm = nullptr;
    } else {
      sorted = nullptr;  // no room: the values are read through the permutation
    }
  }
  (void)hipGetLastError();
  a.C = C;
  a.cube = cube;
  a.wmap = wmap;
  a.wcube = wcube;
  // the circular Gaussian and the other kernel shapes are separate kernels,
  // so the common case carries no general weight path in its registers
  const bool gen = p->kern.type != kGauss, narrow = cells_narrow(a.c2R, p->kern);
  if (mask) {
    if (gen) launch_cells_by_c<true, true, true>(a, stream);
    else if (narrow) launch_cells_by_c<true, false, false>(a, stream);
    else launch_cells_by_c<true, true, false>(a, stream);
  } else {
    if (gen) launch_cells_by_c<false, true, true>(a, stream);
    else if (narrow) launch_cells_by_c<false, false, false>(a, stream);
    else launch_cells_by_c<false, true, false>(a, stream);
  }
  const hipError_t le = hipGetLastError();
  if (sorted) (void)hipFreeAsync(sorted, stream);
  if (le != hipSuccess)
    return fail(HCG_E_DEVICE, "launch of k_gather_cells failed: %s", hipGetErrorString(le));
  return HCG_OK;
}

}  // namespace hcg
