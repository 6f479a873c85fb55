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

template <int kCM, bool kMask, bool kWide, bool kGen, bool kExact, bool kFew>
__global__ void __launch_bounds__((kCellsThreads<kCM, kWide>)) k_gather_cells(const GatherArgs a, int subs, int nk) {
  extern __shared__ __align__(32) unsigned char s_dyn[];
  const int per_tile = CellsShape<kCM, kMask, kGen, kFew>::kSubs / subs;
  const int work = a.ntiles * per_tile;
  const int b = (int)wide_block(), eighth = (work + 7) >> 3;
  const int w = (b & 7) * eighth + (b >> 3);
  if ((b >> 3) >= eighth || w >= work) return;
  const int tile = w / per_tile;
  cells_tile<kCM, kMask, kWide, kGen, kExact, kFew>(a, tile, (w - tile * per_tile) * subs, subs, nk,
                                                    s_dyn);
}

template <int kCM, bool kMask, bool kWide, bool kGen>
__global__ void __launch_bounds__(64) k_gather_lane(const GatherArgs a) {
  extern __shared__ __align__(32) unsigned char s_dyn[];
  const int tile = (int)(blockIdx.x & 7) * a.tiles_per_xcd + (int)(blockIdx.x >> 3);
  if (tile < a.ntiles) cells_lane<kCM, kMask, kWide, kGen>(a, tile, s_dyn);
}

// Fewest tiles whose sixteen-cell sub-blocks, of eight waves each, fill the chip
// with the other kernel shapes (two waves per SIMD): see CellsShape's kFew.
constexpr int kCellsFewTiles = 64;

// Waves per sub-block: no more than fill the chip (four per SIMD; at C = 1,
// whose sub-blocks of sixteen cells do the most work per candidate, four
// rounds of them) and two chunks of 64 candidates for each.  Waves 1 / 2 / 4 /
// 8 / 16, us: 1456 sub-blocks of 393 candidates, C = 2: 15 / 12 / 16 / 22 / 38;
// 5168 of 651, C = 8: 42 / 48 / 64 / 135; 1352 of 64,000, C = 4: 711 / 429 / 426
// / 593; 400 of 866, C = 8: 18 / 13 / 11 / 17; C = 1, 5776 of 7100: 353 / 315 /
// 312 / 344 / 448, 576 of 79,000: eight 629, sixteen 567.
template <int kCM, bool kMask, bool kWide, bool kGen, bool kExact,
          bool kFew = kCM == 1 && kWide && !kGen>
static void launch_cells_kernel(const hcg_plan_s* p, const GatherArgs& a, hipStream_t stream) {
  if (cells_by_lane(p, kCM, kMask)) {
    k_gather_lane<kCM, kMask, kWide, kGen>
        <<<(unsigned)a.tiles_per_xcd * 8u, 64, cells_lane_lds_size<kCM>(a.maxr), stream>>>(a);
    return;
  }
  if constexpr (kGen && kCM == 1 && !kFew)
    if (a.ntiles < kCellsFewTiles)
      return launch_cells_kernel<kCM, kMask, kWide, kGen, kExact, true>(p, a, stream);
  using Sh = CellsShape<kCM, kMask, kGen, kFew>;
  const int64_t all = (int64_t)a.ntiles * Sh::kSubs;
  constexpr int kMost = kCellsThreads<kCM, kWide> / 64;
  constexpr int64_t kWaves = kCM == 1 ? 16384 : 4096;
  int nk = 1;
  while (nk < kMost && all * nk * 2 <= kWaves && p->load.most >= 64.0 * 2 * (nk * 2)) nk *= 2;
  const int subs = nk >= 4 ? 1 : 4 / nk;
  const int64_t work = all / subs;
  const size_t lds = cells_lds_size<Sh::kNC, Sh::kS, kGen>(subs * nk, subs, a.maxr);
  k_gather_cells<kCM, kMask, kWide, kGen, kExact, kFew>
      <<<wide_grid((work + 7) / 8 * 8), 64 * subs * nk, lds, stream>>>(a, subs, nk);
}

template <bool kMask, bool kWide, bool kGen, bool kExact = false>
static void launch_cells_by_c(const hcg_plan_s* p, const GatherArgs& a, hipStream_t stream) {
  if (a.C == 1) launch_cells_kernel<1, kMask, kWide, kGen, kExact>(p, a, stream);
  else if (a.C == 2) launch_cells_kernel<2, kMask, kWide, kGen, kExact>(p, a, stream);
  else if (a.C <= 4) launch_cells_kernel<4, kMask, kWide, kGen, kExact>(p, a, stream);
  else launch_cells_kernel<8, kMask, kWide, kGen, kExact>(p, a, stream);
}

// Values in the plan's order: out[p][c] = spec[perm[p]][c].  One value to a
// thread, several where n C of them would be more threads than a launch holds.
constexpr int64_t kSortBlocks = 1 << 22;
__global__ void __launch_bounds__(256) k_sort_values(const float* __restrict__ spec,
                                                     const uint32_t* __restrict__ perm, int64_t n,
                                                     int C, float* __restrict__ out) {
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n * C; i += step) {
    if (C == 1) {
      out[i] = spec[perm[i]];
    } else {
      const int64_t p = i / C;
      out[i] = spec[(int64_t)perm[p] * C + (i - p * C)];
    }
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
  if (may_alloc && p->n >= kCellsSortFrom) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool open = hipStreamIsCapturing(stream, &cap) == hipSuccess &&
                      cap == hipStreamCaptureStatusNone;
    hipMemPool_t pool = open ? plan_pool() : nullptr;
    const size_t bytes = sizeof(float) * (size_t)p->n * C;
    if (open &&
        (pool ? hipMallocFromPoolAsync((void**)&sorted, bytes, pool, stream)
              : hipMallocAsync((void**)&sorted, bytes, stream)) == hipSuccess) {
      k_sort_values<<<(unsigned)std::min((p->n * C + 255) / 256, kSortBlocks), 256, 0, stream>>>(
          spec, p->perm, p->n, C, sorted);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) {
        (void)hipFreeAsync(sorted, stream);
        return fail(HCG_E_DEVICE, "launch of k_sort_values failed: %s", hipGetErrorString(e));
      }
      a.spec = sorted;
      a.perm = nullptr;
    } else {
      (void)hipGetLastError();
      sorted = nullptr;  // capturing, or no room: the values are read through the permutation
    }
  }
  a.C = C;
  a.cube = cube;
  a.wmap = wmap;
  a.wcube = wcube;
  // the circular Gaussian and the other kernel shapes are separate kernels,
  // so the common case carries no general weight path in its registers
  const bool gen = p->kern.type != kGauss, narrow = cells_narrow(a.c2R, p->kern);
  if (!centred_chords(p)) {
    if (mask) launch_cells_by_c<true, true, true, true>(p, a, stream);
    else launch_cells_by_c<false, true, true, true>(p, a, stream);
  } else if (mask) {
    if (gen) launch_cells_by_c<true, true, true>(p, a, stream);
    else if (narrow) launch_cells_by_c<true, false, false>(p, a, stream);
    else launch_cells_by_c<true, true, false>(p, a, stream);
  } else {
    if (gen) launch_cells_by_c<false, true, true>(p, a, stream);
    else if (narrow) launch_cells_by_c<false, false, false>(p, a, stream);
    else launch_cells_by_c<false, true, false>(p, a, stream);
  }
  const hipError_t le = hipGetLastError();
  if (sorted) (void)hipFreeAsync(sorted, stream);
  if (le != hipSuccess)
    return fail(HCG_E_DEVICE, "launch of k_gather_cells failed: %s", hipGetErrorString(le));
  return HCG_OK;
}

}  // namespace hcg
