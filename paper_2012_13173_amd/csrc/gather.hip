// Data stage of the gridding library: Eq. (1) of HCGrid (Section 2.1) for
// every output cell and channel, gather-side (Section 2.2: each cell pulls
// the samples within its support, so no two workgroups write the same cell).
//
// Work decomposition of the tile gather (the low-precision forms, and FP32 maps
// that neither independent waves, gather_wave.h, nor 16 x 16-cell blocks,
// gather_block.h, are faster for: f32_kernel): one workgroup per 8 x 8 tile of
// output cells and 256- or 512-channel slab.  The tile's candidate samples
// come from the plan's sorted-sample ranges and are staged in blocks of 64,
// one block ahead:
//   1. weights: FP64 great-circle distance of every (cell, candidate) pair
//      of the block that a coarse per-cell-block test cannot rule out (from
//      the chord of the unit vectors), exact support test, Gaussian weight
//      (exponent in FP64, exp2 in FP32), rounded to the operand type of the
//      form; FP64 sums of the weights per cell;
//   2. accumulation: the block is a dense contraction
//      U[cells x channels] += Wt[cells x 64] . S[64 x channels] done on the
//      matrix cores with FP32 accumulation -- FP32 operands
//      (v_mfma_f32_16x16x4_f32) or BF16 / FP16 / FP8 operands (16x16x32),
//      skipping every 16-cell x k-step sub-block whose weights are all zero;
//      the spectra are read in the caller's sample order through the plan's
//      permutation, or (low-precision forms) from an encoding in the plan's
//      sorted order whose groups of 8 samples are ready-made B operands;
//   3. epilogue: V = U / W~ (W~ the sum of the weights actually multiplied,
//      times the channel scale for the scaled forms), NaN where no sample is
//      within the support; W map = FP64 sum of the unrounded weights.
// For a few FP32 channels a wave owns a sub-block of cells and a lane one
// candidate at a time, or a wave a tile, with FP64 sums (cells_tile.h).
#include <cmath>
#include <vector>

#include "gather_tile.h"

namespace hcg {

template <int kForm, int kQW, bool kVec, bool kPacked, bool kWide, bool kGen = false,
          bool kMask = false>
__global__ void __launch_bounds__(256, 2) k_gather_mfma(const GatherArgs a) {
  __shared__ GatherSmem sm;
  // XCD-aware order: the hardware deals consecutive workgroups to the eight
  // XCDs in turn; give each XCD a contiguous run of tiles so that tiles that
  // share candidate rows run together behind the same L2.
  const int per_slab = a.tiles_per_xcd * 8;
  const int slab = blockIdx.x / per_slab;
  const int local = blockIdx.x - slab * per_slab;
  const int tile = (local & 7) * a.tiles_per_xcd + (local >> 3);
  if (tile >= a.ntiles) return;
  gather_tile<kForm, kQW, kVec, kPacked, kWide, true, kGen, kMask>(a, tile, slab, sm);
}

// Exact number of (cell, candidate) pairs within R: one lane per cell.
__global__ void __launch_bounds__(64) k_count_pairs(const GatherArgs a,
                                                    unsigned long long* __restrict__ pair_count) {
  extern __shared__ __align__(16) unsigned char s_dyn[];
  double4* s_xyz = (double4*)s_dyn;             // [kKB]
  uint2* s_rng = (uint2*)(s_xyz + kKB);         // [maxr]
  uint32_t* s_pre = (uint32_t*)(s_rng + a.maxr);  // [maxr + 1]
  const int tile = blockIdx.x, lane = threadIdx.x;
  const int ix = (tile % a.ntx) * kTileX + (lane & 7), iy = (tile / a.ntx) * kTileY + (lane >> 3);
  const CellVec cell = cell_at(a.cells, a.g, ix, iy);
  const uint32_t total =
      stage_ranges(a.ranges + (int64_t)tile * a.maxr, a.nranges[tile], s_rng, s_pre);
  unsigned long long npair = 0;
  uint32_t cur = 0;
  for (uint32_t q0 = 0; q0 < total; q0 += kKB) {
    const uint32_t q = q0 + lane;
    if (q < total) s_xyz[lane] = a.xyz[cand_pos(q, s_rng, s_pre, &cur)];
    __syncthreads();
    const int kmax = (int)min<uint32_t>(kKB, total - q0);
    for (int k = 0; k < kmax; ++k)
      if (chord2(cell, s_xyz[k]) <= a.c2R) ++npair;
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) npair += __shfl_xor(npair, off);
  if (lane == 0) atomicAdd(pair_count, npair);
}

// Below this many 512-channel workgroups (two per CU on 256 CUs, twice
// over) a gather takes 256-channel slabs.
constexpr int64_t kFewGroups = 1024;
// Fewest workgroups of the block gather (one per CU, two rounds).
constexpr int64_t kFewBlocks = 512;

// Workgroups of the 8 x 8 tiles that fill the chip (two on a CU, four rounds).
constexpr int64_t kFullTiles = 2048;

// Most candidates of a tile with which any unflagged map of a narrow Gaussian
// takes the independent waves.
constexpr double kWaveCand = 240.0;

// Which gather an FP32 map of more than 8 channels takes.  (Times in us of
// tiles / independent waves / blocks; 0.5' cells and FWHM 3' unless said.)
//   - Independent waves read a row once per cell block it reaches, up to 19
//     times, and keep all of their matrix work: up to 128 channels, or where
//     the spectra stay in the caches.  2M samples x 64 -> 400 x 400: 2549 /
//     1363 / 2716; x 128: 3174 / 2589 / 2842; x 256: 3858 / 4960 / 3767;
//     20,000 x 1024 -> 400 x 400 of 1.2': 500 / 327 / 533, 100,000: 628 / 591 /
//     753, 500,000: 1585 / 1778 / 1926.  Flagged, 2M x 64: 5790 / 2385 / 2514;
//     x 256: 7525 / 8442 / 5190.
//     The waves also win where a tile has few candidates, whatever the spectra's
//     size (their products stay full): 23,600 x 2048 -> 436 x 436 (45 a tile)
//     1176 / 768, 51,100 x 2048 -> 385 x 385 (110) 1034 / 768, 64,300 x 512 ->
//     424 x 424 (110) 318 / 248; 73,600 x 512 -> 256 x 256 (350) 194 / 178 but
//     99,700 x 2048 -> 329 x 329 (290) 1092 / 1145, 275,000 x 2048 -> 305 x 305
//     (930) 2019 / 2242.
//     Spectra in the caches, of more than 128 channels, and tiles to fill the
//     chip several times: the tiles lose nothing by their fill, and the waves'
//     weights, made anew for each 128 or 256 channels, count where they cost more
//     (FWHM 3', cells of 1.5', 400 x 400; candidates of a tile in brackets):
//     elliptical x 200 [6] 77 / 97, [178] 256 / 272, x 1024 [18] 364 / 482;
//     tapered sinc x 200 [6] 79 / 93, [56] 135 / 122; flagged x 200 [6] 82 / 103,
//     [53] 139 / 152, [178] 297 / 295; unflagged x 200 [6] 60 / 70, [56] 91 / 84,
//     x 256 [6] 72 / 76, x 1024 [6] 483 / 360.
//   - Blocks read a row 3.6 instead of 7.7 times and multiply at 2.7 times the
//     FP32 matrix rate (flags cost them a third more products, the others
//     twice as many), but in k-steps of 32 candidates, which a sparse map
//     fills badly: dense maps (pairs within R per cell) of many channels.
//     9.12M x 1024 -> 600 x 600 (5500 pairs per cell): 59700 / 97950 / 51000;
//     500,000 x 1024 -> 200 x 200 (2300): 4047 / 5094 / 3692; -> 400 x 400
//     (570): 3734 / 4237 / 4061.  Flagged, 500,000 x 256 -> 400 x 400 (570):
//     2081 / 2241 / 1744, 2M x 128 (2300): 7109 / 4299 / 3099.
//   - The tiles take a Gaussian's chords from the pair itself; the other two from
//     offsets to the middle of a block (centred_chords).
F32Kernel f32_kernel(const hcg_plan_s* p, int64_t C, bool mask) {
  if (p->kern.type == kGauss && !centred_chords(p)) return F32Kernel::kTile;
  const bool cached = (double)p->n * (double)C * 4.0 <= 100e6;
  const int64_t slab = mask ? kBlockSlabFlagged : kBlockSlab;
  const double c2R = support_chord2(p);
  const double pairs = p->bmaxr ? mean_pairs(p->n, p->grid, p->support_deg) : 0.0;
  const bool block = p->bmaxr && !cached &&
                     (mask ? C > 64 && pairs >= kBlockPairsFlagged
                           : C >= 512 && pairs >= kBlockPairs) &&
                     (int64_t)p->bntx * p->bnty * ((C + slab - 1) / slab) >= kFewBlocks;
  if (block) return F32Kernel::kBlock;
  const double load = p->load.mean;
  const int64_t tiles = (int64_t)p->ntx * p->nty;
  if (C > 128 && tiles * ((C + 255) / 256) >= kFullTiles &&
      (p->kern.type == kElliptic   ? true
       : p->kern.type == kSinc     ? mask || load < 40.0
       : mask                      ? load < 150.0
                                   : load < 20.0 && C <= 256))
    return F32Kernel::kTile;
  const bool sparse = load < kWaveCand && p->kern.type == kGauss && !mask &&
                      c2R < kNarrowChord2;
  return C <= 128 || cached || sparse ? F32Kernel::kWave : F32Kernel::kTile;
}

template <int kForm, bool kPacked = false, bool kMask = false>
static hcg_status launch_mfma(const hcg_plan_s* p, const void* spec, const void* spec_lo,
                              const float* scale, int64_t C, float* cube, float* wmap,
                              hipStream_t stream, float* wcube = nullptr) {
  static_assert(!(kPacked && kForm == kF32), "plan-ordered spectra are a low-precision input");
  if constexpr (kForm == kF32) {
    const F32Kernel k = f32_kernel(p, C, kMask);
    if (k == F32Kernel::kWave)
      return launch_wave(p, (const float*)spec, C, cube, wmap, wcube, kMask, stream);
    if (k == F32Kernel::kBlock)
      return launch_block(p, (const float*)spec, C, cube, wmap, wcube, kMask, stream);
  }
  GatherArgs a = plan_args(p);
  a.wcube = wcube;
  a.spec = spec;
  a.spec_lo = spec_lo;
  a.scale = scale;
  a.C = C;
  a.cube = cube;
  a.wmap = wmap;
  const size_t esz = (kForm == kF32) ? 4 : is_fp8(kForm) ? 1 : 2;
  if (kPacked && ((uintptr_t)spec % (8 * esz) != 0 || (uintptr_t)spec_lo % (8 * esz) != 0))
    return fail(HCG_E_ARG, "hcg_grid_packed: spectra must be %zu-byte aligned", 8 * esz);
  // plan-ordered spectra are read 8 samples of a channel at a time
  const bool vec = kPacked || ((C % 4 == 0) && ((uintptr_t)spec % (4 * esz) == 0) &&
                               (!spec_lo || (uintptr_t)spec_lo % (4 * esz) == 0));
  a.vec = vec ? 1 : 0;
  // 512-channel slabs (weights computed once per 512 channels) where the
  // registers allow it, else 256; a map of few tiles takes 256-channel slabs
  // too, for twice the workgroups (512-channel slabs would leave CUs idle)
  const int64_t groups512 = (int64_t)a.ntiles * ((C + 511) / 512);
  // the other kernel shapes and the flagged form keep to 256-channel slabs
  // (registers for the cell frame, or for the weight-sum accumulators)
  const bool gen = p->kern.type != kGauss;
  // supports below 0.57 deg (squared chord < 1e-4) take the kernels with the
  // short distance series
  const bool wide = !(a.c2R < kNarrowChord2);
  // the narrow-support 512-channel kernels of BF16, FP16 x scale and FP8 x
  // scale in input order read a row's channels eight at a time
  const bool rows8 = kPacked || wide || !(kForm == kBF16 || kForm == kF16S || kForm == kFP8S) ||
                     (C % 8 == 0 && (uintptr_t)spec % (8 * esz) == 0);
  const int qw = (C > 256 && vec && rows8 && kForm != kBF16Split && !gen && !kMask &&
                  groups512 >= kFewGroups) ? 2 : 1;
  const int64_t slab_ch = 256 * qw;
  const int64_t slabs = (C + slab_ch - 1) / slab_ch;
  const int64_t blocks = slabs * a.tiles_per_xcd * 8;
  if (blocks > INT32_MAX) return fail(HCG_E_UNSUPPORTED, "hcg_grid: too many channels");
  const dim3 grid((unsigned)blocks), block(256);
#define HCG_MFMA(QW, VEC)                                                                \
  do {                                                                                   \
    if (wide) k_gather_mfma<kForm, QW, VEC, kPacked, true><<<grid, block, 0, stream>>>(a); \
    else k_gather_mfma<kForm, QW, VEC, kPacked, false><<<grid, block, 0, stream>>>(a);    \
  } while (0)
  if (gen || kMask) {
    // one instance per form and row access: the general distance series,
    // 256-channel slabs
    if constexpr (kPacked) {
      k_gather_mfma<kForm, 1, true, true, true, true, false><<<grid, block, 0, stream>>>(a);
    } else if constexpr (kMask) {
      if (vec) {
        if (gen) k_gather_mfma<kForm, 1, true, false, true, true, true><<<grid, block, 0, stream>>>(a);
        else k_gather_mfma<kForm, 1, true, false, true, false, true><<<grid, block, 0, stream>>>(a);
      } else {
        if (gen) k_gather_mfma<kForm, 1, false, false, true, true, true><<<grid, block, 0, stream>>>(a);
        else k_gather_mfma<kForm, 1, false, false, true, false, true><<<grid, block, 0, stream>>>(a);
      }
    } else {
      if (vec) k_gather_mfma<kForm, 1, true, false, true, true, false><<<grid, block, 0, stream>>>(a);
      else k_gather_mfma<kForm, 1, false, false, true, true, false><<<grid, block, 0, stream>>>(a);
    }
    HCG_LAUNCH_CHECK("k_gather_mfma");
    return HCG_OK;
  }
  if constexpr (kForm != kBF16Split) {
    if (qw == 2) {
      HCG_MFMA(2, true);
      HCG_LAUNCH_CHECK("k_gather_mfma");
      return HCG_OK;
    }
  }
  if constexpr (kPacked) {
    HCG_MFMA(1, true);
  } else {
    if (vec) HCG_MFMA(1, true);
    else HCG_MFMA(1, false);
  }
#undef HCG_MFMA
  HCG_LAUNCH_CHECK("k_gather_mfma");
  return HCG_OK;
}

}  // namespace hcg

using namespace hcg;

namespace hcg {

// hcg_grid and hcg_grid_noalloc: the same kernels; noalloc forgoes the scratch in
// which the few-channel gather puts the values in the plan's order.
static hcg_status grid_dispatch(const char* where, hcg_plan_t plan, const void* spectra,
                                int64_t nchan, hcg_dtype dtype, const float* chan_scale,
                                float* cube, float* weights, void* hip_stream, bool noalloc) {
  if (!plan) return fail(HCG_E_ARG, "%s: plan is NULL", where);
  if (!plan_is_live(plan)) return fail(HCG_E_STATE, "%s: not a live plan", where);
  if (!spectra || !cube) return fail(HCG_E_ARG, "%s: spectra and cube must not be NULL", where);
  if (nchan < 1) return fail(HCG_E_ARG, "%s: nchan must be >= 1", where);
  const bool scaled = (dtype == HCG_F16_SCALED || dtype == HCG_FP8E4M3_SCALED ||
                       dtype == HCG_FP8E4M3_SPLIT);
  if (dtype < HCG_F32 || dtype > HCG_FP8E4M3_SPLIT)
    return fail(HCG_E_UNSUPPORTED, "%s: unknown dtype %d", where, (int)dtype);
  if (scaled && !chan_scale) return fail(HCG_E_ARG, "%s: chan_scale is required for this dtype", where);
  if (!scaled && chan_scale) return fail(HCG_E_ARG, "%s: chan_scale must be NULL for this dtype", where);
  const hcg_plan_s* p = plan;
  hipStream_t stream = (hipStream_t)hip_stream;
  switch (dtype) {
    case HCG_F32:
      if (nchan <= 8)
        return launch_cells(p, (const float*)spectra, (int)nchan, cube, weights, nullptr, false,
                            !noalloc, stream);
      return launch_mfma<kF32>(p, spectra, nullptr, nullptr, nchan, cube, weights, stream);
    case HCG_BF16:
      return launch_mfma<kBF16>(p, spectra, nullptr, nullptr, nchan, cube, weights, stream);
    case HCG_BF16_SPLIT:
      return launch_mfma<kBF16Split>(p, spectra,
                                     (const char*)spectra + (size_t)2 * p->n * nchan, nullptr,
                                     nchan, cube, weights, stream);
    case HCG_F16_SCALED:
      return launch_mfma<kF16S>(p, spectra, nullptr, chan_scale, nchan, cube, weights, stream);
    case HCG_FP8E4M3_SCALED:
      return launch_mfma<kFP8S>(p, spectra, nullptr, chan_scale, nchan, cube, weights, stream);
    case HCG_FP8E4M3_SPLIT:
      return launch_mfma<kFP8Split>(p, spectra, (const char*)spectra + (size_t)p->n * nchan,
                                    chan_scale, nchan, cube, weights, stream);
  }
  return fail(HCG_E_UNSUPPORTED, "%s: dtype %d", where, (int)dtype);
}

}  // namespace hcg

extern "C" hcg_status hcg_grid(hcg_plan_t plan, const void* spectra, int64_t nchan,
                               hcg_dtype dtype, const float* chan_scale, float* cube,
                               float* weights, void* hip_stream) {
  return grid_dispatch("hcg_grid", plan, spectra, nchan, dtype, chan_scale, cube, weights,
                       hip_stream, false);
}

extern "C" hcg_status hcg_grid_noalloc(hcg_plan_t plan, const void* spectra, int64_t nchan,
                                       hcg_dtype dtype, const float* chan_scale, float* cube,
                                       float* weights, void* hip_stream) {
  return grid_dispatch("hcg_grid_noalloc", plan, spectra, nchan, dtype, chan_scale, cube,
                       weights, hip_stream, true);
}

extern "C" hcg_status hcg_grid_masked(hcg_plan_t plan, const float* spectra, int64_t nchan,
                                      float* cube, float* chan_weights, void* hip_stream) {
  if (!plan) return fail(HCG_E_ARG, "hcg_grid_masked: plan is NULL");
  if (!plan_is_live(plan)) return fail(HCG_E_STATE, "hcg_grid_masked: not a live plan");
  if (!spectra || !cube) return fail(HCG_E_ARG, "hcg_grid_masked: spectra and cube must not be NULL");
  if (nchan < 1) return fail(HCG_E_ARG, "hcg_grid_masked: nchan must be >= 1");
  const hcg_plan_s* p = plan;
  hipStream_t stream = (hipStream_t)hip_stream;
  if (nchan <= 8)
    return launch_cells(p, spectra, (int)nchan, cube, nullptr, chan_weights, true, true,
                        stream);
  return launch_mfma<kF32, false, true>(p, spectra, nullptr, nullptr, nchan, cube, nullptr,
                                        stream, chan_weights);
}

extern "C" hcg_status hcg_packed_bytes(hcg_plan_t plan, int64_t nchan, hcg_dtype dtype,
                                       int64_t* bytes) {
  if (!plan || !bytes) return fail(HCG_E_ARG, "hcg_packed_bytes: NULL pointer");
  if (!plan_is_live(plan)) return fail(HCG_E_STATE, "hcg_packed_bytes: not a live plan");
  if (nchan < 1) return fail(HCG_E_ARG, "hcg_packed_bytes: nchan must be >= 1");
  int64_t esz = 0, planes = 1;
  switch (dtype) {
    case HCG_BF16: case HCG_F16_SCALED: esz = 2; break;
    case HCG_BF16_SPLIT: esz = 2; planes = 2; break;
    case HCG_FP8E4M3_SCALED: esz = 1; break;
    case HCG_FP8E4M3_SPLIT: esz = 1; planes = 2; break;
    default: return fail(HCG_E_ARG, "hcg_packed_bytes: dtype %d is not a low-precision form", (int)dtype);
  }
  const int64_t groups = (plan->n + 7) / 8;
  *bytes = planes * groups * 8 * ((nchan + 15) & ~int64_t(15)) * esz;
  return HCG_OK;
}

extern "C" hcg_status hcg_grid_packed(hcg_plan_t plan, const void* packed, int64_t nchan,
                                      hcg_dtype dtype, const float* chan_scale, float* cube,
                                      float* weights, void* hip_stream) {
  if (!plan) return fail(HCG_E_ARG, "hcg_grid_packed: plan is NULL");
  if (!plan_is_live(plan)) return fail(HCG_E_STATE, "hcg_grid_packed: not a live plan");
  if (!packed || !cube) return fail(HCG_E_ARG, "hcg_grid_packed: spectra and cube must not be NULL");
  if (nchan < 1) return fail(HCG_E_ARG, "hcg_grid_packed: nchan must be >= 1");
  const bool scaled = (dtype == HCG_F16_SCALED || dtype == HCG_FP8E4M3_SCALED ||
                       dtype == HCG_FP8E4M3_SPLIT);
  if (dtype < HCG_BF16 || dtype > HCG_FP8E4M3_SPLIT)
    return fail(HCG_E_ARG, "hcg_grid_packed: dtype %d is not a low-precision form", (int)dtype);
  if (scaled && !chan_scale) return fail(HCG_E_ARG, "hcg_grid_packed: chan_scale is required for this dtype");
  if (!scaled && chan_scale) return fail(HCG_E_ARG, "hcg_grid_packed: chan_scale must be NULL for this dtype");
  const hcg_plan_s* p = plan;
  hipStream_t stream = (hipStream_t)hip_stream;
  // elements per plane: 8 ceil(n / 8) sorted positions x nchan rounded up to 16
  const size_t plane = (size_t)((p->n + 7) / 8) * 8 * (size_t)((nchan + 15) & ~int64_t(15));
  const char* sp = (const char*)packed;
  switch (dtype) {
    case HCG_BF16:
      return launch_mfma<kBF16, true>(p, sp, sp, nullptr, nchan, cube, weights, stream);
    case HCG_BF16_SPLIT:
      return launch_mfma<kBF16Split, true>(p, sp, sp + 2 * plane, nullptr, nchan, cube, weights,
                                           stream);
    case HCG_F16_SCALED:
      return launch_mfma<kF16S, true>(p, sp, sp, chan_scale, nchan, cube, weights, stream);
    case HCG_FP8E4M3_SCALED:
      return launch_mfma<kFP8S, true>(p, sp, sp, chan_scale, nchan, cube, weights, stream);
    case HCG_FP8E4M3_SPLIT:
      return launch_mfma<kFP8Split, true>(p, sp, sp + plane, chan_scale, nchan, cube, weights,
                                          stream);
    default:
      break;
  }
  return fail(HCG_E_ARG, "hcg_grid_packed: dtype %d", (int)dtype);
}

extern "C" hcg_status hcg_get_plan_stats(hcg_plan_t plan, hcg_plan_stats* stats,
                                         void* hip_stream) {
  if (!plan || !stats) return fail(HCG_E_ARG, "hcg_get_plan_stats: NULL pointer");
  if (!plan_is_live(plan)) return fail(HCG_E_STATE, "hcg_get_plan_stats: not a live plan");
  const hcg_plan_s* p = plan;
  hipStream_t stream = (hipStream_t)hip_stream;
  const unsigned ntiles = (unsigned)(p->ntx * p->nty);
  unsigned long long* dcount = nullptr;
  HCG_HIP(hipMalloc(&dcount, sizeof(unsigned long long)));
  struct Free {
    void* q;
    ~Free() { (void)hipFree(q); }
  } fr{dcount};
  HCG_HIP(hipMemsetAsync(dcount, 0, sizeof(unsigned long long), stream));
  const GatherArgs a = plan_args(p);
  const size_t lds = sizeof(double4) * kKB + sizeof(uint2) * a.maxr + sizeof(uint32_t) * (a.maxr + 1);
  k_count_pairs<<<ntiles, 64, lds, stream>>>(a, dcount);
  HCG_LAUNCH_CHECK("k_count_pairs");
  unsigned long long pairs = 0;
  HCG_HIP(hipMemcpyAsync(&pairs, dcount, sizeof(pairs), hipMemcpyDeviceToHost, stream));
  std::vector<uint32_t> nc(ntiles);
  HCG_HIP(hipMemcpyAsync(nc.data(), p->ncand, sizeof(uint32_t) * ntiles, hipMemcpyDeviceToHost,
                         stream));
  HCG_HIP(hipStreamSynchronize(stream));
  int64_t cand = 0;
  for (uint32_t v : nc) cand += v;
  stats->pairs = (int64_t)pairs;
  stats->candidates = cand;
  stats->cells = (int64_t)p->grid.nx * p->grid.ny;
  return HCG_OK;
}
