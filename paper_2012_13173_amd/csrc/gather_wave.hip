// Launches of the independent-wave gather (gather_wave.h) on one plan.
#include <algorithm>

#include "batch_items.h"
#include "gather_wave.h"

namespace hcg {

// Waves per SIMD that a kernel's registers are held to.
template <int kJ, bool kMask, bool kGen>
constexpr int kWaveOccupancy = kGen || kJ == 16 ? 2 : kJ * (kMask ? 2 : 1) <= 4 ? 3 : 2;

template <int kJ, bool kVec, bool kMask, bool kWide, bool kGen>
__global__ void __launch_bounds__(256, (kWaveOccupancy<kJ, kMask, kGen>)) k_gather_wave(const GatherArgs a, int subs, int nk) {
  extern __shared__ __align__(16) unsigned char s_dyn[];
  // one slab after the other; within one, the XCDs (workgroups go to them in
  // turn) take contiguous eighths of the cell blocks
  const int per_tile = 4 / subs;
  const uint32_t work = (uint32_t)a.ntiles * per_tile, eighth = (work + 7) / 8;
  const uint32_t at = wide_block(), slab = __builtin_amdgcn_readfirstlane(at / (8 * eighth));
  const uint32_t b = at - slab * 8 * eighth, w = (b & 7) * eighth + (b >> 3);
  if (w >= work || (int64_t)slab * (16 * kJ) >= a.C) return;
  const int tile = __builtin_amdgcn_readfirstlane(w / per_tile);
  gather_wave<kJ, kVec, kMask, kWide, kGen>(a, tile, (int)slab, (int)(w - tile * per_tile) * subs,
                                            subs, nk, s_dyn);
}

template <int kJ, bool kVec, bool kMask, bool kWide, bool kGen>
static hcg_status launch(const GatherArgs& a, int nk, hipStream_t stream) {
  const int subs = nk > 1 ? 1 : 4;
  const int64_t work = (int64_t)a.ntiles * (4 / subs);
  const int64_t blocks = (work + 7) / 8 * 8 * ((a.C + 16 * kJ - 1) / (16 * kJ));
  if (blocks > INT32_MAX) return fail(HCG_E_UNSUPPORTED, "hcg_grid: too many channels");
  const size_t lds = wave_lds_bytes<kJ, kMask>(subs * nk, nk, a.maxr);
  k_gather_wave<kJ, kVec, kMask, kWide, kGen>
      <<<wide_grid(blocks), 64 * subs * nk, lds, stream>>>(a, subs, nk);
  HCG_LAUNCH_CHECK("k_gather_wave");
  return HCG_OK;
}

template <bool kVec, bool kMask, bool kWide, bool kGen>
static hcg_status launch_j(const GatherArgs& a, int j, int nk, hipStream_t stream) {
  if (j == 4) return launch<4, kVec, kMask, kWide, kGen>(a, nk, stream);
  // (rows read one channel at a time: sixteen loads of a row would spill)
  if constexpr (!kMask && kVec)
    if (j == 16) return launch<16, kVec, kMask, kWide, kGen>(a, nk, stream);
  return launch<8, kVec, kMask, kWide, kGen>(a, nk, stream);
}

hcg_status launch_wave(const hcg_plan_s* p, const float* spec, int64_t C, float* cube, float* wmap,
                       float* wcube, bool mask, hipStream_t stream) {
  GatherArgs a = plan_args(p);
  if (p->kern.type == kGauss) {  // the series factors, in fields a Gaussian leaves unused
    a.kern.kmaj = a.kern.wscale * (1.0 / 12.0);
    a.kern.kmin = a.kern.wscale * (1.0 / 90.0);
  }
  a.spec = spec;
  a.C = C;
  a.cube = cube;
  a.wmap = wmap;
  a.wcube = wcube;
  const bool vec = C % 4 == 0 && (uintptr_t)spec % 16 == 0;
  const bool gen = p->kern.type != kGauss, wide = !(a.c2R < kNarrowChord2);
  const WaveShape sh = wave_shape(p, C, vec, mask);
#define HCG_WAVE(MASK, WIDE, GEN)                                       \
  (vec ? launch_j<true, MASK, WIDE, GEN>(a, sh.j, sh.nk, stream)         \
       : launch_j<false, MASK, WIDE, GEN>(a, sh.j, sh.nk, stream))
  if (mask) return gen ? HCG_WAVE(true, true, true) : HCG_WAVE(true, true, false);
  if (gen) return HCG_WAVE(false, true, true);
  return wide ? HCG_WAVE(false, true, false) : HCG_WAVE(false, false, false);
#undef HCG_WAVE
}

// Channels of a wave and waves of a cell block (times in us, 0.5' to 1.5' cells,
// FWHM 3').  Wide slabs compute the weights less often; 256 channels leave half
// of the waves of 128, so they are for maps that have kWaveFew waves all the
// same (four per SIMD), and not for the elliptical weights, whose registers
// spill there (200 channels -> 150 x 150, 1444 cell blocks: 82 with 128
// channels a wave, 92 with 256; 120 with 64).  A map of very few takes 64
// channels, and so does a flagged circular Gaussian one, whose weights cost
// least (1444 blocks: 46, 50 with 128).  Four waves to a cell block shorten its
// walk where few cell blocks have many candidates (20,000 x 67 -> 45 x 37: 335
// with one workgroup per 8 x 8 tile, 42 so; 1444 blocks, elliptical, 128
// channels: 1150 candidates a tile 140 with one, 128 with four; 115: 28 and 49).
constexpr int64_t kWaveFew = 4096, kWaveVeryFew = 256;
WaveShape wave_shape(const hcg_plan_s* p, int64_t C, bool vec, bool mask) {
  const int64_t blocks = 4 * (int64_t)p->ntx * p->nty;
  auto waves = [&](int j) { return blocks * ((C + 16 * j - 1) / (16 * j)); };
  int j = C <= 64 ? 4 : C <= 128 || mask || !vec || p->kern.type == kElliptic ? 8 : 16;
  if (j == 16 && waves(j) < kWaveFew) j = 8;
  const int64_t least = mask && p->kern.type == kGauss ? kWaveFew : kWaveVeryFew;
  if (j == 8 && waves(j) < least) j = 4;
  const bool split = waves(j) < kWaveFew && p->load.most >= std::max(128.0, 0.6 * (double)waves(j));
  return WaveShape{j, split ? 4 : 1};
}

// ---------------------------------------------------------------------------
// Fields of a batch.  A unit is a tile, or with several waves to a cell block a
// cell block; a workgroup of four waves takes one unit of one channel slab.
// ---------------------------------------------------------------------------
// (One call of gather_wave, on arguments copied to registers: a call for each
// case, on arguments read where they are used, took twice the registers and
// left half the waves -- eight fields of 1 to 2048 channels 1214 us, not 813.)
template <int kJ, bool kVec, bool kWide>
__device__ __forceinline__ void wave_unit(const GatherArgs& a, uint32_t unit, uint32_t slab,
                                          unsigned char* lds) {
  const bool split = a.vec > 1;
  gather_wave<kJ, kVec, false, kWide, false>(a, (int)(split ? unit >> 2 : unit), (int)slab,
                                             split ? (int)(unit & 3u) : 0, split ? 1 : 4, a.vec,
                                             lds);
}

template <int kJ, bool kVec, bool kWide>
__global__ void __launch_bounds__(256, (kWaveOccupancy<kJ, false, false>)) k_wave_items(const GatherArgs* __restrict__ fields,
                                                       const BatchSeg* __restrict__ segs,
                                                       uint32_t nseg, uint32_t nitems) {
  extern __shared__ __align__(16) unsigned char s_dyn[];
  const uint32_t it = wide_block();
  if (it >= nitems) return;
  const BatchSeg sg = batch_seg_of(segs, nseg, it);
  const uint32_t local = it - sg.base;
  const GatherArgs a = fields[sg.field];
  const uint32_t per_slab = (uint32_t)a.tiles_per_xcd * 8u;
  const uint32_t slab = local / per_slab, loc = local - slab * per_slab;
  const uint32_t unit = (loc & 7u) * (uint32_t)a.tiles_per_xcd + (loc >> 3);
  if (unit < (uint32_t)a.ntiles) wave_unit<kJ, kVec, kWide>(a, unit, slab, s_dyn);
}

template <int kJ, bool kVec, bool kWide>
__global__ void __launch_bounds__(256, 2) k_wave_batch(const GatherArgs* __restrict__ fields,
                                                       const BatchSeg* __restrict__ segs,
                                                       uint32_t* __restrict__ ctl) {
  extern __shared__ __align__(16) unsigned char s_dyn[];
  __shared__ uint32_t s_item;
  const uint32_t total = ctl[8], nseg = ctl[9];
  const int home = (int)(blockIdx.x % kBatchXcds);
  int k = 0;
  for (;;) {
    const uint32_t it = batch_next_item(ctl, total, home, &k, &s_item);
    if (it == 0xFFFFFFFFu) break;
    const BatchSeg sg = batch_seg_of(segs, nseg, it);
    const uint32_t local = it - sg.base, slab = local / sg.ntiles;
    const GatherArgs a = fields[sg.field];
    wave_unit<kJ, kVec, kWide>(a, local - slab * sg.ntiles, slab, s_dyn);
    __syncthreads();
  }
}

void launch_wave_items(int j, bool vec, bool wide, bool items, uint32_t blocks,
                       const GatherArgs* fields, const BatchSeg* segs, uint32_t nseg,
                       uint32_t* ctl, int maxr, hipStream_t stream) {
#define HCG_ITEMS(J, VEC, WIDE)                                                                   \
  do {                                                                                            \
    const size_t a = wave_lds_bytes<J, false>(4, 1, maxr), b = wave_lds_bytes<J, false>(4, 4, maxr); \
    const size_t lds = a > b ? a : b;                                                             \
    if (items) k_wave_items<J, VEC, WIDE><<<wide_grid(blocks), 256, lds, stream>>>(fields, segs, nseg, blocks); \
    else k_wave_batch<J, VEC, WIDE><<<blocks, 256, lds, stream>>>(fields, segs, ctl);             \
  } while (0)
#define HCG_ITEMS_W(J, VEC)             \
  do {                                  \
    if (wide) HCG_ITEMS(J, VEC, true);  \
    else HCG_ITEMS(J, VEC, false);      \
  } while (0)
  if (j == 4) {
    if (vec) HCG_ITEMS_W(4, true);
    else HCG_ITEMS_W(4, false);
  } else {
    if (vec) HCG_ITEMS_W(8, true);
    else HCG_ITEMS_W(8, false);
  }
#undef HCG_ITEMS_W
#undef HCG_ITEMS
}

}  // namespace hcg
