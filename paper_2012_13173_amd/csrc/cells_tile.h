// Device code of the few-channel gather (FP32 spectra, C <= 8, FP64 sums),
// shared by the per-plan kernels (cells.hip) and the batch (batch.hip).
//
// A wave owns a sub-block of kNC cells of an 8 x 8 tile and walks the tile's
// candidate list 64 candidates at a time, one candidate per lane; every lane
// keeps its own FP64 sums of the kNC cells, which are added across lanes
// (and across the waves that share a sub-block) once, at the end.
//   - Consecutive candidates lie next to each other on the sky (they are
//     sorted by pixel), so 64 of them are mostly all within R of a cell or
//     none is: a cell costs three FMAs and a comparison where no lane hits,
//     and a chunk that misses the sub-block's circle costs one comparison.
//     (One lane per cell instead, with the candidates staged in LDS, spends
//     the full weight on every candidate that any of the 64 cells reaches:
//     8 % of the lanes did useful work on 90 x 90 cells of 200" with a 382"
//     support.)
//   - Candidates and cells are taken relative to the sub-block's centre c, so
//     |u - v|^2 = |u - c|^2 + |v - c|^2 - 2 (u - c).(v - c) is three FMAs per
//     pair; the terms are of the size of the squared distances themselves,
//     so nothing is lost to cancellation beyond a few units of the last
//     place of (block + R)^2.  (Where that is not small beside R^2, see
//     centred_chords, pairs pass with a margin for it and are then tested and
//     weighted by the chord of the difference.)
//   - No shared staging and no barrier inside the walk: each wave reads its
//     candidates from global memory two chunks ahead (the four sub-blocks of
//     a tile read the same lines), the values only of candidates inside the
//     sub-block's circle.
// 10^7 samples on 90 x 90 cells of 200" (FWHM 300", C = 1): 2780 us with one
// lane per cell and the lists split over workgroups, now 567 us (and
// 172 us to put the values in order);
// 1.98M samples on 400 x 400 cells of 0.5' (C = 4): 2118 -> 871 us.
#pragma once

#include <algorithm>

#include "hcg_internal.h"
#include "sphere.h"

namespace hcg {

// Weight sums per cell (one, or one per channel with flags), sums per cell,
// and cells per sub-block: 16 sums of two registers per lane at C = 1, and
// no more than about 80 registers of sums for any form but the flagged C = 8
// (whose 128 spilled beside the weights of the other kernel shapes, kGen: two
// cells there, 300,000 samples x 8 -> 150 x 150, tapered sinc: 2231 us with
// four, so 1111).  kFew: half the cells at C = 1, for wide circular Gaussians
// (whose registers leave two waves per SIMD with sixteen: 1.5M samples -> 400 x
// 400 of 5' 1159 us, so 1001; 50,000 -> 150 x 150 77 and 59) and for the other
// shapes on maps of few tiles (50,000 -> 40 x 40, tapered sinc: 180 us, so 105;
// 361 tiles the same, 2500 1.1 times as long).
template <int kCM, bool kMask, bool kGen = false, bool kFew = false>
struct CellsShape {
  static constexpr int kW = kMask ? kCM : 1;
  static constexpr int kS = kCM + kW;
  static constexpr int kNC = kS <= 2 ? (kFew ? 8 : 16) : kS <= 5 ? 8 : kGen && kS > 9 ? 2 : 4;
  static constexpr int kSubs = kTileCells / kNC;       // sub-blocks of a tile
  static constexpr int kSX = kNC == 16 ? 4 : kNC == 8 ? 4 : 2;  // cells of a sub-block in x
};

// LDS of a workgroup of `waves` waves serving `subs` sub-blocks: the tile's
// ranges, the cells' records and the waves' sums.
struct CellsRec {
  double mx, my, mz, thr;  // -2 (u - c); t <= thr <=> within R, t = |u - v|^2 - |u - c|^2
};
struct CellsGenRec {
  double ux, uy, uz;       // u - c
  CellFrame f;
};
template <int kNC, int kS, bool kGen>
__host__ __device__ constexpr size_t cells_lds_size(int waves, int subs, int maxr) {
  return sizeof(CellsRec) * kNC * subs + sizeof(double) * kNC * subs +
         (kGen ? sizeof(CellsGenRec) * kNC * subs : 0) + sizeof(double4) * subs +
         sizeof(double) * kNC * kS * waves + sizeof(uint2) * (size_t)maxr +
         sizeof(uint32_t) * ((size_t)maxr + 1);
}

// Loads the tile's ranges with exclusive prefix sums (first wave); returns
// the candidate count after a barrier.
__device__ inline uint32_t cells_stage_ranges(const uint2* __restrict__ ranges, uint32_t nr,
                                              uint2* s_rng, uint32_t* s_pre) {
  if (threadIdx.x < 64) {
    const int l = threadIdx.x;
    uint32_t acc = 0;
    for (uint32_t base = 0; base < nr; base += 64) {
      const uint32_t r = base + l;
      const uint2 v = r < nr ? ranges[r] : make_uint2(0u, 0u);
      uint32_t x = v.y - v.x;
      const uint32_t len = x;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, d);
        if (l >= d) x += y;
      }
      if (r < nr) {
        s_rng[r] = v;
        s_pre[r] = acc + x - len;
      }
      acc += (uint32_t)__shfl((int)x, 63);
    }
    if (l == 0) s_pre[nr] = acc;
  }
  __syncthreads();
  return s_pre[nr];
}

// Sorted position of candidate q < s_pre[nr]; *cur is a cursor that only
// moves forward: the next range is tried first (long ranges), then the rest
// is searched by bisection (a sparse field's ranges hold a few samples each).
__device__ __forceinline__ uint32_t cells_cand_pos(uint32_t q, const uint2* s_rng,
                                                   const uint32_t* s_pre, uint32_t nr,
                                                   uint32_t* cur) {
  uint32_t r = *cur;
  if (q >= s_pre[r + 1]) {
    uint32_t lo = r + 1, hi = nr - 1;  // the last range whose start is <= q
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (s_pre[mid] <= q) lo = mid; else hi = mid - 1;
    }
    r = lo;
    *cur = r;
  }
  return s_rng[r].x + (q - s_pre[r]);
}

// Sums of the lanes' values v[0 .. n): at each step a lane hands half of its
// values to its partner and adds the other half of the partner's, so that
// each value crosses lanes once per halving and ends in one lane: *at is its
// index, and *have > 0 tells that the lane holds one (n <= 64).
template <int n, int o, int kN>
__device__ __forceinline__ void cells_reduce(double (&v)[kN], int lane, int* at, int* have) {
  constexpr int half = (n + 1) / 2;
  const bool up = lane & o;
#pragma unroll
  for (int i = 0; i < half; ++i) {
    const double lo = v[i], hi = (i + half < n) ? v[(i + half < n) ? i + half : 0] : 0.0;
    const double got = __shfl_xor(up ? lo : hi, o);
    v[i] = (up ? hi : lo) + got;
  }
  *at += up ? half : 0;
  *have = up ? *have - half : min(*have, half);
  if constexpr (o > 1) cells_reduce<half, o / 2>(v, lane, at, have);
}

// Sub-blocks [sub0, sub0 + subs) of a tile by blockDim.x / 64 waves, nk waves
// for each (subs * nk = the waves): wave k of a sub-block takes every nk-th
// chunk of 64 candidates.  kWide = false: squared support chord below 1e-4
// and no weight below the normal floats (the launchers check both).  kExact:
// cells too far apart for centred_chords.
template <int kCM, bool kMask, bool kWide, bool kGen, bool kExact = false, bool kFew = false>
__device__ inline void cells_tile(const GatherArgs& a, int tile, int sub0, int subs, int nk,
                                  unsigned char* base) {
  using Sh = CellsShape<kCM, kMask, kGen, kFew>;
  constexpr int kNC = Sh::kNC, kW = Sh::kW, kS = Sh::kS, kSX = Sh::kSX, kSY = kNC / kSX;
  constexpr int kN = kNC * kS;
  static_assert(kN <= 64, "one sum per lane after the reduction");
  const int waves = subs * nk;
  CellsRec* s_rec = (CellsRec*)base;
  double4* s_ctr = (double4*)(s_rec + kNC * subs);
  CellsGenRec* s_gen = (CellsGenRec*)(s_ctr + subs);
  double* s_nu = (double*)(s_gen + (kGen ? kNC * subs : 0));
  double* s_red = s_nu + kNC * subs;
  uint2* s_rng = (uint2*)(s_red + kN * waves);
  uint32_t* s_pre = (uint32_t*)(s_rng + a.maxr);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = wave / nk, kslice = wave - sub * nk;
  const GridGeom& g = a.g;
  const int tx = tile % a.ntx, ty = tile / a.ntx;
  const int C = (int)a.C;

  // cells of the sub-block, lane i < kNC: cell i (x fastest)
  if (kslice == 0) {
    const int sx = (sub0 + sub) % (kTileX / kSX), sy = (sub0 + sub) / (kTileX / kSX);
    const int i = lane < kNC ? lane : 0;
    const int ix = tx * kTileX + sx * kSX + i % kSX, iy = ty * kTileY + sy * kSY + i / kSX;
    const CellVec u = cell_at(a.cells, g, ix, iy);
    const bool valid = lane < kNC && u.x == u.x;
    double sx_ = valid ? u.x : 0.0, sy_ = valid ? u.y : 0.0, sz_ = valid ? u.z : 0.0;
#pragma unroll
    for (int o = 1; o < kNC; o <<= 1) {
      sx_ += __shfl_xor(sx_, o);
      sy_ += __shfl_xor(sy_, o);
      sz_ += __shfl_xor(sz_, o);
    }
    const double nrm = sqrt(sx_ * sx_ + sy_ * sy_ + sz_ * sz_);
    // a sub-block of cells all over the sphere has no useful mean: any centre
    // serves, with a threshold that leaves nothing out
    const bool centred = nrm > 1e-6;
    const double cx = centred ? sx_ / nrm : 0.0, cy = centred ? sy_ / nrm : 0.0,
                 cz = centred ? sz_ / nrm : 1.0;
    const double ux = u.x - cx, uy = u.y - cy, uz = u.z - cz;
    const double nu = valid ? ux * ux + uy * uy + uz * uz : 0.0;
    double h2 = nu;
#pragma unroll
    for (int o = 1; o < kNC; o <<= 1) h2 = fmax(h2, __shfl_xor(h2, o));
    const bool any = __ballot(valid) != 0ull;
    if (lane < kNC) {
      double thr = a.c2R - nu;
      if constexpr (kExact) {  // t of a pair is off by at most 1.4e-15 of this square
        const double all = sqrt(a.c2R) + 2.0 * sqrt(h2);
        thr += 4e-15 * all * all;
      }
      s_rec[sub * kNC + i] = valid ? CellsRec{-2.0 * ux, -2.0 * uy, -2.0 * uz, thr}
                                   : CellsRec{0.0, 0.0, 0.0, -1e300};
      s_nu[sub * kNC + i] = nu;
      if constexpr (kGen)
        s_gen[sub * kNC + i] =
            CellsGenRec{ux, uy, uz,
                        a.kern.type == kElliptic ? cell_frame(u) : CellFrame{0.0, 0.0, 0.0, 0.0, 0.0}};
    }
    if (lane == 0) {
      // chords obey the triangle inequality: a sample within R of a cell is
      // within chord(R) + chord(h) of the centre; slack for rounding
      const double r = sqrt(a.c2R) + sqrt(h2);
      const double thr = !any ? -1.0 : centred ? r * r * (1.0 + 1e-9) + 1e-15 : 8.0;
      s_ctr[sub] = make_double4(cx, cy, cz, thr);
    }
  }
  const uint32_t nr = a.nranges[tile];
  const uint32_t total =
      cells_stage_ranges(a.ranges + (int64_t)tile * a.maxr, nr, s_rng, s_pre);
  const double4 ctr = s_ctr[sub];

  const double w0 = a.kern.wscale, w1 = w0 * (1.0 / 12.0), w2 = w0 * (1.0 / 90.0);
  double sum[kN];  // [cell][channels, then weights]
#pragma unroll
  for (int n = 0; n < kN; ++n) sum[n] = 0.0;

  const bool sorted = a.perm == nullptr;  // the values are in the plan's order
  const float* spec = (const float*)a.spec;
  const double* xyz = (const double*)a.xyz;
  // chunk j of this wave: candidates 64 (kslice + j nk) + lane.  Chunk j's
  // vectors and rows are loaded two chunks ahead, its values one ahead.
  uint32_t cur = 0;
  // All loads are unconditional (a lane past the last candidate reads the
  // last one and drops it at use; a lane outside the circle reads the row of
  // the chunk's first lane): after a load under a branch the compiler waits
  // for every load in flight, which undoes the prefetch.
  struct Vec { double x, y, z; };
  const uint32_t step = 64u * (uint32_t)nk;
  uint32_t q = 64u * (uint32_t)kslice + (uint32_t)lane;  // of the chunk to load next
  auto fetch = [&](Vec* v, uint32_t* row, bool* live) {
    *live = q < total;
    const uint32_t pos = cells_cand_pos(min(q, total - 1u), s_rng, s_pre, nr, &cur);
    const double2 xy = *(const double2*)(xyz + 4 * (size_t)pos);
    v->x = xy.x;
    v->y = xy.y;
    v->z = xyz[4 * (size_t)pos + 2];
    *row = sorted ? pos : a.perm[pos];
    q += step;
  };
  // relative to the centre; returns whether inside the sub-block's circle
  auto relative = [&](const Vec& v, bool live, Vec* d, double* nv) {
    d->x = live ? v.x - ctr.x : __builtin_nan("");
    d->y = v.y - ctr.y;
    d->z = v.z - ctr.z;
    *nv = d->x * d->x + d->y * d->y + d->z * d->z;
    return *nv <= ctr.w;  // false for NaN
  };
  auto values = [&](bool near, uint32_t row, float* s) {
    const uint32_t r = near ? row : (uint32_t)__builtin_amdgcn_readfirstlane((int)row);
    const float* rp = spec + (int64_t)r * C;
#pragma unroll
    for (int c = 0; c < kCM; ++c) s[c] = rp[(kCM == 1 || c < C) ? c : 0];
  };

  const uint32_t first = 64u * (uint32_t)kslice;
  const uint32_t nchunk = total > first ? (total - first + step - 1) / step : 0u;
  if (nchunk) {
    Vec v1, v2, d0, d1;
    uint32_t row1, row2;
    double nv0, nv1;
    float s0[kCM], s1[kCM];
    bool live1, live2;
    fetch(&v1, &row1, &live1);
    fetch(&v2, &row2, &live2);
    bool near0 = relative(v1, live1, &d0, &nv0);
    values(near0, row1, s0);
    for (uint32_t j = 0; j < nchunk; ++j) {
      v1 = v2;
      row1 = row2;
      live1 = live2;
      fetch(&v2, &row2, &live2);
      const bool near1 = relative(v1, live1, &d1, &nv1);
      values(near1, row1, s1);
      if (__ballot(near0)) {
        double sv[kCM];
        bool fine[kCM];
#pragma unroll
        for (int c = 0; c < kCM; ++c) {
          fine[c] = !kMask || (__float_as_uint(s0[c]) & 0x7F800000u) != 0x7F800000u;
          sv[c] = (double)s0[c];
        }
        // (lanes outside the circle hold finite or NaN vectors beyond every
        // threshold: no pair of theirs passes)
#pragma unroll
        for (int i = 0; i < kNC; ++i) {
          const CellsRec m = s_rec[sub * kNC + i];
          const double t = fma(m.mx, d0.x, fma(m.my, d0.y, fma(m.mz, d0.z, nv0)));
          if (t <= m.thr) {
            double c2 = t + s_nu[sub * kNC + i];  // down to -1 ulp of nu where u = v
            double w;
            if constexpr (kGen) {
              const CellsGenRec r = s_gen[sub * kNC + i];
              if constexpr (kExact) {
                const double dx = d0.x - r.ux, dy = d0.y - r.uy, dz = d0.z - r.uz;
                c2 = fma(dx, dx, fma(dy, dy, dz * dz));
                if (!(c2 <= a.c2R)) continue;
              }
              w = pair_weight_gen(a.kern, fmax(c2, 0.0), d0.x - r.ux, d0.y - r.uy, d0.z - r.uz, r.f);
            } else if constexpr (kWide) {
              w = pair_weight64(c2, a.kern.wscale);
            } else {
              // dist2_from_chord2<false>(c2) wscale with the factor in the series
              w = (double)__builtin_amdgcn_exp2f((float)(c2 * fma(c2, fma(c2, w2, w1), w0)));
            }
            if constexpr (kMask) {
#pragma unroll
              for (int c = 0; c < kCM; ++c)
                if (fine[c]) {
                  sum[i * kS + c] += w * sv[c];
                  sum[i * kS + kCM + c] += w;
                }
            } else {
#pragma unroll
              for (int c = 0; c < kCM; ++c) sum[i * kS + c] += w * sv[c];
              sum[i * kS + kCM] += w;
            }
          }
        }
      }
      d0 = d1;
      nv0 = nv1;
      near0 = near1;
#pragma unroll
      for (int c = 0; c < kCM; ++c) s0[c] = s1[c];
    }
  }

  {
    int at = 0, have = kN;
    cells_reduce<kN, 32>(sum, lane, &at, &have);
    if (have > 0) s_red[wave * kN + at] = sum[0];
  }
  __syncthreads();

  // one thread per cell: the waves' sums in order, V and W
  const int nth = (int)blockDim.x;
  const int64_t G = (int64_t)g.nx * g.ny;
  for (int t = (int)threadIdx.x; t < subs * kNC; t += nth) {
    const int sb = t / kNC, i = t - sb * kNC;
    const int sx = (sub0 + sb) % (kTileX / kSX), sy = (sub0 + sb) / (kTileX / kSX);
    const int ix = tx * kTileX + sx * kSX + i % kSX, iy = ty * kTileY + sy * kSY + i / kSX;
    if (ix >= g.nx || iy >= g.ny) continue;
    const double* red = s_red + (size_t)sb * nk * kN + i * kS;
    double wsum[kW], acc[kCM];
#pragma unroll
    for (int c = 0; c < kW; ++c) wsum[c] = 0.0;
#pragma unroll
    for (int c = 0; c < kCM; ++c) acc[c] = 0.0;
    for (int k = 0; k < nk; ++k) {
#pragma unroll
      for (int c = 0; c < kCM; ++c) acc[c] += red[k * kN + c];
#pragma unroll
      for (int c = 0; c < kW; ++c) wsum[c] += red[k * kN + kCM + c];
    }
    const int64_t cell = (int64_t)iy * g.nx + ix;
    if (!kMask && a.wmap) a.wmap[cell] = (float)wsum[0];
#pragma unroll
    for (int c = 0; c < kCM; ++c) {
      if (c >= C) continue;
      const double wc = wsum[kMask ? c : 0];
      a.cube[c * G + cell] = (wc != 0.0) ? (float)(acc[c] / wc) : __builtin_nanf("");
      if (kMask && a.wcube) a.wcube[c * G + cell] = (float)wc;
    }
  }
}

// A whole tile by one wave, one lane per cell: for tiles of few candidates,
// where the sums across lanes, the sub-blocks' frames and the walks of
// sixteen sub-blocks (cells_tile) cost more than the candidates do.  Every
// candidate is read once, by one lane, and handed to the others through LDS.
template <int kCM>
__host__ __device__ constexpr size_t cells_lane_lds_size(int maxr) {
  return (sizeof(double4) + sizeof(float) * kCM) * 64 + sizeof(uint2) * (size_t)maxr +
         sizeof(uint32_t) * ((size_t)maxr + 1);
}

template <int kCM, bool kMask, bool kWide, bool kGen>
__device__ inline void cells_lane(const GatherArgs& a, int tile, unsigned char* base) {
  constexpr int kW = CellsShape<kCM, kMask>::kW;
  double4* s_v = (double4*)base;
  float* s_s = (float*)(s_v + 64);
  uint2* s_rng = (uint2*)(s_s + 64 * kCM);
  uint32_t* s_pre = (uint32_t*)(s_rng + a.maxr);
  const int lane = threadIdx.x;
  const GridGeom& g = a.g;
  const int C = (int)a.C;
  const int ix = (tile % a.ntx) * kTileX + (lane & 7), iy = (tile / a.ntx) * kTileY + (lane >> 3);
  const CellVec u = cell_at(a.cells, g, ix, iy);  // NaN (no cell): within R of nothing
  CellFrame f{0.0, 0.0, 0.0, 0.0, 0.0};
  if constexpr (kGen) {
    if (a.kern.type == kElliptic) f = cell_frame(u);
  }
  const uint32_t nr = a.nranges[tile];
  const uint32_t total =
      cells_stage_ranges(a.ranges + (int64_t)tile * a.maxr, nr, s_rng, s_pre);
  const double w0 = a.kern.wscale, w1 = w0 * (1.0 / 12.0), w2 = w0 * (1.0 / 90.0);
  double acc[kCM], wsum[kW];
#pragma unroll
  for (int c = 0; c < kCM; ++c) acc[c] = 0.0;
#pragma unroll
  for (int c = 0; c < kW; ++c) wsum[c] = 0.0;

  uint32_t cur = 0;
  for (uint32_t q0 = 0; q0 < total; q0 += 64) {
    const uint32_t pos = cells_cand_pos(min(q0 + lane, total - 1u), s_rng, s_pre, nr, &cur);
    const double4 v = a.xyz[pos];
    const float* row = (const float*)a.spec + (int64_t)(a.perm ? a.perm[pos] : pos) * C;
    float s[kCM];
#pragma unroll
    for (int c = 0; c < kCM; ++c) s[c] = row[(kCM == 1 || c < C) ? c : 0];
    __syncthreads();  // the last chunk has been used
    s_v[lane] = v;
#pragma unroll
    for (int c = 0; c < kCM; ++c) s_s[lane * kCM + c] = s[c];
    __syncthreads();
    const int m = (int)min(64u, total - q0);
#pragma unroll 4
    for (int k = 0; k < m; ++k) {
      const double dx = s_v[k].x - u.x, dy = s_v[k].y - u.y, dz = s_v[k].z - u.z;
      const double c2 = fma(dx, dx, fma(dy, dy, dz * dz));
      if (c2 <= a.c2R) {
        double w;
        if constexpr (kGen) w = pair_weight_gen(a.kern, c2, dx, dy, dz, f);
        else if constexpr (kWide) w = pair_weight64(c2, a.kern.wscale);
        else w = (double)__builtin_amdgcn_exp2f((float)(c2 * fma(c2, fma(c2, w2, w1), w0)));
#pragma unroll
        for (int c = 0; c < kCM; ++c) {
          const float x = s_s[k * kCM + c];
          if (kMask && (__float_as_uint(x) & 0x7F800000u) == 0x7F800000u) continue;
          acc[c] += w * (double)x;
          if (kMask) wsum[kMask ? c : 0] += w;
        }
        if (!kMask) wsum[0] += w;
      }
    }
  }
  if (ix >= g.nx || iy >= g.ny) return;
  const int64_t G = (int64_t)g.nx * g.ny, cell = (int64_t)iy * g.nx + ix;
  if (!kMask && a.wmap) a.wmap[cell] = (float)wsum[0];
#pragma unroll
  for (int c = 0; c < kCM; ++c) {
    if (c >= C) continue;
    const double wc = wsum[kMask ? c : 0];
    a.cube[c * G + cell] = (wc != 0.0) ? (float)(acc[c] / wc) : __builtin_nanf("");
    if (kMask && a.wcube) a.wcube[c * G + cell] = (float)wc;
  }
}

// Whether a Gaussian plan's few-channel weights can take the short distance
// series and the hardware exponential alone: narrow support, and the
// exponent at R above the smallest normal float's.
__host__ inline bool cells_narrow(double c2R, const KernelParams& k) {
  return c2R < kNarrowChord2 && k.wscale * c2R * (1.0 + c2R) > -125.0;
}

// Whether a plan's tiles are taken by one wave each (cells_lane), kCM channels.
// In us: a wave takes `wave` per candidate; a full chip `lane` 1e-5 per candidate
// of a tile by lanes, and by sub-blocks `tile` per tile (their frames and sums)
// and `sub` 1e-5 per candidate, `walk` at least.  Circular Gaussian, fitted to 23 maps of 25 to
// 5544 tiles of 2 to 64,000 candidates.  Sub-blocks / lanes: 2500 tiles, C = 1:
// 52 candidates 26 / 12, 208: 39 / 33, 416: 52 / 57; C = 8: 52: 97 / 17, 416: 177
// / 84; 323 tiles of 651, C = 8: 42 / 91; 64 of 231, C = 4: 9 / 30; 5544 of 2, C
// = 8: 170 / 9; wide supports (whose sub-blocks keep two waves per SIMD), C = 8,
// 2500 tiles of 970: 592 / 371, of 4850: 2149 / 1684; C = 4, of 970: 400 / 326,
// flagged 569 / 481, of 4850 2097 / 2243.  The other shapes' weights
// cost several times as much, and by sub-blocks as the cells that a candidate
// reaches, `hits` of a tile's; fitted to 192 maps of 25 to 2500 tiles: elliptical,
// 2500 tiles, C = 1: 160 candidates 159 / 112, 300: 183 / 205, 1530: 584 / 896;
// 361 tiles of 100, C = 8: 41 / 58; tapered sinc 47 / 78.
__host__ inline bool cells_by_lane(const hcg_plan_s* p, int kCM, bool mask) {
  const double n = (double)p->ntx * p->nty, sums = mask ? 2.0 * kCM : kCM + 1.0;
  double wave = 0.11, lane = 4.8 + 0.5 * kCM;
  double tile = 0.005 + 0.0042 * kCM, sub = 2.3 + 0.5 * kCM, walk = 2.0;
  const double R = p->support_rad, reach = 0.8 * p->tile_span + 2.0 * R;
  const double hits = 3.9 * R * R / (reach * reach);
  if (p->kern.type != kGauss) {
    const double subs = sums <= 2.0 ? 4.0 : sums <= 5.0 ? 8.0 : sums <= 9.0 ? 16.0 : 32.0;
    const bool sinc = p->kern.type == kSinc;
    wave = (sinc ? 0.47 : 0.31) + 0.0085 * sums;
    lane = (sinc ? 34.0 : 19.5) + 0.65 * sums;
    tile = (sinc ? 0.0034 : 0.0023) * subs;
    sub = (sinc ? 14.0 : 4.8) + 0.65 * sums + 31.0 * hits;
    walk = 2.0 + 1.4 * sums;
  } else if (!cells_narrow(support_chord2(p), p->kern)) {
    if (kCM == 4) {
      wave = mask ? 0.22 : 0.17;
      lane = mask ? 18.5 : 11.8;
      tile = mask ? 0.055 : 0.033;
      sub = mask ? 7.5 + 23.0 * hits : 5.7 + 16.5 * hits;
    } else if (kCM == 8 && !mask) {
      wave = 0.2;
      lane = 14.0;
      sub = 18.0;
    }
  }
  const double cand = 1e-5 * p->load.mean * n;
  return std::max(wave * p->load.most, lane * cand) < tile * n + sub * cand + walk;
}

}  // namespace hcg
