// Matrix-core gather of FP32 spectra by independent waves: a wave owns one 4 x
// 4 cell block and 16 kJ channels.
//
// The block kernels (gather_tile.h) multiply every group of four listed
// candidates that holds one within reach of a cell block, so a sparse map
// pays for candidates that reach nothing (a few samples per square of R: under
// a tenth of the products were pairs within R), and a wave there owns 64
// channels of all four cell blocks, so that a cube of 64 channels keeps one
// wave of four at work.  Here a wave
//   - tests 64 candidates at a time against its cell block's circle (radius R
//     + h, one comparison) and packs those inside into a queue in LDS, so
//     that every product group of four is full: pairs within R are R^2 / (R +
//     h)^2 of the products whatever the density;
//   - computes the weights of 64 packed candidates straight into the matrix
//     operand's registers (lane: cell lane % 16, candidate 4 s + lane / 16),
//     three FMAs per squared chord: with u and v relative to the cell block's
//     centre c in a frame whose third axis is c, |u - v|^2 = -2 ux vx - 2 uy vy
//     - (2 + 2 uz) vz + |u - c|^2, vz = -|v - c|^2 / 2 (unit vectors);
//   - multiplies them with v_mfma_f32_16x16x4_f32, its rows loaded kDepth
//     product groups ahead;
// with no barrier until the end.  What bounds it is the matrix rate at that
// fill; rows are read once per cell block instead of once per tile, so the
// large dense cubes whose rows leave the caches stay with the block kernels.
// Measured (8 x 8 tiles before): 20,000 samples x 67 channels -> 45 x 37 of 0.75'
// 333 -> 41 us; 500,000 x 64 -> 256 x 240 projected cells, elliptical beam, with
// its plan 1210 -> 858 us.
#pragma once

#include "cells_tile.h"
#include "gather_tile.h"

namespace hcg {

constexpr int kWaveQueue = 128;  // packed candidates per wave (two batches of 64)

struct WaveQueue {
  double x[kWaveQueue], y[kWaveQueue], z[kWaveQueue];  // relative to c (third: see above)
  int64_t row[kWaveQueue];                             // byte offset of the spectrum
  double frame[10];                                    // c, e1, e2, threshold
};

// LDS of a workgroup of `waves` waves, nk of them on each cell block.  The
// partial sums of nk > 1 waves take the queues' place.
template <int kJ, bool kMask>
__host__ __device__ constexpr size_t wave_lds_bytes(int waves, int nk, int maxr) {
  const size_t q = sizeof(WaveQueue) * waves;
  const size_t acc = nk > 1 ? sizeof(float) * 64 * 4 * kJ * (kMask ? 2 : 1) * (waves / 2) : 0;
  return (q > acc ? q : acc) + sizeof(double) * 2 * 16 * waves + sizeof(uint2) * (size_t)maxr +
         sizeof(uint32_t) * ((size_t)maxr + 1);
}

// Product groups whose rows are in flight.
template <int kJ, bool kMask>
constexpr int kWaveDepth = kJ <= 4 ? 6 : 4;

// Cell blocks sub0 .. sub0 + subs - 1 of a tile by subs * nk waves, channels 16 kJ
// slab ..: wave k of a cell block takes every nk-th chunk of 64 candidates.
// kVec: a lane's channels of a row are read four at a time.
template <int kJ, bool kVec, bool kMask, bool kWide, bool kGen>
__device__ __forceinline__ void gather_wave(const GatherArgs& a, int tile, int slab, int sub0,
                                            int subs, int nk, unsigned char* lds) {
  constexpr int kDepth = kWaveDepth<kJ, kMask>;
  constexpr int kH = kVec ? kJ / 4 : kJ;  // loads of a row per lane
  const int waves = subs * nk;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = wave / nk, kslice = wave - sub * nk;
  const int li = lane & 15, lg = lane >> 4;
  const GridGeom& g = a.g;
  const int64_t C = a.C;
  const int64_t G = (int64_t)g.nx * g.ny;

  constexpr size_t kAccBytes = sizeof(float) * 64 * 4 * kJ * (kMask ? 2 : 1);
  const size_t qbytes = sizeof(WaveQueue) * waves;
  const size_t abytes = nk > 1 ? kAccBytes * (waves / 2) : 0;
  double* s_w = (double*)(lds + (qbytes > abytes ? qbytes : abytes));  // [waves][2][16]
  uint2* s_rng = (uint2*)(s_w + 2 * 16 * waves);
  uint32_t* s_pre = (uint32_t*)(s_rng + a.maxr);
  WaveQueue& Q = ((WaveQueue*)lds)[wave];

  // ---- the cell block: lane's cell u, frame at the mean of the cells
  const int cb = sub0 + sub;
  const int x0 = tile % a.ntx * kTileX + (cb & 1) * 4, y0 = tile / a.ntx * kTileY + (cb >> 1) * 4;
  const int my_x = x0 + (li & 3), my_y = y0 + (li >> 2);
  const CellVec u = cell_at(a.cells, g, my_x, my_y);
  const bool valid = u.x == u.x;
  double cx = valid ? u.x : 0.0, cy = valid ? u.y : 0.0, cz = valid ? u.z : 0.0;
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    cx += __shfl_xor(cx, o);
    cy += __shfl_xor(cy, o);
    cz += __shfl_xor(cz, o);
  }
  const double nrm = sqrt(cx * cx + cy * cy + cz * cz);
  const bool centred = nrm > 1e-6;  // else the cells are all over the sphere: any centre serves
  cx = centred ? cx / nrm : 0.0;
  cy = centred ? cy / nrm : 0.0;
  cz = centred ? cz / nrm : 1.0;
  double e1x, e1y, e1z;  // unit vector across c
  if (fabs(cz) < 0.9) {
    const double r = 1.0 / sqrt(cx * cx + cy * cy);
    e1x = -cy * r; e1y = cx * r; e1z = 0.0;
  } else {
    const double r = 1.0 / sqrt(cy * cy + cz * cz);
    e1x = 0.0; e1y = -cz * r; e1z = cy * r;
  }
  const double e2x = cy * e1z - cz * e1y, e2y = cz * e1x - cx * e1z, e2z = cx * e1y - cy * e1x;
  const double ux = u.x - cx, uy = u.y - cy, uz = u.z - cz;
  const double nu = valid ? ux * ux + uy * uy + uz * uz : 0.0;
  double h2 = nu;
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) h2 = fmax(h2, __shfl_xor(h2, o));
  const bool any = __ballot(valid) != 0ull;
  const double rr = sqrt(a.c2R) + sqrt(h2);
  const double thr = !any ? -1.0 : centred ? rr * rr * (1.0 + 1e-9) + 1e-15 : 8.0;
  // Gaussian: chord operand of the cell; other shapes: its offset and frame
  const double bx = kGen ? ux : valid ? -2.0 * (ux * e1x + uy * e1y + uz * e1z) : 0.0;
  const double by = kGen ? uy : valid ? -2.0 * (ux * e2x + uy * e2y + uz * e2z) : 0.0;
  const double bz = kGen ? uz : -2.0 + nu;
  const double bw = valid ? nu : 1e30;  // no cell: beyond every candidate
  const CellFrame frame = kGen ? cell_frame(u) : CellFrame{0.0, 0.0, 0.0, 0.0, 0.0};
  const double w0 = a.kern.wscale, w1 = a.kern.kmaj, w2 = a.kern.kmin;  // Gaussian: w0 / 12, w0 / 90
  if (lane == 0) {  // (read back per chunk: registers)
    const double f[10] = {cx, cy, cz, e1x, e1y, e1z, e2x, e2y, e2z, thr};
#pragma unroll
    for (int k = 0; k < 10; ++k) Q.frame[k] = f[k];
  }

  const uint32_t nr = a.nranges[tile];
  const uint32_t total =
      cells_stage_ranges(a.ranges + (int64_t)tile * a.maxr, nr, s_rng, s_pre);

  floatx4 acc[kJ], accw[kMask ? kJ : 1];
#pragma unroll
  for (int j = 0; j < kJ; ++j) {
    acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    if constexpr (kMask) accw[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  double wsum = 0.0;

  // channels: kVec 64 h + 4 li + q, else 16 j + li, from c_w on (offsets from
  // there fit 32 bits whatever the channel count); a lane past the last channel
  // reads the slab's first ones (those products are not stored)
  const int64_t c_w = (int64_t)slab * (16 * kJ);
  const int jlive = (int)min<int64_t>(kJ, kVec ? (C - c_w + 63) / 64 * 4 : (C - c_w + 15) / 16);
  int32_t off[kH];
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    const int64_t ch = c_w + (kVec ? 64 * h + 4 * li : 16 * h + li);
    off[h] = ch < C ? (int32_t)(4 * (ch - c_w)) : 0;
  }
  const char* spec = (const char*)a.spec + 4 * c_w;
  float bb[kDepth][kJ];
  auto load = [&](int q0, int s, int set) {
    const char* rp = spec + Q.row[q0 + 4 * s + lg];
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      if constexpr (kVec) {
        const floatx4 v = *(const floatx4*)(rp + off[h]);
#pragma unroll
        for (int q = 0; q < 4; ++q) bb[set][4 * h + q] = v[q];
      } else {
        bb[set][h] = *(const float*)(rp + off[h]);
      }
    }
  };

  // One batch: the 64 queue entries from q0, of which the first 4 ns count.
  auto batch = [&](int q0, int ns) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) load(q0, d, d);
    float w[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int e = q0 + 4 * s + lg;
      const double vx = Q.x[e], vy = Q.y[e], vz = Q.z[e];
      float x = 0.f;
      if constexpr (kGen) {
        const double dx = vx - bx, dy = vy - by, dz = vz - bz;
        const double c2 = dx * dx + dy * dy + dz * dz;
        if (c2 <= a.c2R) x = (float)pair_weight_gen(a.kern, c2, dx, dy, dz, frame);
      } else {
        const double c2 = fma(bx, vx, fma(by, vy, fma(bz, vz, bw)));
        if constexpr (kWide) {
          if (c2 <= a.c2R) x = pair_weight<true>(c2, w0);
        } else {
          // dist2_from_chord2<false>(c2) wscale, the factor inside the series
          const float ex = __builtin_amdgcn_exp2f((float)(c2 * fma(c2, fma(c2, w2, w1), w0)));
          x = c2 <= a.c2R ? ex : 0.f;
        }
      }
      // (kept here: sunk to its product, every weight would hold its chord in
      // registers instead)
      asm volatile("" : "+v"(x));
      w[s] = x;
      wsum += (double)x;
      // four at a time: all sixteen interleaved would take the registers
      if (s % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      if (s < ns) {
        float b[kJ], m[kMask ? kJ : 1];
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
          b[j] = bb[s % kDepth][j];
          if constexpr (kMask) {
            const bool fin = (__float_as_uint(b[j]) & 0x7F800000u) != 0x7F800000u;
            m[j] = fin ? 1.f : 0.f;
            b[j] = fin ? b[j] : 0.f;
          }
        }
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
          if (j % 4 && kVec ? j / 4 * 4 >= jlive : j >= jlive) continue;
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], b[j], acc[j], 0, 0, 0);
          if constexpr (kMask)
            accw[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], m[j], accw[j], 0, 0, 0);
        }
      }
      if (s + kDepth < 16) load(q0, s + kDepth, s % kDepth);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- walk: chunk after chunk of 64 candidates, the next one in flight
  const uint32_t step = 64u * (uint32_t)nk;
  uint32_t q = 64u * (uint32_t)kslice + (uint32_t)lane;
  uint32_t cur = 0, head = 0, count = 0;
  struct Vec { double x, y, z; };
  auto fetch = [&](Vec* v, uint32_t* row) {
    const uint32_t pos = cells_cand_pos(min(q, total - 1u), s_rng, s_pre, nr, &cur);
    const double* p = (const double*)(a.xyz + pos);
    v->x = p[0];
    v->y = p[1];
    v->z = p[2];
    *row = a.perm[pos];
    q += step;
  };
  const int64_t row_bytes = 4 * C;
  const uint32_t first = 64u * (uint32_t)kslice;
  const uint32_t nchunk = total > first && any ? (total - first + step - 1) / step : 0u;
  if (nchunk) {
    Vec v, vn;
    uint32_t row, rown;
    fetch(&vn, &rown);
    for (uint32_t j = 0; j < nchunk; ++j) {
      v = vn;
      row = rown;
      const bool in = q - step < total;  // of the chunk in v
      fetch(&vn, &rown);
      const double* F = Q.frame;
      const double dx = v.x - F[0], dy = v.y - F[1], dz = v.z - F[2];
      const double nv = dx * dx + dy * dy + dz * dz;
      const bool near = in && nv <= F[9];
      const uint64_t b = __ballot(near);
      if (near) {
        const uint32_t at = (head + count + (uint32_t)__builtin_amdgcn_mbcnt_hi(
                                                (uint32_t)(b >> 32),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))) %
                            kWaveQueue;
        Q.x[at] = kGen ? dx : dx * F[3] + dy * F[4] + dz * F[5];
        Q.y[at] = kGen ? dy : dx * F[6] + dy * F[7] + dz * F[8];
        Q.z[at] = kGen ? dz : -0.5 * nv;
        Q.row[at] = (int64_t)row * row_bytes;
      }
      count += (uint32_t)__popcll(b);
      if (count >= 64u) {
        batch((int)head, 16);
        head = (head + 64u) % kWaveQueue;
        count -= 64u;
      }
    }
    if (count) {
      // the last, partial batch: padded with candidates within R of no cell
      // (NaN: any finite place in the chord's expanded form is close to some
      // cell more than 90 degrees from c), on the first one's row
      const uint32_t at = (head + (uint32_t)lane) % kWaveQueue;
      const int64_t r0 = Q.row[head];
      if ((uint32_t)lane >= count) {
        Q.x[at] = Q.y[at] = Q.z[at] = __builtin_nan("");
        Q.row[at] = r0;
      }
      batch((int)head, (int)((count + 3u) / 4u));
    }
  }

  // ---- sums over the four lanes of a cell, and over the waves of a cell block
  wsum += __shfl_xor(wsum, 16);
  wsum += __shfl_xor(wsum, 32);
  if (nk > 1) {
    __syncthreads();  // the queues are free
    float* s_acc = (float*)lds;
    if (lane < 16) s_w[wave * 16 + lane] = wsum;
    // halves fold onto halves: wave k + n of a cell block onto wave k
    for (int n = nk / 2; n > 0; n /= 2) {
      const int slot = sub * (nk / 2) + (kslice - n);
      if (kslice >= n && kslice < 2 * n) {
        float* out = s_acc + (size_t)slot * (kAccBytes / 4) + lane;
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            out[(4 * j + r) * 64] = acc[j][r];
            if constexpr (kMask) out[(4 * (kJ + j) + r) * 64] = accw[j][r];
          }
      }
      __syncthreads();
      if (kslice < n) {
        const float* in = s_acc + (size_t)(sub * (nk / 2) + kslice) * (kAccBytes / 4) + lane;
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            acc[j][r] += in[(4 * j + r) * 64];
            if constexpr (kMask) accw[j][r] += in[(4 * (kJ + j) + r) * 64];
          }
      }
      __syncthreads();
    }
    if (kslice > 0) return;  // (a persistent workgroup meets at its own barrier)
    wsum = 0.0;
    for (int k = 0; k < nk; ++k) wsum += s_w[(sub * nk + k) * 16 + li];
  }
  if (!kMask && a.wmap && slab == 0 && lane < 16 && my_x < g.nx && my_y < g.ny)
    a.wmap[(int64_t)my_y * g.nx + my_x] = (float)wsum;

  // ---- V: lane li holds its channels of cells (x0 .. x0 + 3, y0 + lg)
  const int y = y0 + lg;
  float inv[4];
  bool has[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double wt = __shfl(wsum, 4 * lg + r);
    has[r] = wt != 0.0;
    inv[r] = has[r] ? (float)(1.0 / wt) : 0.f;
  }
  if (y >= g.ny || x0 >= g.nx) return;
  const float qnan = __builtin_nanf("");
  const int64_t at = (int64_t)y * g.nx + x0;
  const bool full = x0 + 3 < g.nx;
#pragma unroll
  for (int j = 0; j < kJ; ++j) {
    const int64_t ch = c_w + (kVec ? 64 * (j >> 2) + 4 * li + (j & 3) : 16 * j + li);
    if (ch >= C) continue;
    float v[4], wc[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (kMask) {
        wc[r] = accw[j][r];
        v[r] = (wc[r] != 0.f) ? acc[j][r] / wc[r] : qnan;
      } else {
        v[r] = has[r] ? acc[j][r] * inv[r] : qnan;
      }
    }
    float* dst = a.cube + ch * G + at;
    float* wdst = kMask && a.wcube ? a.wcube + ch * G + at : nullptr;
    if (full) {
      store4(dst, v);
      if (kMask && wdst) store4(wdst, wc);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (x0 + r < g.nx) {
          dst[r] = v[r];
          if (kMask && wdst) wdst[r] = wc[r];
        }
    }
  }
}

}  // namespace hcg
