// Matrix-core gather of a block of kT x kT cell blocks (16 cells each: 16 x 16
// output cells for kT = 4) x one channel slab, for narrow supports and the
// circular Gaussian.
//
// What bounds the many-channel gather is the spectrum rows: every tile reads
// all rows within R of it, so the bytes go as ((tile + 2R) / tile)^2 (7.7 times
// the spectra for 8 x 8 cells of 0.5' and R = 3.8', 3.6 times for 16 x 16), and
// FP32 products on the FP32 matrix instruction take as long again.  Here
//   - a workgroup of eight waves owns 16 x 16 cells x 256 channels (128 with
//     flags), the accumulators taking half of a CU's registers: wave w holds
//     channels 32 w .. of all sixteen cell blocks;
//   - FP32 operands are split into three BF16 pieces (round to nearest even:
//     x = hi + mid + lo exactly, 24 bits, for |x| from 2^-110 to the largest
//     BF16) and multiplied by six v_mfma_f32_16x16x32_bf16 (hi.hi, hi.mid,
//     mid.hi, mid.mid, hi.lo, lo.hi, smallest first).  The dropped terms are
//     below 2^-26 of a product, the accumulator rounds once per 32 candidates
//     instead of once per 4: the error against 64 bits is no larger than with
//     v_mfma_f32_16x16x4_f32 (largest per-channel relative L2 of the two maps
//     below: 9.4e-7 and 6.9e-7, both 1.2e-6 with that), at 2.7 times its rate.
//     BF16 has FP32's exponents, so below 2^-110 the last piece runs into the
//     smallest number, 2^-133 (spectra of 1e-36 would be off by 3.7e-5): a
//     block that meets such values runs a second time on values times 2^64
//     and takes its small results from there; larger and non-finite values
//     are dealt with in convert() as well;
//   - squared chords come from v_mfma_f64_16x16x4_f64: with cells u and
//     candidates v relative to the block's centre c in a frame whose third
//     axis is c, |u - v|^2 = -2 ux vx - 2 uy vy - (2 + 2 uz) vz + |u - c|^2 with
//     vz = -|v - c|^2 / 2 -- four terms, one instruction for 16 cells x 16
//     candidates, whose output layout hands every lane the eight candidates
//     of its cell that the BF16 operand wants;
//   - candidates go through in groups of up to four k-steps of 32 (as many
//     as have sixteen marked fragments in all), a barrier each: while a
//     group is multiplied, the weights of the next are computed, one
//     fragment (cell block x k-step, those that a coarse test marks) after
//     the other dealt to the waves; half of the waves multiply first and half
//     prepare first, so that the two waves of a SIMD use different units.
// It measured 59.4 -> 50.7 ms (9.12M samples x 1024 -> 600 x 600 of 0.5', FWHM
// 3') and, flagged, 4.63 -> 3.05 ms (1.14M x 256 -> 300 x 300).  What
// bounds it now: 18 ms of matrix and 21 ms of vector instructions, which the
// two waves of a SIMD overlap only in part, and the barriers.
#pragma once

#include <type_traits>

#include "gather_tile.h"

namespace hcg {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kStep = 32;      // candidates of a k-step (the K of the 16-bit MFMAs)
constexpr int kGroup = 4;      // k-steps of a group at most (16 bits of a mask each)
constexpr int kRing = 8;       // staged blocks of 64 candidates (two k-steps) in LDS

// Two floats to packed BF16, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t d) { return __uint_as_float(d << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t d) { return __uint_as_float(d & 0xFFFF0000u); }

// The three BF16 pieces of two floats.  *rest: what the first two leave of a and
// b together: NaN exactly when a piece is not finite (a or b non-finite, or
// beyond the largest BF16); at most 2^-127 and not 0 where the third piece is
// not exact (below 2^-110; larger values leave 0 or multiples of 2^-133 that it
// holds).
__device__ __forceinline__ void split3(float a, float b, uint32_t* hi, uint32_t* mid, uint32_t* lo,
                                       float* rest) {
  const uint32_t h = pk_bf16(a, b);
  const float a1 = a - bf16_lo(h), b1 = b - bf16_hi(h);
  const uint32_t m = pk_bf16(a1, b1);
  const float a2 = a1 - bf16_lo(m), b2 = b1 - bf16_hi(m);
  *hi = h;
  *mid = m;
  *lo = pk_bf16(a2, b2);
  *rest = a2 + b2;
}

// Passes over the candidates after the first: see gather_block's convert().
constexpr int kPassSmall = 1, kPassPos = 2, kPassNeg = 3;

// Fragments (cell block x k-step) of a group's weights in LDS, twice.
constexpr int kSlots = 16;

template <int kT>
struct BlockSmem {
  static constexpr int kCB = kT * kT;
  uint4 A[2][kSlots][3][64];       // pieces of the weights
  double ws[2][kSlots][64];        // weight sums of a fragment
  double cell[kCB][64];            // chord operand of the cells
  double xyz[kRing][3][72];        // chord operand of the candidates, 64 used
  int64_t row[kRing][64];          // byte offsets of the rows
  double4 ctr[kCB];                // coarse test: -2 c, |c|^2 - threshold
  uint2 rng[kMaxRangesLimit];
  uint32_t pre[kMaxRangesLimit + 1];
  uint32_t nrng;
  uint32_t odd;                    // a non-finite value was left out of the products
  uint32_t small;                  // a value's pieces were not exact
  uint32_t mark[2 * kRing];        // marked cell blocks of the staged k-steps
  double mean[8][4];
  double frame[12];                // c, e1, e2
  double Wt[kCB * 16];
};

// One (block of cells, channel slab); all 64 kWaves threads take part.  a is
// as block_args makes it.
template <int kT, int kWaves, int kJ, bool kVec, bool kMask>
__device__ __forceinline__ void gather_block(const GatherArgs& a, int tile, int slab,
                                             BlockSmem<kT>& sm) {
  constexpr int kCB = kT * kT;
  constexpr int kOwn = (kCB + kWaves - 1) / kWaves;  // cell blocks whose weights a wave sums

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const int tx = tile % a.ntx, ty = tile / a.ntx;
  const GridGeom& g = a.g;
  const int64_t C = a.C;
  const int64_t G = (int64_t)g.nx * g.ny;
  const int x0 = tx * 4 * kT, y0 = ty * 4 * kT;

  const uint32_t total =
      stage_ranges<true>(a.ranges + (int64_t)tile * a.maxr, a.nranges[tile], sm.rng, sm.pre,
                         0u, &sm.nrng);
  const uint32_t nrng = sm.nrng;

  // ---- frame of the block and the cells in it (threads 0 .. 16 kCB - 1)
  CellVec u{0.0, 0.0, 0.0};
  bool valid = false;
  if (tid < 16 * kCB) {
    const int cb = tid >> 4, i = tid & 15;
    u = cell_at(a.cells, g, x0 + (cb % kT) * 4 + (i & 3), y0 + (cb / kT) * 4 + (i >> 2));
    valid = u.x == u.x;
    double sx = valid ? u.x : 0.0, sy = valid ? u.y : 0.0, sz = valid ? u.z : 0.0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      sx += __shfl_xor(sx, o);
      sy += __shfl_xor(sy, o);
      sz += __shfl_xor(sz, o);
    }
    if (lane == 0) {
      sm.mean[wave][0] = sx;
      sm.mean[wave][1] = sy;
      sm.mean[wave][2] = sz;
    }
  }
  __syncthreads();
  double cx = 0.0, cy = 0.0, cz = 0.0;
#pragma unroll
  for (int w = 0; w < kCB / 4; ++w) {
    cx += sm.mean[w][0];
    cy += sm.mean[w][1];
    cz += sm.mean[w][2];
  }
  {
    const double n = sqrt(cx * cx + cy * cy + cz * cz);
    const bool ok = n > 1e-6;  // else the cells are all over the sphere: any centre serves
    cx = ok ? cx / n : 0.0;
    cy = ok ? cy / n : 0.0;
    cz = ok ? cz / n : 1.0;
  }
  // e1, e2: unit vectors across c (from the axis that c is far from)
  double e1x, e1y, e1z;
  if (fabs(cz) < 0.9) {
    const double r = 1.0 / sqrt(cx * cx + cy * cy);
    e1x = -cy * r; e1y = cx * r; e1z = 0.0;
  } else {
    const double r = 1.0 / sqrt(cy * cy + cz * cz);
    e1x = 0.0; e1y = -cz * r; e1z = cy * r;
  }
  const double e2x = cy * e1z - cz * e1y, e2y = cz * e1x - cx * e1z, e2z = cx * e1y - cy * e1x;
  if (tid < 16 * kCB) {
    const int cb = tid >> 4, i = tid & 15;
    const double dx = u.x - cx, dy = u.y - cy, dz = u.z - cz;
    const double ux = valid ? dx * e1x + dy * e1y + dz * e1z : 0.0;
    const double uy = valid ? dx * e2x + dy * e2y + dz * e2z : 0.0;
    const double nu = valid ? dx * dx + dy * dy + dz * dz : 0.0;
    // a cell without a centre, or outside the grid: beyond every candidate
    sm.cell[cb][i] = -2.0 * ux;
    sm.cell[cb][16 + i] = -2.0 * uy;
    sm.cell[cb][32 + i] = -2.0 + nu;
    sm.cell[cb][48 + i] = valid ? nu : 1e30;
    // the cell block's mean point and the largest distance of its cells: a
    // candidate within R of a cell is within R + h of the mean (chords)
    double mx = ux, my = uy, mz = -0.5 * nu, cnt = valid ? 1.0 : 0.0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      mx += __shfl_xor(mx, o);
      my += __shfl_xor(my, o);
      mz += __shfl_xor(mz, o);
      cnt += __shfl_xor(cnt, o);
    }
    const double inv = cnt > 0.0 ? 1.0 / cnt : 0.0;
    mx *= inv;
    my *= inv;
    mz *= inv;
    double h2 = valid ? (ux - mx) * (ux - mx) + (uy - my) * (uy - my) +
                            (-0.5 * nu - mz) * (-0.5 * nu - mz)
                      : 0.0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) h2 = fmax(h2, __shfl_xor(h2, o));
    const double r = sqrt(a.c2R) + sqrt(h2);
    const double thr = r * r * (1.0 + 1e-9) + 1e-15;
    if (i == 0)
      sm.ctr[cb] = make_double4(-2.0 * mx, -2.0 * my, -2.0 - 2.0 * mz,
                                cnt > 0.0 ? mx * mx + my * my + mz * mz - thr : 1e30);
  }

  if (tid == 0) {
    const double f[9] = {cx, cy, cz, e1x, e1y, e1z, e2x, e2y, e2z};
#pragma unroll
    for (int k = 0; k < 9; ++k) sm.frame[k] = f[k];
  }

  if (tid == 0) sm.odd = sm.small = 0u;
  int pass = 0;  // kPassSmall, kPassPos, kPassNeg: see convert()
  floatx4 acc[kCB][kJ];
  floatx4 accw[kMask ? kCB : 1][kMask ? kJ : 1];  // flagged form: channel weight sums
  double wsum[kOwn];

  // channels of this wave: lane i holds channels kJ i .. kJ i + kJ - 1 of them
  const int64_t c_w = (int64_t)slab * (kWaves * 16 * kJ) + wave * (16 * kJ);
  const bool live = c_w < C;  // a wave past the last channel still computes weights

  // ---- staging: blocks of 64 candidates (two steps), by the waves in turn.
  // Padding past the last candidate takes the last one's row (see gather_tile)
  // and a NaN position, within R of no cell and marked by no coarse test (a
  // finite one in this frame is close to some cell more than 90 degrees from
  // c).  In the FP64 product a candidate is a row of its own.
  auto cand = [&](uint32_t q) -> uint32_t {
    uint32_t lo = 0, hi = nrng - 1;
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (sm.pre[mid] <= q) lo = mid; else hi = mid - 1;
    }
    return sm.rng[lo].x + (q - sm.pre[lo]);
  };
  // (k-steps past the last candidate are all padding and unmarked)
  const uint32_t nk = (total + kStep - 1) / kStep;
  double nx = 0.0, ny = 0.0, nz = 0.0;
  uint32_t nrow = 0u;
  const int64_t row_bytes = C * 4;
  auto fetch = [&](uint32_t blk) {
    const uint32_t pos = cand(min(64u * blk + lane, total - 1u));
    const double4 v = a.xyz[pos];
    nx = v.x;
    ny = v.y;
    nz = v.z;
    nrow = a.perm[pos];
  };
  auto stage = [&](uint32_t blk) {
    const int buf = blk % kRing;
    const bool in = 64u * blk + lane < total;
    const double* F = sm.frame;
    const double dx = nx - F[0], dy = ny - F[1], dz = nz - F[2];
    const double vx = dx * F[3] + dy * F[4] + dz * F[5];
    const double vy = dx * F[6] + dy * F[7] + dz * F[8];
    double vz = -0.5 * (dx * dx + dy * dy + dz * dz);
    vz = in ? vz : __builtin_nan("");
    sm.xyz[buf][0][lane] = vx;
    sm.xyz[buf][1][lane] = vy;
    sm.xyz[buf][2][lane] = vz;
    sm.row[buf][lane] = (int64_t)nrow * row_bytes;
    if (lane < 2) sm.mark[2 * buf + lane] = 0u;
  };
  // coarse test of a staged block (a barrier after it is staged): each wave
  // marks the k-steps that can hold a pair with its own cell blocks
  auto coarse = [&](uint32_t blk) {
    const int buf = blk % kRing;
    const double vx = sm.xyz[buf][0][lane], vy = sm.xyz[buf][1][lane], vz = sm.xyz[buf][2][lane];
    uint32_t m0 = 0, m1 = 0;
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      const int cb = wave + o * kWaves;
      if (cb >= kCB) break;
      const double4 c = sm.ctr[cb];
      const uint64_t bm = __ballot(fma(c.x, vx, fma(c.y, vy, fma(c.z, vz, c.w))) <= 0.0);
      m0 |= ((uint32_t)bm ? 1u : 0u) << cb;
      m1 |= ((uint32_t)(bm >> 32) ? 1u : 0u) << cb;
    }
    if (lane == 0 && (m0 | m1)) {
      atomicOr(&sm.mark[2 * buf], m0);
      atomicOr(&sm.mark[2 * buf + 1], m1);
    }
  };
  // The group that begins at k-step k: as many k-steps (below kend) as have at
  // most kSlots marked fragments in all, one at least.  *bits: the marked cell
  // blocks, kCB bits a k-step.
  auto group = [&](uint32_t k, uint32_t kend, uint64_t* bits) -> uint32_t {
    const int kk = lane / kCB;  // lane: (k-step, cell block)
    const uint32_t m = sm.mark[(k + (kk < kGroup ? kk : 0)) % (2 * kRing)];
    uint64_t B = __ballot(kk < kGroup && k + kk < kend && ((m >> (lane % kCB)) & 1u));
    uint32_t n = 1;
#pragma unroll
    for (int g = 1; g < kGroup; ++g)
      if (k + g < kend && __popcll(B & ((2ull << (kCB * (g + 1) - 1)) - 1ull)) <= kSlots) n = g + 1;
    *bits = B & ((2ull << (kCB * n - 1)) - 1ull);
    return k + n;
  };

  // ---- weights of a group: its fragments dealt to the waves in turn
  const double w0 = a.kern.wscale, w1 = a.kern.kmaj, w2 = a.kern.kmin;  // scalars: w0 / 12, w0 / 90
  auto weights = [&](uint32_t k, uint64_t bits, int ab) {
    const int cnt = __popcll(bits);
    const bool set = (bits >> lane) & 1ull;
    const int mine = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0u));
    const int at = 8 * (li & 3) + (li >> 2);
    for (int f = (wave + (int)(k >> 1)) % kWaves; f < cnt; f += kWaves) {
      const int bit = (int)__builtin_ctzll(__ballot(set && mine == f));
      const int cb = bit % kCB;
      const uint32_t ks = k + bit / kCB;
      const double* x = sm.xyz[(ks >> 1) % kRing][lg < 3 ? lg : 0] + kStep * (ks & 1) + at;
      const double b = sm.cell[cb][lane];
      doublex4 d[2];
#pragma unroll
      for (int h = 0; h < 2; ++h)
        d[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(lg < 3 ? x[4 * h] : 1.0, b,
                                                    doublex4{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
      float w[8];
      double sum = 0.0;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const double c2 = d[t >> 2][t & 3];
        // dist2_from_chord2<false>(c2) wscale, the factor inside the series
        const float e = (float)(c2 * fma(c2, fma(c2, w2, w1), w0));
        const float x = __builtin_amdgcn_exp2f(e);
        w[t] = c2 <= a.c2R ? x : 0.f;
        sum += (double)w[t];
      }
      sm.ws[ab][f][lane] = sum;
      uint32_t hi[4], mid[4], lo[4];
      float rest;
#pragma unroll
      for (int p = 0; p < 4; ++p) split3(w[2 * p], w[2 * p + 1], &hi[p], &mid[p], &lo[p], &rest);
      sm.A[ab][f][0][lane] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      sm.A[ab][f][1][lane] = make_uint4(mid[0], mid[1], mid[2], mid[3]);
      sm.A[ab][f][2][lane] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    }
  };

  // ---- spectra of a k-step into registers: 8 rows x kJ channels per lane
  // (unconditional: a lane past the last channel reads the row's first ones,
  // see gather_tile)
  float raw[8][kJ];
  const int64_t ch0 = c_w + kJ * li;
  const char* base = (const char*)a.spec + 4 * (kVec && ch0 + kJ > C ? 0 : ch0);
  auto load = [&](uint32_t k) {
    const int64_t* rows = sm.row[(k >> 1) % kRing] + kStep * (k & 1) + 8 * lg;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const char* rp = base + rows[t];
      if constexpr (kVec) {
        static_assert(kJ == 2, "two channels in one load");
        const floatx2 v = *(const floatx2*)rp;
        raw[t][0] = v.x;
        raw[t][1] = v.y;
      } else {
#pragma unroll
        for (int j = 0; j < kJ; ++j) raw[t][j] = *(const float*)(rp + (ch0 + j < C ? 4 * j : -4 * ch0));
      }
    }
  };

  // the loaded rows as BF16 pieces (and flags)
  uint4 bh[kJ], bm[kJ], bl[kJ], fl[kMask ? kJ : 1];
  auto convert = [&](auto first) {
    if constexpr (!first()) {
      const uint32_t other = pass == kPassPos ? 0xFF800000u : 0x7F800000u;  // -inf, +inf
#pragma unroll
      for (int j = 0; j < kJ; ++j)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const float x = raw[t][j];
          const uint32_t u = __float_as_uint(x);
          const bool fin = (u & 0x7F800000u) != 0x7F800000u;
          // (a value that 2^64 takes past 2^127 stays finite: its cells keep
          // what the first pass gave them)
          const float big = __builtin_amdgcn_fmed3f(x * 0x1p64f, -0x1p127f, 0x1p127f);
          raw[t][j] = pass == kPassSmall ? (fin ? big : kMask ? x : 0.f)
                                         : (!fin && u != other ? 1.f : 0.f);
        }
    }
    // rest of each channel: a small sum shows where no larger value's hides it
    float rest[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
      rest[j] = 0.f;
      uint32_t h[4], m[4], l[4], k[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float va = raw[2 * p][j], vb = raw[2 * p + 1][j], r;
        if constexpr (kMask) {
          // flags: a non-finite value becomes 0 in the product and 0 in the
          // channel's weight operand (BF16 1.0 = 0x3F80)
          const bool fa = (__float_as_uint(va) & 0x7F800000u) != 0x7F800000u;
          const bool fb = (__float_as_uint(vb) & 0x7F800000u) != 0x7F800000u;
          k[p] = (fa ? 0x3F80u : 0u) | (fb ? 0x3F800000u : 0u);
          va = fa ? va : 0.f;
          vb = fb ? vb : 0.f;
        }
        split3(va, vb, &h[p], &m[p], &l[p], &r);
        rest[j] += r;
      }
      bh[j] = make_uint4(h[0], h[1], h[2], h[3]);
      bm[j] = make_uint4(m[0], m[1], m[2], m[3]);
      bl[j] = make_uint4(l[0], l[1], l[2], l[3]);
      if constexpr (kMask) fl[j] = make_uint4(k[0], k[1], k[2], k[3]);
    }
    // Values without exact pieces are rare.  One that is not finite, or beyond
    // the largest BF16: those steps split by truncation (exact for every finite
    // value from 2^-110 on) with the non-finite values left out; two further
    // passes over the candidates (kPassPos, kPassNeg) then find the cells
    // within R of a sample that is +inf or NaN, and -inf or NaN.  One below
    // 2^-110: a further pass multiplies values times 2^64 (kPassSmall).
    bool special = false;
#pragma unroll
    for (int j = 0; j < kJ; ++j) special |= __builtin_amdgcn_classf(rest[j], 0x093);  // NaN, subnormal
    if (first() && __builtin_expect(__ballot(special) != 0ull, 0)) {
      bool nan = false, tiny = false;
#pragma unroll
      for (int j = 0; j < kJ; ++j) {
        nan |= rest[j] != rest[j];
        tiny |= __builtin_amdgcn_classf(rest[j], 0x090);
      }
      if (__ballot(tiny)) sm.small = 1u;
      if (__ballot(nan)) {
        asm volatile("; split by truncation");
        bool lost = false;
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
          uint32_t H[4], M[4], L[4];
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            H[p] = M[p] = L[p] = 0u;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const float x = raw[2 * p + e][j];
              const bool fin = (__float_as_uint(x) & 0x7F800000u) != 0x7F800000u;
              lost = lost || !fin;
              const float v = fin ? x : 0.f;
              const uint32_t hb = __float_as_uint(v) & 0xFFFF0000u;
              const float r1 = v - __uint_as_float(hb);
              const uint32_t mb = __float_as_uint(r1) & 0xFFFF0000u;
              const uint32_t lb = __float_as_uint(r1 - __uint_as_float(mb)) & 0xFFFF0000u;
              H[p] |= hb >> (e ? 0 : 16);
              M[p] |= mb >> (e ? 0 : 16);
              L[p] |= lb >> (e ? 0 : 16);
            }
          }
          bh[j] = make_uint4(H[0], H[1], H[2], H[3]);
          bm[j] = make_uint4(M[0], M[1], M[2], M[3]);
          bl[j] = make_uint4(L[0], L[1], L[2], L[3]);
        }
        if (!kMask && __ballot(lost) && lane == 0) sm.odd = 1u;
      }
    }
  };

  // k-steps k .. kn - 1, whose weights are in buffer ab; starts the loads of
  // the next k-step
  auto products = [&](uint32_t k, uint32_t kn, uint64_t bits, int ab, auto first) {
    // the weight sums of this wave's own cell blocks
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      const int cb = wave + o * kWaves;
      if (cb >= kCB) break;
      uint64_t own = bits;
      if constexpr (kCB == 16) own &= 0x0001000100010001ull << cb;
      else own &= 0x1111ull << cb;
      while (own) {
        const int bit = (int)__builtin_ctzll(own);
        own &= own - 1ull;
        const int f = __popcll(bits & ((1ull << bit) - 1ull));
        wsum[o] += sm.ws[ab][f][lane];
      }
    }
    if (!live) bits = 0ull;
    uint4 nh, nm, nl;  // weights of the next fragment, read while one is multiplied
    uint32_t slot = 0;
    auto read = [&](uint32_t f) {
      f = min(f, (uint32_t)kSlots - 1u);
      nh = sm.A[ab][f][0][lane];
      nm = sm.A[ab][f][1][lane];
      nl = sm.A[ab][f][2][lane];
    };
    read(0);
    auto mm = [](const uint4& x, const uint4& y, const floatx4& z) {
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x),
                                                     __builtin_bit_cast(bf16x8, y), z, 0, 0, 0);
    };
#pragma nounroll
    for (; k < kn; ++k) {
      convert(first);
      load(k + 1);
      const uint32_t mask = (uint32_t)bits & ((1u << kCB) - 1u);
      bits >>= kCB;
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        if (!((mask >> cb) & 1u)) continue;
        const uint4 ah = nh, am = nm, al = nl;
        read(++slot);
        // (the kJ chains take turns: a product waits for the one before it
        // on the same accumulator)
#pragma unroll
        for (int p = 0; p < 6; ++p)
#pragma unroll
          for (int j = 0; j < kJ; ++j) {
            const uint4& x = p == 0 ? al : p == 2 || p == 3 ? am : ah;
            const uint4& y = p == 1 ? bl[j] : p == 2 || p == 4 ? bm[j] : bh[j];
            acc[cb][j] = mm(x, y, acc[cb][j]);
            if constexpr (kMask)
              if (p < 3) accw[cb][j] = mm(p == 0 ? al : p == 1 ? am : ah, fl[j], accw[cb][j]);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  auto walk = [&](auto first) {
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb)
#pragma unroll
      for (int j = 0; j < kJ; ++j) {
        acc[cb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (kMask) accw[cb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
    for (int o = 0; o < kOwn; ++o) wsum[o] = 0.0;

    // ---- pipeline, a barrier per group: group i is multiplied while the weights
    // of group i + 1 are computed, blocks staged before the last barrier are
    // tested and blocks up to kRing - 1 after group i's first are staged, each
    // by its wave (block b: wave b % kWaves), which loads its next one at once
    __syncthreads();
    if (total > 0u) {
      static_assert(kRing == 8, "every wave stages its first block below");
      for (uint32_t blk = wave; blk < kRing; blk += kWaves) {
        fetch(blk);
        stage(blk);
      }
      uint32_t next = kRing + wave;  // the block this wave stages next
      fetch(next);
      __syncthreads();
      for (uint32_t blk = 0; blk < kRing; ++blk) coarse(blk);
      uint32_t tested = kRing, staged = kRing;  // blocks
      __syncthreads();
      uint64_t bits, bits_n = 0ull;
      uint32_t k0 = 0, k1 = group(0, min(nk, 2 * tested), &bits), k2 = k1;
      weights(0, bits, 0);
      load(0);
      // Waves w and w + 4 share a SIMD: one prepares the next group (tests,
      // staging, weights) while the other multiplies, then they change places.
      const int turn = wave >> 2;
      int ab = 0;
      __syncthreads();
      while (k0 < nk) {
        const uint32_t known = 2 * tested, upto = staged;  // marked and staged before the last barrier
        staged = k0 / 2 + kRing;
        k2 = k1;
        if (k1 < nk) k2 = group(k1, min(nk, known), &bits_n);
        if (turn) products(k0, k1, bits, ab, first);
        if (k1 < k2) weights(k1, bits_n, ab ^ 1);
        for (; tested < upto; ++tested) coarse(tested);
        while (next < staged) {
          stage(next);
          next += kWaves;
          fetch(next);
        }
        if (!turn) products(k0, k1, bits, ab, first);
        k0 = k1;
        k1 = k2;
        bits = bits_n;
        ab ^= 1;
        __syncthreads();
      }
    }

    // ---- weight sums of the cells: the four lanes that share one
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      const int cb = wave + o * kWaves;
      double w = wsum[o];
      w += __shfl_xor(w, 16);
      w += __shfl_xor(w, 32);
      if (first() && cb < kCB && lane < 16) {
        sm.Wt[cb * 16 + lane] = w;
        const int x = x0 + (cb % kT) * 4 + (lane & 3), y = y0 + (cb / kT) * 4 + (lane >> 2);
        if (!kMask && a.wmap && slab == 0 && x < g.nx && y < g.ny)
          a.wmap[(int64_t)y * g.nx + x] = (float)w;
      }
    }
    __syncthreads();

    const float qnan = __builtin_nanf("");
    // (opaque, so that the addresses of the outputs are worked out here: made
    // before the passes they would take the products' registers)
    int row = y0 + lg;
    int64_t chan = ch0;
    asm volatile("" : "+v"(row), "+v"(chan));
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb) {
      const int y = row + (cb / kT) * 4;
      const int x = x0 + (cb % kT) * 4;
      if (!live || y >= g.ny || x >= g.nx) continue;
      float inv[4];
      bool has[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double wt = sm.Wt[cb * 16 + 4 * lg + r];
        has[r] = wt != 0.0;
        inv[r] = has[r] ? (float)(1.0 / wt) : 0.f;
      }
      const int64_t at = (int64_t)y * g.nx + x;
      const bool full = x + 3 < g.nx;
#pragma unroll
      for (int j = 0; j < kJ; ++j) {
        const int64_t ch = chan + j;
        if (ch >= C) continue;
        float* dst = a.cube + ch * G + at;
        if (!first() && pass == kPassSmall) {
          // results below 2^-100 (times 2^64 here), or whose sums are
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float U = acc[cb][j][r];
            float v;
            if constexpr (kMask) v = U / accw[cb][j][r];
            else v = has[r] ? U * inv[r] : qnan;
            if (x + r < g.nx && (fabsf(U) < 0x1p-36f || fabsf(v) < 0x1p-36f) && v == v)
              dst[r] = v * 0x1p-64f;
          }
          continue;
        }
        if (!first()) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (x + r < g.nx && acc[cb][j][r] > 0.f) {
              const float inf = __builtin_inff();
              dst[r] = pass == kPassPos ? inf : dst[r] == inf ? qnan : -inf;
            }
          continue;
        }
        float v[4], wc[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (kMask) {
            wc[r] = accw[cb][j][r];
            v[r] = (wc[r] != 0.f) ? acc[cb][j][r] / wc[r] : qnan;
          } else {
            v[r] = has[r] ? acc[cb][j][r] * inv[r] : qnan;
          }
        }
        float* wdst = kMask && a.wcube ? a.wcube + ch * G + at : nullptr;
        if (full) {
          store4(dst, v);
          if (kMask && wdst) store4(wdst, wc);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (x + r < g.nx) {
              dst[r] = v[r];
              if (kMask && wdst) wdst[r] = wc[r];
            }
        }
      }
    }
  };

  // The further passes are code of their own: with their tests in one common
  // loop the drift scan took 51.1 ms, so 50.4 (and 50.7 without passes for
  // small values; flagged 3.11, 3.05 and 3.02).
  walk(std::true_type{});
  if (sm.small == 0u && (kMask || sm.odd == 0u)) return;
  const bool odd = !kMask && sm.odd != 0u;
  for (pass = sm.small ? kPassSmall : kPassPos; pass <= (odd ? kPassNeg : kPassSmall); ++pass) {
    __syncthreads();
    walk(std::false_type{});
  }
}

}  // namespace hcg
