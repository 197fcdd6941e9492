// wave_util.h -- wave-level helpers shared by the kernels of the 3D Gaussian
// and 2D surfel paths: the FP64 cross-lane swaps and DPP moves, the
// transposing wave sum built on them, the XCD-grouped tile schedule, and the
// 8 x 8 pixel blocks the compositing kernels work over with the test of an
// entry against a block.
#pragma once
#include "gsr_device.h"

namespace gsr {

// Tile schedule groups: one per XCD (workgroup b runs on XCD b % kQueues).
constexpr int kQueues = 8;

// The tile of workgroup `bid` under the grouped, longest-first schedule
// `order` (tile ids, group after group); -1 for the padding workgroups.
__device__ __forceinline__ int tile_of_block(int bid, int n_tiles, int groups,
                                             const uint32_t* __restrict__ order) {
  const int per = (n_tiles + groups - 1) / groups;
  const int q = bid % groups, i = bid / groups;
  const int pos = q * per + i;
  if (i >= per || pos >= n_tiles) return -1;
  return (int)order[pos];
}

// Cross-lane helpers of the FP64 wave reduction (all VALU, no LDS traffic).
//
// swap_sum<32>(a, b): with v_permlane32_swap the upper half-wave of a trades
// places with the lower half-wave of b, so that afterwards a' + b' is
// a(l) + a(l ^ 32) on lanes l < 32 and b(l ^ 32) + b(l) on lanes l >= 32: the
// butterfly step over lane bit 5 that keeps a on the lower and b on the
// upper half, in one swap and one add.  swap_sum<16> does the same over lane
// bit 4 with v_permlane16_swap (odd 16-lane rows of a trade with even rows
// of b).
template <int W>
__device__ __forceinline__ double swap_sum(double a, double b) {
  const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
  uint32_t lo0, lo1, hi0, hi1;
  if constexpr (W == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32),
                                                     false, false);
    lo0 = lo[0]; lo1 = lo[1]; hi0 = hi[0]; hi1 = hi[1];
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32),
                                                     false, false);
    lo0 = lo[0]; lo1 = lo[1]; hi0 = hi[0]; hi1 = hi[1];
  }
  return __longlong_as_double((long long)(((uint64_t)hi0 << 32) | lo0)) +
         __longlong_as_double((long long)(((uint64_t)hi1 << 32) | lo1));
}

// The value of v on a partner lane inside the lane's 16-lane row: DPP row
// mirror (partner 15 - l) for lane bit 3, half-row mirror (7 - l) for bit 2,
// quad permutes (l ^ 2, l ^ 1) for bits 1 and 0.  The mirrors also flip the
// lower lane bits; the rounds that follow sum over those anyway.  A row
// rotation by 8 is l ^ 8, and one by 4 after it completes the sum over lane
// bits 3 and 2.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  // every lane's partner lies in its own row, so no lane reads out of
  // bounds and no old value is needed (bound_ctrl)
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf,
                                                         true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
constexpr int kDppRowRor8 = 0x128, kDppRowRor4 = 0x124, kDppRowMirror = 0x140,
              kDppHalfMirror = 0x141, kDppQuadXor2 = 0x4e, kDppQuadXor1 = 0xb1;

// Sum over the wave of N FP64 values per lane by recursive halving: at lane
// bit b a lane keeps the lower or the upper half of its values (by that bit)
// and adds its partner's copy of the same half.  The partners are those of
// the swaps and DPP moves above (bit 5: permlane32 swap, bit 4: permlane16
// swap, bits 3..0: row mirror, half-row mirror, quad xor 2, quad xor 1); a
// mirror also flips the lower bits, which later rounds sum over anyway, so
// after six rounds each total covers all 64 lanes and sits on exactly one
// lane.  Returns that lane's total, its index `idx` and `writer` = true on
// the N lanes that hold one (the rest hold padding).  All VALU, fixed order.
template <int C, int B>
__device__ __forceinline__ void halve_round(const double* in, double* out, int lane, int& base,
                                            int& cnt) {
  constexpr int H = (C + 1) / 2;
  const bool hi = (lane >> B) & 1;
#pragma unroll
  for (int j = 0; j < H; ++j) {
    const double lo_v = in[j];
    const double hi_v = (H + j < C) ? in[H + j] : 0.0;
    if constexpr (B == 5) {
      out[j] = swap_sum<32>(lo_v, hi_v);
    } else if constexpr (B == 4) {
      out[j] = swap_sum<16>(lo_v, hi_v);
    } else {
      const double keep = hi ? hi_v : lo_v;
      const double send = hi ? lo_v : hi_v;
      constexpr int ctrl = B == 3 ? kDppRowMirror
                         : B == 2 ? kDppHalfMirror
                         : B == 1 ? kDppQuadXor2 : kDppQuadXor1;
      out[j] = keep + dpp<ctrl>(send);
    }
  }
  if (hi) {
    base += H;
    cnt = cnt > H ? cnt - H : 0;
  } else {
    cnt = cnt < H ? cnt : H;
  }
}

template <int N>
__device__ __forceinline__ double wave_transpose_sum(const double (&v)[N], int lane, int& idx,
                                                     bool& writer) {
  static_assert(N >= 1 && N <= kWave, "one total per lane");
  constexpr int C4 = (N + 1) / 2, C3 = (C4 + 1) / 2, C2 = (C3 + 1) / 2, C1 = (C2 + 1) / 2,
                C0 = (C1 + 1) / 2;
  double r4[C4], r3[C3], r2[C2], r1[C1], r0[C0], rr[(C0 + 1) / 2];
  int base = 0, cnt = N;
  halve_round<N, 5>(v, r4, lane, base, cnt);
  halve_round<C4, 4>(r4, r3, lane, base, cnt);
  halve_round<C3, 3>(r3, r2, lane, base, cnt);
  halve_round<C2, 2>(r2, r1, lane, base, cnt);
  halve_round<C1, 1>(r1, r0, lane, base, cnt);
  halve_round<C0, 0>(r0, rr, lane, base, cnt);
  idx = base;
  writer = cnt > 0;
  return rr[0];
}

// Pixel blocks.
// A tile of TW x TH pixels is cut into 8 x 8 blocks, one pixel per lane (lane
// l owns pixel (l % 8, l / 8) of a block).  A square block has the smallest
// perimeter of 64 pixels, so the fewest Gaussians touch it.
constexpr int kBlk = 8;

template <int TW, int TH>
struct TileBlocks {
  static constexpr int kX = TW / kBlk, kY = TH / kBlk, kN = kX * kY;
};

// The part of the block at (bx, by) inside an entry's pixel bounds sqx, sqy
// (lo | hi << 16).
struct BlockPart {
  int xlo, xhi, ylo, yhi;
  __device__ __forceinline__ bool empty() const { return xlo > xhi || ylo > yhi; }
};

__device__ __forceinline__ BlockPart block_part(uint32_t sqx, uint32_t sqy, int bx, int by) {
  return {max(bx, (int)(sqx & 0xffff)), min(bx + kBlk - 1, (int)(sqx >> 16)),
          max(by, (int)(sqy & 0xffff)), min(by + kBlk - 1, (int)(sqy >> 16))};
}

// Its pixels, one bit per lane.
__device__ __forceinline__ uint64_t block_lanes(const BlockPart& b, int bx, int by) {
  const uint32_t cols = (0xffu >> (kBlk - 1 - (b.xhi - b.xlo))) << (b.xlo - bx);
  const uint64_t rows = (~0ull >> (kBlk * (kBlk - 1 - (b.yhi - b.ylo)))) << (kBlk * (b.ylo - by));
  const uint32_t c4 = cols * 0x01010101u;
  return (((uint64_t)c4 << 32) | c4) & rows;
}

// The least q = (a1 dx + a2 dy)^2 + (a3 dy)^2 over such a part, d = centre
// minus pixel (centre as FP32 hi/lo pairs).  Each lane asks this of its own
// entry, so 64 entries cost one evaluation.  q is convex with its minimum at
// d = 0: over the half-plane beyond the side nearest to 0 it is least at dy =
// -a1 a2 x / (a2^2 + a3^2), so over the part it is least in the row nearest
// to that dy, where m = a1 dx + a2 dy runs over an interval.  `big` receives
// the size of the terms that can cancel in m: a caller that compares q
// with a bound widens the bound by a few ulps of it (4e-6 is 64 FP32 ulps,
// far above the rounding of this test and of the per-pixel q), so that a part
// that fails holds no pixel whose computed value would pass.
__device__ __forceinline__ float least_q(float a1, float a2, float a3, float u_hi, float u_lo,
                                         float v_hi, float v_lo, const BlockPart& b, float& big) {
  const float dxl = dx_of(u_hi, u_lo, b.xhi), dxh = dx_of(u_hi, u_lo, b.xlo);
  const float dyl = dx_of(v_hi, v_lo, b.yhi), dyh = dx_of(v_hi, v_lo, b.ylo);
  const float xn = __builtin_amdgcn_fmed3f(0.0f, dxl, dxh);
  const float ys = -(a1 * a2 * xn) * __builtin_amdgcn_rcpf(a2 * a2 + a3 * a3);
  const float yc = __builtin_amdgcn_fmed3f(ys, dyl, dyh);
  const float m = __builtin_amdgcn_fmed3f(0.0f, a1 * dxl + a2 * yc, a1 * dxh + a2 * yc);
  const float t = a3 * yc;
  big = a1 * fmaxf(fabsf(dxl), fabsf(dxh)) + (fabsf(a2) + a3) * fmaxf(fabsf(dyl), fabsf(dyh));
  return m * m + t * t;
}

// lane j's value of v (j wave-uniform)
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int j) {
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), j);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, j);
  return ((uint64_t)hi << 32) | lo;
}

// What a launch does: all of a tile's list per workgroup; or, where that leaves
// SIMDs without work, a segment of it (blockIdx.y), for which the state behind
// the segment has to be known: an entry maps the pixel's (T, E) behind it to
// those in front by T / (1 - a) and (1 - a) E + a G . c, so a segment is the
// product of its 1 - a and the E it makes of 0.  One launch computes these for
// all segments but the first, the other starts each segment behind the later
// ones' maps.
enum BwdPass { kBwdWhole, kBwdMaps, kBwdSegments };

__device__ __forceinline__ uint32_t segment_len(uint32_t nproc, uint32_t batch,
                                               uint32_t segments) {
  return ((nproc + segments - 1) / segments + batch - 1) / batch * batch;
}

}  // namespace gsr
