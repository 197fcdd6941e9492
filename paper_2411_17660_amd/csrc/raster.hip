// raster.hip -- front-to-back compositing (forward) and its reverse-order
// backward, over 8 x 8 pixel blocks of the tiles.
//
// Forward, per pixel, over its tile's list in (depth, index) order
// (DROID-Splat eqn:rendering, C = sum_i c_i a_i prod_{j<i}(1 - a_j), with
// a_i = sigma_i G_i): entries whose 3-sigma square misses the pixel are
// skipped; a = min(0.99, sigma exp(-q/2)); a < 1/255 is skipped; the pixel
// stops before an entry that would drop T below 1e-4.  Outputs RGB + T bg,
// the alpha-blended depth sum z_i a_i T_i and accumulated alpha 1 - T.
//
// Layout on CDNA4: a wave composites one 8 x 8 block, a pixel per lane.  For
// every 64 list entries each lane tests its own entry against the block
// (exact ellipse against rectangle), so the wave visits only entries that
// reach it (on 500k Gaussians over 8 x 1200x680, 98 % of the visits blend at
// least one pixel; with 16 x 4 strips and the entries' boxes 46 % did).  What
// bounds the forward is VALU issue, ~26 instructions a visit; it took 1081 us
// there with one wave per 16 x 16 tile, 738 us with one per block, and on one
// 640x480 frame, whose 1,200 tiles left one wave to a SIMD, 509 and 65 us.
//
// Backward: the waves of a tile walk the tile's processed prefix from the
// back.  Each lane recomputes alpha bit-identically (same helpers, explicit
// fma), rebuilds T_i = T_{i+1} / (1 - a_i) (reciprocal plus one Newton step)
// and carries what is seen behind each entry through the convex recurrence
// B_{i-1} = a_i c_i + (1 - a_i) B_i from B = background (depth from 0, the
// transmittance behind from 1), so that dC/da_i = T_i (c_i - B_i): T_i only
// scales the result and the recurrence damps rounding instead of
// accumulating it.  Colour and depth enter only through G . B (G the pixel's
// upstream gradient), which is what the lane keeps, in FP64.  The
// screen-space gradient of an entry is taken with respect to (u, v, Sigma'):
// with Q = Sigma'^-1 = L L^T (L the factor the forward already uses) and d
// the offset, dq/dd = 2 Q d and dq/dSigma' = -(Q d)(Q d)^T,
// Q d = L (L^T d); this avoids the ill-conditioned -Q dQ Q step from conic
// gradients for elongated Gaussians.  What an entry receives from its pixels
// are moments, summed across the wave in FP64 by matrix products (below); the
// result for this (tile, entry) key goes to its own slot (no atomics),
// stamped with the backward's epoch so the per-record reduction can skip
// slots of keys that no pixel reached.  It took 2531 us on the 8 x 1200x680
// batch and 708 us on the 640x480 frame with one wave per tile and a
// reduction through LDS (an LDS pipe shared by four SIMDs, which that
// reduction held for ~104 clocks a key), 1806 and 233 us as it is now.
#include "launch.h"
#include "wave_util.h"
#include <algorithm>

namespace gsr {

// Tile schedule.  The tiles are split into kQueues groups of contiguous tile
// ids (neighbouring tiles share Gaussians, so a group shares one XCD's L2);
// workgroups are dealt to the XCDs in turn, so workgroup b runs on XCD
// b % kQueues and takes the (b / kQueues)-th tile of that group.  The
// hardware dispatches workgroups in index order, so sorting each group by
// descending expected work gives a longest-first list schedule without any
// queue or atomic: long tiles start first and the short ones fill the tail.
constexpr int kOrderBins = 1024;

__device__ __forceinline__ uint32_t work_bucket(uint32_t w) {
  if (w == 0) return 0;
  const int lz = __clz(w);
  const int e = 31 - lz;                                      // floor(log2 w)
  const uint32_t frac = e > 0 ? ((w << (lz + 1)) >> 27) : 0;  // next 5 bits
  return min((uint32_t)kOrderBins - 1, 1u + (uint32_t)e * 32u + frac);
}

// One workgroup per group: a counting sort of the group's tiles by
// descending work bucket (order inside a bucket is arbitrary; results do not
// depend on it).  Work = processed entries of a previous forward over the
// same tiles (`nproc`); without it the tiles keep their spatial order.
__global__ void __launch_bounds__(1024) tile_order_kernel(int n_tiles, int groups,
                                                          const uint32_t* nproc,
                                                          uint32_t* __restrict__ order,
                                                          uint32_t* clear) {
  static_assert(kOrderBins == 1024, "one thread per bin in the offsets scan");
  __shared__ uint32_t bins[kOrderBins];
  const int q = blockIdx.x;
  const int per = (n_tiles + groups - 1) / groups;
  const int t0 = q * per, t1 = min(n_tiles, t0 + per);
  for (int i = threadIdx.x; i < kOrderBins; i += blockDim.x) bins[i] = 0;
  __syncthreads();
  if (!nproc) {
    for (int t = t0 + (int)threadIdx.x; t < t1; t += blockDim.x) {
      order[t] = (uint32_t)t;
      if (clear) clear[t] = 0u;
    }
    return;
  }
  for (int t = t0 + (int)threadIdx.x; t < t1; t += blockDim.x)
    atomicAdd(&bins[work_bucket(nproc[t])], 1u);
  __syncthreads();
  {  // exclusive offsets, largest bucket first: thread i takes bin 1023 - i
    __shared__ uint32_t wtot[kOrderBins / kWave];
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const int bin = kOrderBins - 1 - (int)threadIdx.x;
    const uint32_t c = bins[bin];
    uint32_t v = c;  // inclusive scan over the wave's lanes
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t u = __shfl_up(v, o, kWave);
      if (lane >= o) v += u;
    }
    if (lane == kWave - 1) wtot[wv] = v;
    __syncthreads();
    uint32_t base = 0;
    for (int k = 0; k < wv; ++k) base += wtot[k];
    bins[bin] = base + v - c;
  }
  __syncthreads();
  for (int t = t0 + (int)threadIdx.x; t < t1; t += blockDim.x) {
    const uint32_t pos = atomicAdd(&bins[work_bucket(nproc[t])], 1u);
    order[t0 + pos] = (uint32_t)t;
    if (clear) clear[t] = 0u;  // (may be nproc: this thread has read its tiles' counts)
  }
}

// block_lanes with the entry's ellipse: 0 where the block's part inside its
// bounds cannot reach alpha >= 1/255 (least_q against cull_r^2, q where alpha
// reaches 1/255, with a margin).  ALL: the bounds alone.
template <bool ALL>
__device__ __forceinline__ uint64_t block_pixels(const Record& R, int bx, int by) {
  const BlockPart b = block_part(R.sqx, R.sqy, bx, by);
  if (b.empty()) return 0;
  float big;
  const float q = least_q(R.a1, R.a2, R.a3, R.u_hi, R.u_lo, R.v_hi, R.v_lo, b, big);
  const float r = R.cull_r + 4e-6f * big;
  if (!ALL && q > r * r) return 0;
  return block_lanes(b, bx, by);
}

// The entry fields that the compositing reads per pixel, staged in LDS.
struct alignas(16) Entry {
  float4 c;    // u_hi, u_lo, v_hi, v_lo
  float4 q;    // a1, a2, a3, opacity
  float4 col;  // c0, c1, c2, z
};

__device__ __forceinline__ Entry entry_of(const Record& R) {
  return {make_float4(R.u_hi, R.u_lo, R.v_hi, R.v_lo), make_float4(R.a1, R.a2, R.a3, R.opacity),
          make_float4(R.c0, R.c1, R.c2, R.z)};
}

// The forward's LDS entry: also the block's pixels inside the entry's bounds
// and one past its list position.
struct alignas(16) FwdEntry {
  Entry e;
  uint32_t px_lo, px_hi, pos, pad;
};

// One wave composites one 8 x 8 block, a pixel per lane.  Records of 64
// entries at a time wait in registers (their loads are issued while the batch
// before them is composited), each lane culls its record against the block,
// and the ones that reach it are packed into LDS in list order, where the wave
// reads them back as broadcasts one entry ahead of their use.  Which lanes
// take part is kept as wave-uniform lane masks.
template <int TW, int TH, bool COUNT, bool MEDIAN>
__global__ void __launch_bounds__(kWave) composite_fwd_kernel(
    int first, int n_tiles, int groups, const uint32_t* __restrict__ order, int n_frames,
    const FrameDesc* __restrict__ frames, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ vals, const Record* __restrict__ rec, float bg0, float bg1,
    float bg2, float* __restrict__ rgb, float* __restrict__ depth, float* __restrict__ alpha,
    float* __restrict__ t_final, int32_t* __restrict__ n_last, uint32_t* __restrict__ tile_nproc,
    unsigned long long* __restrict__ pair_count, int32_t* __restrict__ med_pos) {
  using TB = TileBlocks<TW, TH>;
  __shared__ FwdEntry sm[kWave + 2];
  // workgroup i of a group takes block i % kN of its (i / kN)-th tile, so that
  // a tile's blocks share the XCD of its group (and the records in its L2)
  const int group = blockIdx.x % groups, i_wg = first + blockIdx.x / groups;
  const int tile = tile_of_block((i_wg / TB::kN) * groups + group, n_tiles, groups, order);
  if (tile < 0) return;
  const int blk = i_wg % TB::kN;
  const int f = frame_of_tile(frames, n_frames, tile);
  const FrameDesc fr = frames[f];
  const int lt = tile - fr.tile_offset;
  const int bx = (lt % fr.grid_x) * TW + (blk % TB::kX) * kBlk;
  const int by = (lt / fr.grid_x) * TH + (blk / TB::kX) * kBlk;
  const int lane = threadIdx.x;
  const int px = bx + (lane & 7), py = by + (lane >> 3);
  const uint2 rg = ranges[tile];

  // D: alpha-blended depth, or (MEDIAN) the depth of the entry after which
  // T first falls below 1/2, one past list position mpos (0: none yet)
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, D = 0.0f;
  uint32_t last = 0, mpos = 0;
  uint64_t open = __ballot(px < fr.width && py < fr.height);  // pixels that have not stopped
  uint64_t hits = 0;  // (pixel, entry) pairs whose square test passed (COUNT only)
  const auto blend = [&](const FwdEntry& E) {
    const uint64_t in = (((uint64_t)__builtin_amdgcn_readfirstlane(E.px_hi) << 32) |
                         (uint32_t)__builtin_amdgcn_readfirstlane(E.px_lo)) & open;
    if (COUNT) hits += __popcll(in);
    const float dx = dx_of(E.e.c.x, E.e.c.y, px), dy = dx_of(E.e.c.z, E.e.c.w, py);
    const float q = q_of(E.e.q.x, E.e.q.y, E.e.q.z, dx, dy);
    const float a = fminf(kAlphaMax, E.e.q.w * gauss_of(q));
    const float Tn = T * (1.0f - a);
    uint64_t act = __ballot(!(a < kAlphaMin)) & in;
    const uint64_t stop = __ballot(Tn < kTMin) & act;
    open &= ~stop;
    act &= ~stop;
    if (__builtin_amdgcn_inverse_ballot_w64(act)) {
      const float w = a * T;
      C0 += E.e.col.x * w;
      C1 += E.e.col.y * w;
      C2 += E.e.col.z * w;
      if (MEDIAN) {
        if (mpos == 0 && Tn < 0.5f) {
          mpos = E.pos;
          D = E.e.col.w;
        }
      } else {
        D += E.e.col.w * w;
      }
      T = Tn;
      last = E.pos;
    }
  };
  // the batch's record in registers, and the next batch's list entry
  Record R{};
  uint32_t v_next = 0;
  if (rg.x + lane < rg.y) R = rec[vals[rg.x + lane]];
  if (rg.x + kWave + lane < rg.y) v_next = vals[rg.x + kWave + lane];
  for (uint32_t b = rg.x; b < rg.y && open; b += kWave) {
    uint64_t in = 0;
    asm volatile("" ::"v"(R.reserved));  // (below)
    if (b + lane < rg.y) in = block_pixels<COUNT>(R, bx, by);
    const uint64_t mk = __ballot(in != 0);
    const int n = __popcll(mk);
    const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u));
    if (in) sm[at] = {entry_of(R), (uint32_t)in, (uint32_t)(in >> 32), b + lane + 1 - rg.x, 0u};
    if (lane < 2) sm[n + lane].px_lo = sm[n + lane].px_hi = 0u;  // (entries are taken in pairs)
    // Every register the record's loads write has a reader, at the latest the
    // empty asm above: the register of a word that nothing reads would go to
    // another value, whose first write then waits for the load.
    if (b + kWave + lane < rg.y) R = rec[v_next];
    if (b + 2 * kWave + lane < rg.y) v_next = vals[b + 2 * kWave + lane];
    __syncthreads();
    FwdEntry E0 = sm[0];
    for (int i = 0; i < n && open; i += 2) {
      const FwdEntry E1 = sm[i + 1];
      blend(E0);
      E0 = sm[i + 2];
      blend(E1);
    }
    __syncthreads();
  }
  if (px < fr.width && py < fr.height) {
    const int64_t plane = (int64_t)fr.width * fr.height;
    const int64_t p = (int64_t)py * fr.width + px;
    float* img = rgb + 3 * fr.pixel_offset;
    img[p] = C0 + T * bg0;
    img[plane + p] = C1 + T * bg1;
    img[2 * plane + p] = C2 + T * bg2;
    depth[fr.pixel_offset + p] = D;
    alpha[fr.pixel_offset + p] = 1.0f - T;
    t_final[fr.pixel_offset + p] = T;
    n_last[fr.pixel_offset + p] = (int32_t)last;
    if (MEDIAN) med_pos[fr.pixel_offset + p] = (int32_t)mpos - 1;
  }
  int mx = (int)last;
  for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) {
    if (TB::kN == 1) tile_nproc[tile] = (uint32_t)mx;
    else if (mx > 0) atomicMax(&tile_nproc[tile], (uint32_t)mx);  // cleared by the order kernel
  }
  if (COUNT && lane == 0) atomicAdd(pair_count, (unsigned long long)hits);
}

// Backward.  A workgroup takes a tile with WAVES waves of PIX blocks each (one
// pixel of a block per lane); the waves walk the same batches of list entries
// from the back, each visiting the entries that reach one of its blocks.  Per
// pixel and visit a lane forms p = a dL/da and w = a T; an entry receives the
// sums over pixels of w times the upstream colour and depth gradient and of p
// times 1, X, Y, X^2, X Y, Y^2 (X, Y the pixel's position in the tile).  Sums
// over the lanes of a wave are products with constant matrices, taken in FP64
// by v_mfma_f64_4x4x4, whose lane 16 k + 4 b + i holds element (i, k) of the
// left and (k, i) of the right operand and whose lane 16 i + 4 b + j holds
// (i, j) of the result, for four independent products b.  With the pixels as
// they lie in the lanes (i = x % 4, b = x / 4 + 2 (y % 2), k = y / 2) a first
// product with (1, Y, Y^2) sums over k; its result is laid out as the left
// operand of a second one with (1, X, X^2) that sums over i; two row rotations
// add the four b.  The colour and depth sums take the same way with unit
// matrices and land in the fourth column.  No data goes through LDS and no
// lane selects anything; a transposing reduction took 62 VALU instructions
// and 14 more per visit for the products.  One lane per entry then adds the
// waves' totals in wave order, moves the moments from the tile's origin to the
// entry's centre, whitens them (all FP64) and stores the key's slot as FP32.
// What bounds it: VALU issue.
constexpr int kBatchB = 64;          // list entries per batch
constexpr int kBwdMinWaves = 4096;  // four waves on each of the 1,024 SIMDs
static_assert(kNG == 10, "4 colour and depth sums and 6 moments");

struct alignas(16) BwdEntry {  // as Entry, the colour and depth already FP64
  float4 c, q;
  double c0, c1, c2, z;
};

template <int WAVES>
struct BwdLds {
  BwdEntry sm[WAVES > 1 ? 2 : 1][kBatchB];
  uint32_t slot[WAVES > 1 ? 2 : 1][kBatchB];
  alignas(16) double tot[WAVES][kBatchB][kNG];  // 4 colour / depth sums, 6 moments
  uint64_t summed[WAVES];                       // the batch's entries the wave has sums for
};

template <int TW, int TH, int PIX, bool MEDIAN, BwdPass PASS>
__global__ void __launch_bounds__(TW* TH / PIX, PIX == 4 ? 3 : 4) composite_bwd_kernel(
    double2* __restrict__ maps, int n_tiles, int groups, const uint32_t* __restrict__ order,
    int n_frames, const FrameDesc* __restrict__ frames, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ vals, const Record* __restrict__ rec,
    const uint32_t* __restrict__ keyoff, const uint32_t* __restrict__ tile_nproc, float bg0,
    float bg1, float bg2, const float* __restrict__ g_rgb, const float* __restrict__ g_depth,
    const float* __restrict__ g_alpha, const float* __restrict__ t_final,
    const int32_t* __restrict__ n_last, float* __restrict__ partial,
    uint32_t* __restrict__ stamp, const uint32_t* __restrict__ epoch_dev,
    const int32_t* __restrict__ med_pos) {
  using TB = TileBlocks<TW, TH>;
  constexpr int WAVES = TB::kN / PIX;
  // a wave's blocks: kCols x kRows neighbouring ones (whole rows of the tile,
  // or a part of one row)
  constexpr int kCols = PIX < TB::kX ? PIX : TB::kX, kRows = PIX / kCols;
  static_assert(TB::kX % kCols == 0, "blocks of a wave form a rectangle");
  __shared__ BwdLds<WAVES> L;
  const int tile = tile_of_block(blockIdx.x, n_tiles, groups, order);
  if (tile < 0) return;
  uint32_t nproc = tile_nproc[tile];
  // the segment's entries, from now on positions 0 .. nproc of a list of its own
  uint32_t seg0 = 0;
  const int seg = PASS == kBwdMaps ? blockIdx.y + 1 : blockIdx.y;
  if (PASS != kBwdWhole) {
    const uint32_t len = segment_len(nproc, kBatchB, PASS == kBwdMaps ? gridDim.y + 1 : gridDim.y);
    seg0 = min(nproc, seg * len);
    nproc = min(nproc - seg0, len);
  }
  if (nproc == 0 && PASS != kBwdMaps) return;  // uniform over the workgroup
  const uint32_t epoch = *epoch_dev;
  const int f = frame_of_tile(frames, n_frames, tile);
  const FrameDesc fr = frames[f];
  const int lt = tile - fr.tile_offset;
  const int tx = lt % fr.grid_x, ty = lt / fr.grid_x;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int blk0 = wave * PIX;
  const int bx0 = tx * TW + (blk0 % TB::kX) * kBlk, by0 = ty * TH + (blk0 / TB::kX) * kBlk;
  const int px0 = bx0 + (lane & 7), py0 = by0 + (lane >> 3);
  uint2 rg = ranges[tile];
  rg.x += seg0;
  const int64_t plane = (int64_t)fr.width * fr.height;
  // the maps of the tile's pixels, segment after segment from the second
  double2* my_maps = nullptr;
  if (PASS != kBwdWhole)
    my_maps = maps + (int64_t)tile * (PASS == kBwdMaps ? gridDim.y : gridDim.y - 1) * (TW * TH) +
              wave * kWave + lane;

  // per pixel: T_{i+1} and the upstream gradients G.  dL/da_i = T_i G . (c_i -
  // B_i), the upstream-weighted difference between the entry's colour, depth
  // and alpha (which is 1) and what is seen behind it, B_i.  That difference
  // cancels on surfaces of uniform colour, and the gradient of a large
  // Gaussian sums it over up to 10^5 pixels, so it is formed in FP64.  G is
  // fixed per pixel, so the recursion B_i = B_{i+1} + a_i (c_i - B_{i+1})
  // carries over to the scalar E = G . B - G_A, which is what the pixel keeps
  // (in FP64), together with G itself in FP64.
  float T[PIX];
  double E[PIX], H0[PIX], H1[PIX], H2[PIX], HZ[PIX];
  int last[PIX], mp[PIX];  // mp: MEDIAN, the list position of the pixel's depth
  uint32_t most[PIX];      // the block's longest walk (wave-uniform)
#pragma unroll
  for (int k = 0; k < PIX; ++k) {
    const int px = px0 + (k % kCols) * kBlk, py = py0 + (k / kCols) * kBlk;
    T[k] = 1.0f;
    E[k] = H0[k] = H1[k] = H2[k] = HZ[k] = 0.0;
    last[k] = 0;
    mp[k] = -1;
    if (px < fr.width && py < fr.height) {
      const int64_t p = (int64_t)py * fr.width + px, q = fr.pixel_offset + p;
      const float* gi = g_rgb + 3 * fr.pixel_offset;
      last[k] = n_last[q] - (int)seg0;
      if (MEDIAN) mp[k] = med_pos[q] - (int)seg0;
      T[k] = t_final[q];
      H0[k] = gi[p];
      H1[k] = gi[plane + p];
      H2[k] = gi[2 * plane + p];
      HZ[k] = g_depth[q];
      // behind the last entry: the background colour at depth 0 and alpha 0
      E[k] = __builtin_fma(H2[k], (double)bg2,
                           __builtin_fma(H1[k], (double)bg1, H0[k] * (double)bg0)) -
             (double)g_alpha[q];
    }
    if (PASS == kBwdMaps) {
      T[k] = 1.0f;
      E[k] = 0.0;
    } else if (PASS == kBwdSegments) {
      // from behind the list to behind the segment
      double t = T[k];
      for (int s = (int)gridDim.y - 2; s >= seg; --s) {
        const double2 m = my_maps[s * (TW * TH)];
        E[k] = __builtin_fma(m.x, E[k], m.y);
        t /= m.x;
      }
      T[k] = (float)t;
    }
    int mx = max(last[k], 0);
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, kWave));
    most[k] = __builtin_amdgcn_readfirstlane((uint32_t)mx);
  }
  double through = 1.0;  // kBwdMaps: the product of 1 - alpha
  // right operands: powers of Y by block row (k the row pair) and of X by
  // block column, unit columns for the colours
  double wy[kRows], wx[kCols], unit[4];
  {
    const int j = lane & 3, k = lane >> 4, b = (lane >> 2) & 3;
    const auto power = [&](double v) {
      return j == 0 ? 1.0 : j == 1 ? v : j == 2 ? v * v : 0.0;
    };
#pragma unroll
    for (int r = 0; r < kRows; ++r) wy[r] = power(by0 - ty * TH + r * kBlk + 2 * k + (b >> 1));
#pragma unroll
    for (int c = 0; c < kCols; ++c) wx[c] = power(bx0 - tx * TW + c * kBlk + k + 4 * (b & 1));
#pragma unroll
    for (int c = 0; c < 4; ++c) unit[c] = j == c ? 1.0 : 0.0;
  }
  // lane 16 a + c of the result: moment Y^a X^c (c < 3), colour / depth sum a
  // (c = 3); its place in a row of totals (negative: not used)
  int out_v = -1;
  {
    const int c = lane & 3, a = lane >> 4;
    if (!(lane & 12)) {
      if (c == 3) out_v = a;
      else if (a + c <= 2) out_v = 4 + (a == 0 ? c : a == 1 ? 3 + c : 5);
    }
  }
  // colour / depth sums of the lane's pixels; reset after each entry that was
  // reduced (a lane adds only past the alpha test)
  double gc0 = 0.0, gc1 = 0.0, gc2 = 0.0, gz = 0.0;
  asm volatile("" : "+v"(gc0), "+v"(gc1), "+v"(gc2), "+v"(gz));
  // Batches of list entries from the back: [hi - kBatchB, hi).  The batch's
  // record waits in registers, the next batch's list entry is loaded ahead.
  int hi = (int)nproc, buf = 0;
  Record R{};
  uint32_t r_cur = 0, r_next = 0;
  if (lane < hi) r_cur = vals[rg.x + max(0, hi - kBatchB) + lane];
  if (lane < hi) R = rec[r_cur];
  if (lane < hi - kBatchB) r_next = vals[rg.x + max(0, hi - 2 * kBatchB) + lane];
  for (; hi > 0; hi -= kBatchB, buf ^= WAVES > 1) {
    const int lo = max(0, hi - kBatchB);
    const bool has = lane < hi - lo;
    asm volatile("" ::"v"(R.reserved));  // as in the forward
    uint64_t mk[PIX], in[PIX], any = 0;
#pragma unroll
    for (int k = 0; k < PIX; ++k) {
      in[k] = 0;
      if (has && (uint32_t)(lo + lane) < most[k])
        in[k] = block_pixels<false>(R, bx0 + (k % kCols) * kBlk, by0 + (k / kCols) * kBlk);
      mk[k] = __ballot(in[k] != 0);
      any |= mk[k];
    }
    if (WAVES == 1 ? (any >> lane) & 1 : has && (lane & (WAVES - 1)) == wave) {
      const Entry e = entry_of(R);
      L.sm[buf][lane] = {e.c, e.q, R.c0, R.c1, R.c2, R.z};
      // the record's tile rect, from its pixel bounds
      const int rx0 = (int)(R.sqx & 0xffff) / TW, rx1 = (int)(R.sqx >> 16) / TW;
      const int ry0 = (int)(R.sqy & 0xffff) / TH;
      L.slot[buf][lane] = keyoff[r_cur] + (uint32_t)((ty - ry0) * (rx1 - rx0 + 1) + (tx - rx0));
    }
    r_cur = r_next;
    if (lane < lo) R = rec[r_cur];
    if (lane < lo - kBatchB) r_next = vals[rg.x + max(0, lo - 2 * kBatchB) + lane];
    __syncthreads();  // (also: the previous batch's sums have been read)
    uint64_t summed = 0;
    while (any) {
      const int j = 63 - __builtin_clzll(any);
      any &= ~(1ull << j);
      const int pos = lo + j;
      const BwdEntry En = L.sm[buf][j];
      // the block columns' a1 dx, the block rows' dy and (a3 dy)^2
      float ax[kCols], dy[kRows], bb[kRows];
#pragma unroll
      for (int c = 0; c < kCols; ++c) ax[c] = En.q.x * dx_of(En.c.x, En.c.y, px0 + c * kBlk);
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        dy[r] = dx_of(En.c.z, En.c.w, py0 + r * kBlk);
        const float b = En.q.z * dy[r];
        bb[r] = b * b;
      }
      double my[kCols];  // sums over k of p Y^j, by block column
#pragma unroll
      for (int c = 0; c < kCols; ++c) {
        my[c] = 0.0;
        asm volatile("" : "+v"(my[c]));
      }
      uint64_t hit = 0;
#pragma unroll
      for (int k = 0; k < PIX; ++k) {
        if (PIX > 1 && !((mk[k] >> j) & 1)) continue;  // block missed (uniform)
        const float m = __builtin_fmaf(En.q.y, dy[k / kCols], ax[k % kCols]);
        const float g = gauss_of(__builtin_fmaf(m, m, bb[k / kCols]));  // q_of
        const float sg = En.q.w * g;
        const float a = fminf(kAlphaMax, sg);
        const uint64_t act = __ballot(!(a < kAlphaMin)) & __ballot(pos < last[k]) &
                             readlane64(in[k], j);
        hit |= act;
        float p = 0.0f;
        if (PASS == kBwdMaps) {
          if (__builtin_amdgcn_inverse_ballot_w64(act)) {
            through *= (double)(1.0f - a);
            double diff = __builtin_fma(H0[k], En.c0, -E[k]);
            diff = __builtin_fma(H1[k], En.c1, diff);
            diff = __builtin_fma(H2[k], En.c2, diff);
            if (!MEDIAN) diff = __builtin_fma(HZ[k], En.z, diff);
            E[k] = __builtin_fma((double)a, diff, E[k]);
          }
          continue;
        }
        if (__builtin_amdgcn_inverse_ballot_w64(act)) {
          const float om = 1.0f - a;
          const float inv = __builtin_amdgcn_rcpf(om);
          float Ti = T[k] * inv;
          Ti = __builtin_fmaf(__builtin_fmaf(-Ti, om, T[k]), inv, Ti);  // Newton step
          const float w = a * Ti;
          T[k] = Ti;
          // G . (c_i - B_i) = G . c_i - E
          double diff = __builtin_fma(H0[k], En.c0, -E[k]);
          diff = __builtin_fma(H1[k], En.c1, diff);
          diff = __builtin_fma(H2[k], En.c2, diff);
          if (!MEDIAN) diff = __builtin_fma(HZ[k], En.z, diff);
          // step the 'behind' state in front of entry i
          E[k] = __builtin_fma((double)a, diff, E[k]);
          const double wd = w;
          gc0 = __builtin_fma(H0[k], wd, gc0);
          gc1 = __builtin_fma(H1[k], wd, gc1);
          gc2 = __builtin_fma(H2[k], wd, gc2);
          if (MEDIAN)
            gz += pos == mp[k] ? HZ[k] : 0.0;
          else
            gz = __builtin_fma(HZ[k], wd, gz);
          // p = a dL/da; clamped: alpha does not move
          p = sg > kAlphaMax ? 0.0f : w * (float)diff;
        }
        my[k % kCols] =
            __builtin_amdgcn_mfma_f64_4x4x4f64((double)p, wy[k / kCols], my[k % kCols], 0, 0, 0);
      }
      if (PASS == kBwdMaps || hit == 0) continue;
      double mom = __builtin_amdgcn_mfma_f64_4x4x4f64(my[0], wx[0], 0.0, 0, 0, 0);
#pragma unroll
      for (int c = 1; c < kCols; ++c)
        mom = __builtin_amdgcn_mfma_f64_4x4x4f64(my[c], wx[c], mom, 0, 0, 0);
      double cs = __builtin_amdgcn_mfma_f64_4x4x4f64(gc0, unit[0], 0.0, 0, 0, 0);
      cs = __builtin_amdgcn_mfma_f64_4x4x4f64(gc1, unit[1], cs, 0, 0, 0);
      cs = __builtin_amdgcn_mfma_f64_4x4x4f64(gc2, unit[2], cs, 0, 0, 0);
      cs = __builtin_amdgcn_mfma_f64_4x4x4f64(gz, unit[3], cs, 0, 0, 0);
      double tot = __builtin_amdgcn_mfma_f64_4x4x4f64(cs, unit[3], mom, 0, 0, 0);
      if (__builtin_expect(__ballot(!isfinite(tot)) != 0, 0)) {
        // A p or colour sum that is not finite (an upstream gradient or a
        // colour that is not, a p that overflows) has met the zeros of the
        // others' columns: sum each colour by itself and select.  Every such
        // value is seen here, as each also meets a one.
        const int col = lane & 3;
        const double v[4] = {gc0, gc1, gc2, gz};
        cs = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double d = __builtin_amdgcn_mfma_f64_4x4x4f64(v[c], 1.0, 0.0, 0, 0, 0);
          if (col == c) cs = d;
        }
        cs = __builtin_amdgcn_mfma_f64_4x4x4f64(cs, 1.0, 0.0, 0, 0, 0);
        tot = col == 3 ? cs : mom;
      }
      gc0 = gc1 = gc2 = gz = 0.0;
      asm volatile("" : "+v"(gc0), "+v"(gc1), "+v"(gc2), "+v"(gz));
      tot += dpp<kDppRowRor8>(tot);
      tot += dpp<kDppRowRor4>(tot);
      if (out_v >= 0) L.tot[wave][j][out_v] = tot;
      summed |= 1ull << j;
    }
    if (PASS == kBwdMaps) {
      __syncthreads();
      continue;
    }
    if (lane == 0) L.summed[wave] = summed;
    __syncthreads();
    // one wave (in turn) finishes the batch's entries while the others go on
    if (((nproc - hi) / kBatchB) % WAVES == (uint32_t)wave) {
      double t[kNG];
#pragma unroll
      for (int v = 0; v < kNG; ++v) t[v] = 0.0;
      bool any_sum = false;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        if (!((L.summed[w] >> lane) & 1)) continue;
        any_sum = true;
        const double2* src = reinterpret_cast<const double2*>(L.tot[w][lane]);
#pragma unroll
        for (int v = 0; v < kNG / 2; ++v) {
          t[2 * v] += src[v].x;
          t[2 * v + 1] += src[v].y;
        }
      }
      if (any_sum) {
        const BwdEntry& En = L.sm[buf][lane];
        const double ux = ((double)En.c.x + En.c.y) - tx * TW;
        const double uy = ((double)En.c.z + En.c.w) - ty * TH;
        const double a1 = En.q.x, a2 = En.q.y, a3 = En.q.z;
        const double P = t[4], Px = t[5], Pxx = t[6], Py = t[7], Pxy = t[8], Pyy = t[9];
        const double sx = ux * P - Px, sy = uy * P - Py;  // sums of p dx, p dy
        const double sxx = ux * (sx - Px) + Pxx, syy = uy * (sy - Py) + Pyy;
        const double sxy = uy * sx - ux * Py + Pxy;
        const double ym = a1 * sxy + a2 * syy;
        const uint32_t sl = L.slot[buf][lane];
        float2* out = reinterpret_cast<float2*>(partial + (size_t)sl * kNG);
        out[0] = make_float2((float)(a1 * sx + a2 * sy), (float)(a3 * sy));
        out[1] = make_float2((float)(a1 * (a1 * sxx + a2 * sxy) + a2 * ym), (float)(a3 * ym));
        out[2] = make_float2((float)(a3 * a3 * syy), (float)(P / En.q.w));
        out[3] = make_float2((float)t[0], (float)t[1]);
        out[4] = make_float2((float)t[2], (float)t[3]);
        stamp[sl] = epoch;
      }
    }
    if (WAVES == 1) __syncthreads();
  }
  if (PASS == kBwdMaps) my_maps[(seg - 1) * (TW * TH)] = make_double2(through, E[0]);
}

static void launch_order(hipStream_t st, int n_tiles, int groups, const uint32_t* nproc,
                         uint32_t* order, uint32_t* clear = nullptr) {
  hipLaunchKernelGGL(tile_order_kernel, dim3((unsigned)groups), dim3(1024), 0, st, n_tiles,
                     groups, nproc, order, clear);
}

static unsigned grid_of(int n_tiles, int groups) {
  return (unsigned)(((n_tiles + groups - 1) / groups) * groups);
}

void launch_tile_order(hipStream_t st, int n_tiles, int groups, const uint32_t* nproc,
                       uint32_t* order, uint32_t* clear) {
  if (n_tiles > 0) launch_order(st, n_tiles, groups, nproc, order, clear);
}

unsigned tile_schedule_grid(int n_tiles, int groups) { return grid_of(n_tiles, groups); }
int tile_schedule_groups(bool xcd_groups) { return xcd_groups ? kQueues : 1; }

template <int TW, int TH>
static void launch_fwd_t(hipStream_t st, int n_tiles, int groups, const uint32_t* order, int F,
                         const FrameDesc* frames, const uint2* ranges, const uint32_t* vals,
                         const Record* rec, const float* bg, float* rgb, float* depth,
                         float* alpha, float* t_final, int32_t* n_last, uint32_t* nproc,
                         unsigned long long* pairs, int32_t* med_pos) {
  const auto go = [&](auto* k) {
    for_block_runs(n_tiles, groups, TileBlocks<TW, TH>::kN, [&](int first, unsigned blocks) {
      hipLaunchKernelGGL(k, dim3(blocks), dim3(kWave), 0, st, first, n_tiles, groups, order, F,
                         frames, ranges, vals, rec, bg[0], bg[1], bg[2], rgb, depth, alpha, t_final,
                         n_last, nproc, pairs, med_pos);
    });
  };
  if (pairs && med_pos) go(composite_fwd_kernel<TW, TH, true, true>);
  else if (pairs) go(composite_fwd_kernel<TW, TH, true, false>);
  else if (med_pos) go(composite_fwd_kernel<TW, TH, false, true>);
  else go(composite_fwd_kernel<TW, TH, false, false>);
}

template <int TW, int TH, int PIX>
static void launch_bwd_t(hipStream_t st, int pix, int n_tiles, int groups, const uint32_t* order,
                         int F, const FrameDesc* frames, const uint2* ranges,
                         const uint32_t* vals, const Record* rec, const uint32_t* keyoff,
                         const uint32_t* nproc, const float* bg, const float* g_rgb,
                         const float* g_depth, const float* g_alpha, const float* t_final,
                         const int32_t* n_last, float* partial, uint32_t* stamp,
                         const uint32_t* epoch, const int32_t* med_pos, int segments,
                         double2* maps) {
  if constexpr (PIX > 1) {
    if (pix < PIX) {
      launch_bwd_t<TW, TH, PIX / 2>(st, pix, n_tiles, groups, order, F, frames, ranges, vals, rec,
                                    keyoff, nproc, bg, g_rgb, g_depth, g_alpha, t_final, n_last,
                                    partial, stamp, epoch, med_pos, segments, maps);
      return;
    }
  }
  const auto go = [&](auto* k, int parts) {
    hipLaunchKernelGGL(k, dim3(grid_of(n_tiles, groups), (unsigned)parts), dim3(TW * TH / PIX), 0,
                       st, maps, n_tiles, groups, order, F, frames, ranges, vals, rec, keyoff,
                       nproc, bg[0], bg[1], bg[2], g_rgb, g_depth, g_alpha, t_final, n_last,
                       partial, stamp, epoch, med_pos);
  };
  if constexpr (PIX == 1) {
    if (segments > 1) {
      if (med_pos) {
        go(composite_bwd_kernel<TW, TH, 1, true, kBwdMaps>, segments - 1);
        go(composite_bwd_kernel<TW, TH, 1, true, kBwdSegments>, segments);
      } else {
        go(composite_bwd_kernel<TW, TH, 1, false, kBwdMaps>, segments - 1);
        go(composite_bwd_kernel<TW, TH, 1, false, kBwdSegments>, segments);
      }
      return;
    }
  }
  if (med_pos) go(composite_bwd_kernel<TW, TH, PIX, true, kBwdWhole>, 1);
  else go(composite_bwd_kernel<TW, TH, PIX, false, kBwdWhole>, 1);
}

void launch_composite_fwd(hipStream_t st, int tw, int th, int n_tiles, int F,
                          const FrameDesc* frames, const uint2* ranges, const uint32_t* vals,
                          const Record* rec, const float* bg, float* rgb, float* depth,
                          float* alpha, float* t_final, int32_t* n_last, uint32_t* nproc,
                          const uint32_t* prev_nproc, uint32_t* order, bool xcd_groups,
                          unsigned long long* pairs, int32_t* med_pos) {
  if (n_tiles <= 0) return;
  const int groups = xcd_groups ? kQueues : 1;
  launch_order(st, n_tiles, groups, prev_nproc, order, nproc);
#define GSR_FWD(W, H)                                                                        \
  launch_fwd_t<W, H>(st, n_tiles, groups, order, F, frames, ranges, vals, rec, bg, rgb, depth,  \
                     alpha, t_final, n_last, nproc, pairs, med_pos)
  if (tw == 16 && th == 16) GSR_FWD(16, 16);
  else if (tw == 8 && th == 8) GSR_FWD(8, 8);
  else if (tw == 32 && th == 8) GSR_FWD(32, 8);
  else if (tw == 16 && th == 8) GSR_FWD(16, 8);
  else if (tw == 32 && th == 16) GSR_FWD(32, 16);
#undef GSR_FWD
}

// Below 1.5 waves per SIMD, and with lists of two batches and more on average,
// the lists are worked on in segments.  Whole against eight segments (both
// launches), us: 2 x 131x97 (504 waves, 209 keys per tile) 83 / 46; 321x243
// (1,344 waves, 235) 80 / 62; but 400x300 (1,900, 210) 71 / 73 and 640x480
// (4,800, 965) 229 / 294, where the state pass costs more than the idle SIMDs,
// and 97x81 (168, 59), whose lists are one batch, 24 / 28.
constexpr int64_t kFewWaves = 1536;
constexpr int kSegments = 8;

int bwd_segments(uint64_t keys, int64_t n_tiles, int tw, int th) {
  const bool few = n_tiles * (tw * th / kWave) <= kFewWaves;
  return few && keys >= 2 * kBatchB * (uint64_t)n_tiles ? kSegments : 1;
}

// For every call that takes segments (11 MB), whatever the one before it took:
// a capture may follow with fewer frames, another tile shape or capacity.
size_t bwd_map_bytes() { return (size_t)kFewWaves * kWave * (kSegments - 1) * sizeof(double2); }

void launch_composite_bwd(hipStream_t st, int tw, int th, int n_tiles, int F,
                          const FrameDesc* frames, const uint2* ranges, const uint32_t* vals,
                          const Record* rec, const uint32_t* keyoff, const uint32_t* nproc,
                          const float* bg, const float* g_rgb,
                          const float* g_depth, const float* g_alpha, const float* t_final,
                          const int32_t* n_last, float* partial, uint32_t* stamp,
                          const uint32_t* epoch, uint32_t* order, bool xcd_groups,
                          const int32_t* med_pos, int segments, double2* maps) {
  if (n_tiles <= 0) return;
  const int groups = xcd_groups ? kQueues : 1;
  launch_order(st, n_tiles, groups, nproc, order);
  // Blocks per wave: as many as leave kBwdMinWaves waves (four per SIMD).  More
  // blocks per wave share an entry's overhead and its reduction, fewer keep the
  // SIMDs busy when there are few tiles.  Measured with 1 / 2 / 4 blocks (us):
  // 8 x 1200x680 (25,800 tiles of 16x16) 2802 / 2148 / 1806; 4 x 640x480
  // (4,800) 610 / 487 / 440; 1 x 640x480 (1,200) 233 / 244 / 314; 2 x 131x97
  // (126) 83 / 110 / 155; 7,800 tiles of 32x16 1522 / 1036 / 923.
  const int blocks = tw * th / kWave;
  int pix = 4;
  while (pix > 1 && (int64_t)n_tiles * blocks / pix < kBwdMinWaves) pix /= 2;
#define GSR_BWD(W, H)                                                                            \
  launch_bwd_t<W, H, std::min(4, TileBlocks<W, H>::kN)>(                                         \
      st, pix, n_tiles, groups, order, F, frames, ranges, vals, rec, keyoff, nproc, bg, g_rgb,    \
      g_depth, g_alpha, t_final, n_last, partial, stamp, epoch, med_pos,                        \
      segments, maps)
  if (tw == 16 && th == 16) GSR_BWD(16, 16);
  else if (tw == 8 && th == 8) GSR_BWD(8, 8);
  else if (tw == 32 && th == 8) GSR_BWD(32, 8);
  else if (tw == 16 && th == 8) GSR_BWD(16, 8);
  else if (tw == 32 && th == 16) GSR_BWD(32, 16);
#undef GSR_BWD
}

}  // namespace gsr
