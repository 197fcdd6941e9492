// sort.hip -- key generation and ordering of the (tile, Gaussian) lists.
//
// The compositing order of a pixel is its Gaussians by ascending (fp32 view
// depth, index) (front-to-back compositing, DROID-Splat eqn:rendering; tile
// lists of the 3DGS rasterizer it builds on).  Instead of one wide sort of
// (tile | depth) keys, the path sorts twice:
//   1. the N*F records by depth bits (stable LSD radix, 4 x 8-bit passes over
//      N*F elements), which puts each frame's Gaussians front to back with
//      ties broken by index;
//   2. keygen walks the records in that order and writes one tile id per
//      covered tile (the "slot" order), 16 bits wide while the tile ids fit
//      (up to 65,535 tiles), else 32; a stable LSD radix over only the
//      tile-id bits (two passes of <= 10 bits up to 2^20 tiles) then groups
//      the keys by tile while keeping the depth order inside each tile.
// With 16-bit keys, keygen and the two passes move 34 bytes per key, instead of
// 6-7 passes over 12-byte (tile | depth, value) pairs; the ranges search.
//
// The radix passes use a hand-written LDS multi-split: each wave ranks its
// 64 keys per round with one ballot per digit bit (lanes with equal digits
// form one mask), keeps running digit counts in LDS, and the block combines
// its waves' counts into stable block offsets; no global atomics.  A
// pass's digit counts are stored one row per block, so the histogram writes
// and the scatter reads them as whole rows, and their scan runs down the
// columns: in the scatter's blocks themselves while there are few rows (2
// launches a pass), else in 3 launches of its own.  A few thousand elements
// are ordered in one launch, by counting for each the ones in front of it.
// Scatter blocks are dealt so that consecutive blocks run on one XCD: the
// partial cache lines at the two ends of a block's digit run are completed by
// its neighbour in the same L2 instead of leaving as partial writes.  All
// kernels read the element count from device memory so the sequence is
// capturable.
#include "launch.h"

#include <algorithm>
#include <cmath>

namespace gsr {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;  // elements per block

constexpr int kScanFew = 2;  // gather: records per thread up to kGatherBig records
constexpr uint64_t kGatherBig = 1ull << 22;

constexpr int kSortRounds = 16;  // 64-key rounds per wave in the radix passes
constexpr int kMaxDigitBits = 10;
constexpr int kMaxBins = 1 << kMaxDigitBits;
constexpr unsigned kXcds = 8;  // XCDs of an MI355X: workgroup b runs on XCD b % 8

// Exclusive scan of one value per thread over a block of blockDim.x threads
// (a multiple of 64, at most 1024); wsum holds 16 values.
template <typename T>
__device__ __forceinline__ T block_scan_excl(T v, T* wsum, T& total) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
  T x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const T y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  if (lane == kWave - 1) wsum[w] = x;
  __syncthreads();
  T base = 0, tot = 0;
  for (int k = 0; k < nw; ++k) {
    const T s = wsum[k];
    if (k < w) base += s;
    tot += s;
  }
  __syncthreads();
  total = tot;
  return base + x - v;
}

// The tile counts in depth order, cnt_sorted[i] = ntiles[perm[i]], gathered
// once so that the offsets scan and keygen read them in order, together
// with the tile rects (keygen's one random read per record happens here, as
// part of the gather that has to be random anyway).  A record is kept iff its
// sorted depth key is not the all-ones of a culled record, and a kept
// record's tile count is the area of its rect (the preprocess writes the two
// together; a culled record has neither).
__device__ __forceinline__ uint32_t kept_tiles(uint32_t skey, uint32_t r,
                                               const uint2* __restrict__ trect, uint2& tr) {
  tr = make_uint2(0u, 0u);
  if (skey == 0xffffffffu) return 0u;
  tr = trect[r];
  return ((tr.x >> 16) - (tr.x & 0xffffu) + 1u) * ((tr.y >> 16) - (tr.y & 0xffffu) + 1u);
}

// Gathers a block's ITEMS * kScanThreads records (all loads of a thread in
// flight) and leaves their total.
template <int ITEMS>
__global__ void __launch_bounds__(kScanThreads) gather_counts_kernel(
    uint64_t m, const uint32_t* __restrict__ skey, const uint32_t* __restrict__ perm,
    const uint2* __restrict__ trect, uint32_t* __restrict__ cnt_sorted,
    uint2* __restrict__ trect_sorted, uint64_t* __restrict__ block_sums) {
  __shared__ uint64_t wsum[kScanThreads / kWave];
  const uint64_t base = (uint64_t)blockIdx.x * (ITEMS * kScanThreads);
  uint64_t s = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint64_t i = base + (uint64_t)k * kScanThreads + threadIdx.x;
    if (i >= m) continue;
    uint2 tr;
    const uint32_t c = kept_tiles(skey[i], perm[i], trect, tr);
    cnt_sorted[i] = c;
    trect_sorted[i] = tr;
    s += c;
  }
  for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
  if (threadIdx.x % kWave == 0) wsum[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t = 0;
    for (int w = 0; w < kScanThreads / kWave; ++w) t += wsum[w];
    block_sums[blockIdx.x] = t;
  }
}

// The total for the kernels that follow, and (unless NULL) for the host that
// waits for it.
__device__ __forceinline__ void post_total(uint64_t v, uint64_t* total, uint64_t* mailbox) {
  *total = v;
  if (mailbox) __hip_atomic_store(mailbox, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One workgroup: the sums of nb blocks become the sums in front of each.
constexpr int kSpineThreads = 1024;
__global__ void __launch_bounds__(kSpineThreads) scan_spine_kernel(uint64_t* __restrict__ sums,
                                                                   unsigned nb) {
  __shared__ uint64_t wsum[kSpineThreads / kWave];
  uint64_t run = 0, all;
  for (unsigned b0 = 0; b0 < nb; b0 += kSpineThreads) {
    const unsigned b = b0 + threadIdx.x;
    const uint64_t front = run + block_scan_excl<uint64_t>(b < nb ? sums[b] : 0u, wsum, all);
    if (b < nb) sums[b] = front;
    run += all;
  }
}

// Exclusive scan of cnt into out.  A block adds up the sums (`per` of them for
// each scan block) in front of it by itself, which costs less than a launch
// between the two kernels, or (per = 0) finds that in block_sums.  Its kScanTile
// elements pass through LDS rows of kScanItems + 1 (padded against bank
// conflicts) so that global loads and stores are coalesced while each thread
// scans kScanItems consecutive elements.
__global__ void __launch_bounds__(kScanThreads) scan_down_kernel(
    const uint32_t* __restrict__ cnt, uint64_t n, const uint64_t* __restrict__ block_sums,
    unsigned per, uint64_t* __restrict__ out, uint64_t* __restrict__ total,
    uint64_t* __restrict__ mailbox) {
  constexpr int kRow = kScanItems + 1;
  __shared__ uint64_t wsum[kScanThreads / kWave];
  __shared__ uint64_t stage[kScanThreads * kRow];
  const uint64_t b0 = (uint64_t)blockIdx.x * kScanTile;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int e = k * kScanThreads + (int)threadIdx.x;  // element of the tile
    const uint64_t i = b0 + (uint64_t)e;
    stage[(e / kScanItems) * kRow + e % kScanItems] = i < n ? (uint64_t)cnt[i] : 0u;
  }
  uint64_t front = 0, base, all;
  if (per == 0 && threadIdx.x == 0) front = block_sums[blockIdx.x];
  for (unsigned b = threadIdx.x; b < blockIdx.x * per; b += kScanThreads) front += block_sums[b];
  block_scan_excl<uint64_t>(front, wsum, base);  // (its barriers also cover stage)
  uint64_t v[kScanItems];
  uint64_t s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = stage[threadIdx.x * kRow + k];
    s += v[k];
  }
  uint64_t run = block_scan_excl<uint64_t>(s, wsum, all) + base;
  for (int k = 0; k < kScanItems; ++k) {
    stage[threadIdx.x * kRow + k] = run;
    run += v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int e = k * kScanThreads + (int)threadIdx.x;
    const uint64_t i = b0 + (uint64_t)e;
    if (i < n) out[i] = stage[(e / kScanItems) * kRow + e % kScanItems];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) post_total(base + all, total, mailbox);
}

// One workgroup: the scan of up to kScanFewThreads * 16 counts, 16 or fewer
// consecutive ones per thread.
constexpr int kScanFewThreads = 1024;
__global__ void __launch_bounds__(kScanFewThreads) scan_few_kernel(
    const uint32_t* __restrict__ cnt, uint32_t n, uint64_t* __restrict__ out,
    uint64_t* __restrict__ total, uint64_t* __restrict__ mailbox) {
  __shared__ uint64_t wsum[kScanFewThreads / kWave];
  const uint32_t per = ((n + kScanFewThreads - 1) / kScanFewThreads + 3) & ~3u;
  const uint32_t i0 = threadIdx.x * per;
  uint32_t v[16];
  uint64_t s = 0, all;
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) {
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    const uint32_t i = i0 + 4 * q;
    if (4 * q < per) {
      if (i + 4 <= n) {
        x = *reinterpret_cast<const uint4*>(cnt + i);  // i % 4 == 0
      } else {
        if (i < n) x.x = cnt[i];
        if (i + 1 < n) x.y = cnt[i + 1];
        if (i + 2 < n) x.z = cnt[i + 2];
      }
    }
    v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) s += v[k];
  uint64_t run = block_scan_excl<uint64_t>(s, wsum, all);
#pragma unroll
  for (uint32_t k = 0; k < 16; ++k) {
    if (k < per && i0 + k < n) out[i0 + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) post_total(all, total, mailbox);
}

// ---------------------------------------------------------------------------
// Stable LSD radix pass over the digit of `width` <= 10 bits at `shift`.
//
// A block of WAVES waves owns WAVES * 64 R consecutive keys, wave w the
// contiguous 64 R keys from w * 64 R as R rounds of 64 (16, or 8 where there
// are few keys).  Each lane loads its R keys and values straight into registers
// (fully unrolled, so all the loads are in flight at once).  Per round a wave
// ranks its 64 keys by digit with one ballot per digit bit, 8 or 10 whatever
// the width (lanes with equal digits form one mask); the lowest lane of each
// group bumps the wave's LDS counter.  No atomics there, so the ranks are
// deterministic and the scatter is stable.  The keys then pass through LDS in
// digit order so that each digit's run leaves the block as consecutive stores.
// BINS (256 or 1024) sizes the LDS counters; the pass uses 2^width of them.
// ---------------------------------------------------------------------------

// The lanes whose digits d agree with this lane's on the bits [0, NBITS).
// A digit narrower than NBITS has zeros above its width, where every lane
// agrees, so those steps leave the mask as it is: the loop runs a fixed
// NBITS steps with no per-bit width test.
template <int NBITS>
__device__ __forceinline__ uint64_t digit_peers(uint32_t d) {
  uint32_t m_lo = 0xffffffffu, m_hi = 0xffffffffu;
#pragma unroll
  for (int b = 0; b < NBITS; ++b) {
    // x: all ones where the lane's bit b is set; the lanes that agree with
    // it on bit b are ~(ballot ^ x), which gfx950 forms with the mask update
    // in one three-input bit operation per half (the empty asm keeps the
    // steps from being refolded into a longer xor / or chain)
    const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int32_t)d, (uint32_t)b, 1u);
    const uint64_t bb = __ballot((int32_t)x < 0);
    asm volatile("" : "+v"(m_lo), "+v"(m_hi));
    m_lo &= ~((uint32_t)bb ^ x);
    m_hi &= ~((uint32_t)(bb >> 32) ^ x);
  }
  return ((uint64_t)m_hi << 32) | m_lo;
}

// The logical block of workgroup `bid` when the grid (kXcds * per
// workgroups) is dealt so that XCD x (workgroups x, x + kXcds, ...) runs the
// consecutive logical blocks [x per, (x + 1) per) in order.  Neighbouring
// blocks write the two ends of each digit run's cache lines; on one XCD they
// meet in one L2 instead of leaving as partial-line writes.
__device__ __forceinline__ unsigned xcd_block(unsigned bid, unsigned per) {
  return (bid % kXcds) * per + bid / kXcds;
}

template <int WAVES, int R>
struct RadixShape {
  static constexpr int kThreads = WAVES * kWave;
  static constexpr int kTile = kThreads * R;  // keys per block
};

// Where a pass reads its (key, value) pairs.  kPer: keys per 16-byte load.
template <typename K>
struct StoredPairs {  // K: uint32_t, or uint16_t (tile ids below 2^16)
  using KeyT = K;
  static constexpr int kPer = 16 / (int)sizeof(K);
  const K* __restrict__ keys;
  const uint32_t* __restrict__ vals;
  __device__ uint32_t key(uint64_t i) const { return keys[i]; }
  __device__ uint32_t val(uint64_t i) const { return vals[i]; }
  __device__ void load(uint64_t i, uint32_t (&k)[kPer]) const {  // i % kPer == 0
    union {
      uint4 v;
      K k[kPer];
    } u;
    u.v = *reinterpret_cast<const uint4*>(keys + i);
#pragma unroll
    for (int t = 0; t < kPer; ++t) k[t] = u.k[t];
  }
};

// The records by size class, 0 for no key and else 1 + floor(log2 of the key
// count): the keys come from the counts and the values are the indices, so
// neither is stored.
struct SizeClasses {
  using KeyT = uint32_t;
  static constexpr int kPer = 4;
  const uint32_t* __restrict__ ntiles;
  __device__ static uint32_t of(uint32_t c) { return c == 0 ? 0u : 32u - (uint32_t)__clz(c); }
  __device__ uint32_t key(uint64_t i) const { return of(ntiles[i]); }
  __device__ uint32_t val(uint64_t i) const { return (uint32_t)i; }
  __device__ void load(uint64_t i, uint32_t (&k)[kPer]) const {
    const uint4 v = *reinterpret_cast<const uint4*>(ntiles + i);
    k[0] = of(v.x); k[1] = of(v.y); k[2] = of(v.z); k[3] = of(v.w);
  }
};
constexpr int kClassBits = 6;  // classes 0 .. 32

// Where a pass leaves its pairs: the class order keeps the values only, and
// the position of the first key at or above `mark` (the pass's count n if
// there is none) unless `first` is NULL.
template <typename K>
struct StorePairs {
  K* __restrict__ keys;
  uint32_t* __restrict__ vals;
  __device__ void put(uint32_t i, uint32_t k, uint32_t v) const {
    keys[i] = (K)k;
    vals[i] = v;
  }
  __device__ void start(uint32_t, uint32_t) const {}
};
struct StoreOrder {
  uint32_t* __restrict__ vals;
  uint32_t mark;
  uint32_t* first;
  __device__ void put(uint32_t i, uint32_t, uint32_t v) const { vals[i] = v; }
  __device__ void start(uint32_t d, uint32_t at) const {
    if (first && d == mark) *first = at;
  }
};

// Digit counts of one block's keys.  A count does not depend on the order,
// so each thread loads 16 bytes of keys at once and bumps LDS counters with
// atomics.  The rate of these bounds the kernel (about 23 clocks per wave and
// key), and lanes of one wave that meet in a counter are served one after the
// other: with up to 256 digits a wave has four copies of its counters, 16
// banks apart, for the lanes mod 4.  All are summed at the end.  111M 16-bit
// keys: 77 us with one copy, 67 with four (2M 32-bit keys, 256 digits: 6.4 / 4.9).
template <int BINS, int WAVES, int R, typename Load>
__global__ void __launch_bounds__(256) radix_hist_kernel(
    Load in, const uint64_t* n_dev, uint64_t n_host, int shift,
    int width, uint32_t* __restrict__ hist /* [nblocks][2^width] */) {
  constexpr int kTile = RadixShape<WAVES, R>::kTile;
  constexpr int kHW = 256 / kWave;  // waves of this kernel
  constexpr int kPer = Load::kPer;
  static_assert(kTile % (kPer * 256) == 0, "whole 16-byte loads");
  constexpr int kCopies = BINS == 256 ? 4 : 1;
  constexpr int kStride = BINS + (kCopies > 1 ? 16 : 0);
  __shared__ uint32_t wcnt[kHW * kCopies][kStride];
  const uint64_t n = n_dev ? min(*n_dev, n_host) : n_host;
  const int bins = 1 << width;
  const uint32_t mask = (uint32_t)bins - 1u;
  const int w = threadIdx.x / kWave;
  for (int i = threadIdx.x; i < kHW * kCopies * kStride; i += 256) (&wcnt[0][0])[i] = 0;
  __syncthreads();
  const uint64_t bbase = (uint64_t)blockIdx.x * kTile;
  uint32_t* cw = wcnt[w * kCopies + (threadIdx.x & (kCopies - 1))];
#pragma unroll
  for (int j = 0; j < kTile / (kPer * 256); ++j) {
    const uint64_t i = bbase + kPer * ((uint64_t)threadIdx.x + (uint64_t)j * 256);
    if (i + kPer <= n) {
      uint32_t k[kPer];
      in.load(i, k);
#pragma unroll
      for (int t = 0; t < kPer; ++t) atomicAdd(&cw[(k[t] >> shift) & mask], 1u);
    } else {
      for (uint64_t t = i; t < n && t < i + kPer; ++t)
        atomicAdd(&cw[(in.key(t) >> shift) & mask], 1u);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < bins; d += 256) {
    uint32_t c = 0;
    for (int ww = 0; ww < kHW * kCopies; ++ww) c += wcnt[ww][d];
    hist[(uint64_t)blockIdx.x * bins + d] = c;
  }
}

// Exclusive offsets from the block-major counts H[b][d]: the scatter of block
// b puts its digit-d keys at sum_{d' < d} total(d') + sum_{b' < b} H[b'][d],
// the exclusive scan of the counts taken in (digit, block) order.  The blocks
// are cut into chunks of `rows`; one thread per digit walks a chunk's rows,
// so every access is a whole row.  Rows are loaded kColBatch at a time so
// that a thread's serial walk waits on one load latency per batch.
// rows = ceil(sqrt(nb)) balances a chunk's walk against the spine's walk
// over the chunks; then there are at most ceil(sqrt(nb)) chunks (and at most
// kColMaxChunks).  The three kernels run max(bins, 64) threads; threads past
// the digit count only take part in the spine's block scan.
constexpr unsigned kColMaxChunks = 1024;
constexpr int kColBatch = 16;

static inline uint64_t isqrt_ceil(uint64_t x) {
  uint64_t r = (uint64_t)std::sqrt((double)x);
  while (r * r < x) ++r;
  while (r > 0 && (r - 1) * (r - 1) >= x) --r;
  return r;
}

static inline unsigned col_rows(unsigned nb) {
  return (unsigned)std::max<uint64_t>(isqrt_ceil(nb), (nb + kColMaxChunks - 1) / kColMaxChunks);
}

// csum[c][d] = sum of H[b][d] over the rows b of chunk c
__global__ void __launch_bounds__(kMaxBins) radix_colsum_kernel(
    const uint32_t* __restrict__ hist, unsigned nb, unsigned rows, int bins,
    uint32_t* __restrict__ csum) {
  const unsigned d = threadIdx.x;
  if ((int)d >= bins) return;
  const unsigned b0 = blockIdx.x * rows, b1 = min(nb, b0 + rows);
  uint32_t s = 0;
  for (unsigned b = b0; b < b1; b += kColBatch) {
    uint32_t v[kColBatch];
#pragma unroll
    for (int j = 0; j < kColBatch; ++j)
      v[j] = b + j < b1 ? hist[(uint64_t)(b + j) * bins + d] : 0u;
#pragma unroll
    for (int j = 0; j < kColBatch; ++j) s += v[j];
  }
  csum[(uint64_t)blockIdx.x * bins + d] = s;
}

// One block: csum[c][d] becomes the exclusive scan over chunks of digit d;
// row nc receives the exclusive scan of the digit totals.
__global__ void __launch_bounds__(kMaxBins) radix_colspine_kernel(uint32_t* __restrict__ csum,
                                                                  unsigned nc, int bins) {
  __shared__ uint32_t wsum[kMaxBins / kWave];
  const unsigned d = threadIdx.x;
  const bool own = (int)d < bins;
  uint32_t run = 0;
  if (own) {
    for (unsigned c = 0; c < nc; c += kColBatch) {
      uint32_t v[kColBatch];
#pragma unroll
      for (int j = 0; j < kColBatch; ++j)
        v[j] = c + j < nc ? csum[(uint64_t)(c + j) * bins + d] : 0u;
#pragma unroll
      for (int j = 0; j < kColBatch; ++j)
        if (c + j < nc) {
          csum[(uint64_t)(c + j) * bins + d] = run;
          run += v[j];
        }
    }
  }
  uint32_t total;
  const uint32_t base = block_scan_excl<uint32_t>(run, wsum, total);
  if (own) csum[(uint64_t)nc * bins + d] = base;
}

// H[b][d] becomes block b's global start of digit d
__global__ void __launch_bounds__(kMaxBins) radix_coldown_kernel(
    uint32_t* __restrict__ hist, unsigned nb, unsigned rows, int bins,
    const uint32_t* __restrict__ csum, unsigned nc) {
  const unsigned d = threadIdx.x;
  if ((int)d >= bins) return;
  const unsigned b0 = blockIdx.x * rows, b1 = min(nb, b0 + rows);
  uint32_t run = csum[(uint64_t)blockIdx.x * bins + d] + csum[(uint64_t)nc * bins + d];
  for (unsigned b = b0; b < b1; b += kColBatch) {
    uint32_t v[kColBatch];
#pragma unroll
    for (int j = 0; j < kColBatch; ++j)
      v[j] = b + j < b1 ? hist[(uint64_t)(b + j) * bins + d] : 0u;
#pragma unroll
    for (int j = 0; j < kColBatch; ++j)
      if (b + j < b1) {
        hist[(uint64_t)(b + j) * bins + d] = run;
        run += v[j];
      }
  }
}

template <int BINS, int WAVES, int R>
struct ScatterLds {
  uint32_t wcnt[WAVES][BINS];  // counts, then each wave's block-local start in digit
  uint32_t gofs[BINS];         // global start of digit d minus its block-local start
  uint32_t wsum[WAVES];
  uint32_t sk[RadixShape<WAVES, R>::kTile], sv[RadixShape<WAVES, R>::kTile];
};

// Ranks the block's keys (lane's round-k key is block-local index
// w 64 R + 64 k + lane; L.wcnt zeroed and the zeroing visible to all waves),
// moves them into digit order through L.sk / L.sv and writes them to
// (global start of digit d) + (position inside the block's run of digit d).
// The combine folds the block-local digit starts into the waves' bases and
// the global offsets, so that each key reads one LDS word on its way into
// the staging rows and one on its way out.  offs: the global starts of the
// DPT digits that this thread combines.
template <int BINS, int WAVES, int R, int DPT, typename Store>
__device__ __forceinline__ void rank_and_scatter(ScatterLds<BINS, WAVES, R>& L,
                                                 const uint32_t (&key)[R],
                                                 const uint32_t (&val)[R],
                                                 uint32_t nkeys, int shift, int width,
                                                 const uint32_t (&offs)[DPT],
                                                 const Store& out) {
  constexpr int kThreads = RadixShape<WAVES, R>::kThreads;
  static_assert(BINS == 256 || BINS == kMaxBins, "8- or 10-bit digit counters");
  constexpr int kBinBits = BINS == 256 ? 8 : kMaxDigitBits;
  const int bins = 1 << width;
  const uint32_t mask = (uint32_t)bins - 1u;
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  const uint32_t wbase = (uint32_t)w * (kWave * R);
  const uint32_t wbase_s = __builtin_amdgcn_readfirstlane(wbase);  // wave-uniform
  uint32_t rank[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const uint32_t i = wbase + (uint32_t)k * kWave + lane;
    const bool valid = i < nkeys;
    const uint32_t d = (key[k] >> shift) & mask;
    uint64_t m = digit_peers<kBinBits>(d);
    if (wbase_s + (uint32_t)k * kWave + kWave > nkeys) m &= __ballot(valid);  // partial round
    // LDS ops of one wave complete in issue order: the read precedes the
    // leader's write of the same counter
    const uint32_t before = L.wcnt[w][d];
    // peers below this lane: mbcnt counts the mask's bits under the lane
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    rank[k] = before + below;
    if (valid && below == 0) L.wcnt[w][d] = before + (uint32_t)__popcll(m);
  }
  __syncthreads();
  {
    // thread t owns digits [t DPT, t DPT + DPT): wave bases per digit, then
    // the block-local digit starts by a scan over the threads
    uint32_t tot[DPT];
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      const int d = threadIdx.x * DPT + j;
      uint32_t run = 0;
      if (d < bins) {
        for (int ww = 0; ww < WAVES; ++ww) {
          const uint32_t c = L.wcnt[ww][d];
          L.wcnt[ww][d] = run;
          run += c;
        }
      }
      tot[j] = run;
      mine += run;
    }
    uint32_t total;
    uint32_t base = block_scan_excl<uint32_t>(mine, L.wsum, total);
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      const int d = threadIdx.x * DPT + j;
      if (d < bins) {
        for (int ww = 0; ww < WAVES; ++ww) L.wcnt[ww][d] += base;
        L.gofs[d] = offs[j] - base;  // mod 2^32: the output index adds base back
      }
      base += tot[j];
    }
  }
  __syncthreads();  // (also: every wave is done with whatever L.sk held)
  // A full block (all but the last) takes the loops without a per-key test,
  // so that the unrolled rounds' LDS reads are all in flight before the
  // dependent writes and stores; the test made each round wait for its own.
  const bool full = nkeys == (uint32_t)RadixShape<WAVES, R>::kTile;  // block-uniform
  if (full) {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t lp = L.wcnt[w][__builtin_amdgcn_ubfe(key[k], shift, width)] + rank[k];
      L.sk[lp] = key[k];
      L.sv[lp] = val[k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t i = wbase + (uint32_t)k * kWave + lane;
      if (i < nkeys) {
        const uint32_t lp = L.wcnt[w][__builtin_amdgcn_ubfe(key[k], shift, width)] + rank[k];
        L.sk[lp] = key[k];
        L.sv[lp] = val[k];
      }
    }
  }
  __syncthreads();
  // R slots per thread: consecutive threads take consecutive
  // slots, so each digit's run leaves as consecutive stores
  if (full) {
    uint32_t kk[R], vv[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t idx = threadIdx.x + (uint32_t)k * kThreads;
      kk[k] = L.sk[idx];
      vv[k] = L.sv[idx];
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t idx = threadIdx.x + (uint32_t)k * kThreads;
      const uint32_t dst = L.gofs[__builtin_amdgcn_ubfe(kk[k], shift, width)] + idx;
      out.put(dst, kk[k], vv[k]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t idx = threadIdx.x + (uint32_t)k * kThreads;
      if (idx < nkeys) {
        const uint32_t kk = L.sk[idx];
        const uint32_t dst = L.gofs[__builtin_amdgcn_ubfe(kk, shift, width)] + idx;
        out.put(dst, kk, L.sv[idx]);
      }
    }
  }
}

// offsets: the block-major digit counts, scanned by the column kernels or
// (FOLD) as the histogram left them.  With FOLD a block walks down the whole
// columns itself: the counts in front of it and the digit totals, whose scan
// over the digits completes the starts.
template <int BINS, int WAVES, int R, bool FOLD, typename Load, typename Store>
__global__ void __launch_bounds__(WAVES * kWave) radix_scatter_kernel(
    Load in, const uint64_t* n_dev, uint64_t n_host, int shift, int width, unsigned nb,
    unsigned per, const uint32_t* __restrict__ offsets /* [nblocks][2^width] */, Store out) {
  constexpr int kThreads = RadixShape<WAVES, R>::kThreads;
  constexpr int kTile = RadixShape<WAVES, R>::kTile;
  constexpr int DPT = (BINS + kThreads - 1) / kThreads;  // digits per thread in the combine
  __shared__ ScatterLds<BINS, WAVES, R> L;
  const unsigned b = xcd_block(blockIdx.x, per);
  if (b >= nb) return;  // padding workgroup: before any barrier
  const uint64_t n = n_dev ? min(*n_dev, n_host) : n_host;
  const uint64_t bbase = (uint64_t)b * kTile;
  const uint32_t nkeys = (uint32_t)(n > bbase ? min((uint64_t)kTile, n - bbase) : 0);
  for (int i = threadIdx.x; i < WAVES * BINS; i += kThreads) (&L.wcnt[0][0])[i] = 0;
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wbase = (uint32_t)(threadIdx.x / kWave) * (kWave * R);
  uint32_t key[R], val[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const uint32_t i = wbase + (uint32_t)k * kWave + lane;
    key[k] = i < nkeys ? in.key(bbase + i) : 0u;
    val[k] = i < nkeys ? in.val(bbase + i) : 0u;
  }
  const unsigned bins = 1u << width;
  const unsigned d0 = threadIdx.x * DPT;
  uint32_t offs[DPT];
  if constexpr (FOLD) {
    constexpr int kBatch = kColBatch / DPT;
    uint32_t tot[DPT], mine = 0;
#pragma unroll
    for (int j = 0; j < DPT; ++j) offs[j] = tot[j] = 0;
    // fewer digits than threads: every parts-th row each, so that the threads
    // read whole lines; bins % DPT == 0 (DPT is 1, or 4 with 512 digits or more)
    const unsigned parts = DPT == 1 ? max((unsigned)kThreads >> width, 1u) : 1u;
    const unsigned part = DPT == 1 ? threadIdx.x >> width : 0u;
    const unsigned dw = DPT == 1 ? threadIdx.x & (bins - 1) : d0;
    if (part < parts && dw < bins) {
      for (unsigned r0 = part; r0 < nb; r0 += kBatch * parts) {
        uint32_t v[kBatch][DPT];
#pragma unroll
        for (int r = 0; r < kBatch; ++r)
#pragma unroll
          for (int j = 0; j < DPT; ++j)
            v[r][j] = r0 + r * parts < nb ? offsets[(uint64_t)(r0 + r * parts) * bins + dw + j]
                                          : 0u;
#pragma unroll
        for (int r = 0; r < kBatch; ++r)
#pragma unroll
          for (int j = 0; j < DPT; ++j) {
            tot[j] += v[r][j];
            offs[j] += r0 + r * parts < b ? v[r][j] : 0u;
          }
      }
    }
    if (DPT == 1 && parts > 1) {  // uniform
      L.sk[threadIdx.x] = tot[0];
      L.sv[threadIdx.x] = offs[0];
      __syncthreads();
      tot[0] = offs[0] = 0;
      if (threadIdx.x < bins)
        for (unsigned q = 0; q < parts; ++q) {
          tot[0] += L.sk[q * bins + threadIdx.x];
          offs[0] += L.sv[q * bins + threadIdx.x];
        }
    }
#pragma unroll
    for (int j = 0; j < DPT; ++j) mine += tot[j];
    uint32_t all;
    uint32_t run = block_scan_excl<uint32_t>(mine, L.wsum, all);
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      offs[j] += run;
      run += tot[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < DPT; ++j)
      offs[j] = d0 + j < bins ? offsets[(uint64_t)b * bins + d0 + j] : 0u;
  }
  if (b == 0)
#pragma unroll
    for (int j = 0; j < DPT; ++j) out.start(d0 + j, offs[j]);
  __syncthreads();
  rank_and_scatter<BINS, WAVES, R, DPT, Store>(L, key, val, nkeys, shift, width, offs, out);
}

// ---------------------------------------------------------------------------
// Few elements: the position of an element in the stable order is the number
// of elements in front of it, counted outright.  A workgroup takes 64
// elements, one per lane, and each of its 16 waves counts over a sixteenth
// of all keys, which arrive as scalars (two VALU instructions per pair); the
// counts meet in LDS and the first wave moves the elements.
//
// An element precedes this lane's if its key is <= `le` (elements with a lower
// index) or < `lt` (elements with a higher one).
// ---------------------------------------------------------------------------
constexpr int kRankWaves = 16;
constexpr unsigned kRankBatch = 16;  // keys per scalar load

// The number of elements in front of this lane's element blockIdx.x * 64 +
// lane, valid in the first wave.
template <typename KeyT>
__device__ __forceinline__ uint32_t rank_of(const KeyT* __restrict__ keys, uint32_t n, uint32_t le,
                                            uint32_t lt) {
  __shared__ uint32_t part[kRankWaves][kWave];
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t own = blockIdx.x * kWave;
  const uint32_t chunk = ((n + kRankWaves - 1) / kRankWaves + kRankBatch - 1) / kRankBatch *
                         kRankBatch;
  const uint32_t j1 = min(n, (w + 1) * chunk);
  uint32_t c = 0;
  uint32_t j = w * chunk;
  for (; j + kRankBatch <= j1; j += kRankBatch) {
    // (the buffers are 16-byte aligned and j % 16 == 0)
    constexpr unsigned kPack = 4 / sizeof(KeyT);
    uint32_t k[kRankBatch];
    const uint32_t* words = reinterpret_cast<const uint32_t*>(keys + j);
#pragma unroll
    for (unsigned t = 0; t < kRankBatch; ++t)
      k[t] = kPack == 1 ? words[t] : words[t / kPack] >> (16 * (t % kPack)) & 0xffffu;
    if (j + kRankBatch <= own) {
#pragma unroll
      for (unsigned t = 0; t < kRankBatch; ++t) c += k[t] <= le ? 1u : 0u;
    } else if (j >= own + kWave) {
#pragma unroll
      for (unsigned t = 0; t < kRankBatch; ++t) c += k[t] < lt ? 1u : 0u;
    } else {
#pragma unroll
      for (unsigned t = 0; t < kRankBatch; ++t)
        c += (j + t < own + lane ? k[t] <= le : k[t] < lt) ? 1u : 0u;
    }
  }
  for (; j < j1; ++j) c += (j < own + lane ? keys[j] <= le : keys[j] < lt) ? 1u : 0u;
  part[w][lane] = c;
  __syncthreads();
  uint32_t r = 0;
#pragma unroll
  for (int v = 0; v < kRankWaves; ++v) r += part[v][lane];
  return r;
}

// Stable sort of min(*n_dev, n_max) pairs (n_dev NULL: n_max).
template <typename KeyT>
__global__ void __launch_bounds__(kRankWaves* kWave) rank_pairs_kernel(
    const KeyT* __restrict__ keys, const uint32_t* __restrict__ vals, const uint64_t* n_dev,
    uint32_t n_max, KeyT* __restrict__ keys_out, uint32_t* __restrict__ vals_out) {
  const uint32_t n = n_dev ? (uint32_t)min(*n_dev, (uint64_t)n_max) : n_max;
  const uint32_t i = blockIdx.x * kWave + (threadIdx.x & (kWave - 1));
  if (blockIdx.x * kWave >= n) return;  // uniform
  const uint32_t k = i < n ? (uint32_t)keys[i] : 0u;
  const uint32_t r = rank_of(keys, n, k, k);
  if (threadIdx.x >= kWave || i >= n) return;
  keys_out[r] = (KeyT)k;
  vals_out[r] = vals[i];
}

// The depth sort, with each record's tile rect and count (kept_tiles).
__global__ void __launch_bounds__(kRankWaves* kWave) rank_records_kernel(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint32_t n,
    const uint2* __restrict__ trect, uint32_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, uint32_t* __restrict__ cnt_sorted,
    uint2* __restrict__ trect_sorted) {
  const uint32_t i = blockIdx.x * kWave + (threadIdx.x & (kWave - 1));
  const uint32_t k = i < n ? keys[i] : 0u;
  const uint32_t r = rank_of(keys, n, k, k);
  if (threadIdx.x >= kWave || i >= n) return;
  const uint32_t v = vals[i];
  uint2 tr;
  const uint32_t c = kept_tiles(k, v, trect, tr);
  keys_out[r] = k;
  vals_out[r] = v;
  cnt_sorted[r] = c;
  trect_sorted[r] = tr;
}

// The class order.  Lane n stands for the mark: the records whose count lies
// below 2^(mark - 1) are the ones of a lower class.
__global__ void __launch_bounds__(kRankWaves* kWave) rank_classes_kernel(
    const uint32_t* __restrict__ ntiles, uint32_t n, StoreOrder out) {
  const uint32_t i = blockIdx.x * kWave + (threadIdx.x & (kWave - 1));
  const uint32_t k = i < n ? ntiles[i] : 0u;
  // bits of the count set to ones: the largest count of its class
  uint32_t le = k ? 0xffffffffu >> __clz(k) : 0u;
  const uint32_t lt = k ? (le >> 1) + 1u : 0u;
  if (i == n) le = out.mark ? (1u << (out.mark - 1)) - 1u : 0u;
  const uint32_t r = rank_of(ntiles, n, le, lt);
  if (threadIdx.x >= kWave) return;
  if (i < n) out.put(r, 0u, i);
  if (i == n) out.start(out.mark, r);
}

// q = floor(a / b), r = a - q b for b >= 1: a float estimate corrected by
// one step each way (exact while a < 2^21, where the estimate is off by at
// most one), else the integer division.
__device__ __forceinline__ uint32_t div_rem(uint32_t a, uint32_t b, uint32_t& r) {
  if (a >= (1u << 21)) {
    const uint32_t q = a / b;
    r = a - q * b;
    return q;
  }
  uint32_t q = (uint32_t)((float)a * __builtin_amdgcn_rcpf((float)b));
  int32_t rr = (int32_t)(a - q * b);
  if (rr < 0) {
    --q;
    rr += (int32_t)b;
  } else if (rr >= (int32_t)b) {
    ++q;
    rr -= (int32_t)b;
  }
  r = (uint32_t)rr;
  return q;
}

// ---------------------------------------------------------------------------
// keygen: key slot o (0 <= o < K) belongs to the depth-ordered record i with
// offsets[i] <= o < offsets[i] + cnt[i]; its key is the global id of the
// (o - offsets[i])-th tile of the record's tile rect, row by row, and its
// value the record id perm[i].  A wave owns 64 consecutive depth-ordered
// records; their slots form one contiguous range, which the lanes write
// cooperatively (slot o by lane o % 64, every store instruction 64
// consecutive keys).  The owner of each slot of a 64-slot round comes from
// the record starts that fall in the round: those records mark their slot in
// LDS, and a slot's owner is the number of records started at or before it,
// less one (one LDS write, one read and a ballot per round; a binary search
// over the 64 starts took six dependent LDS reads and twice the VALU work,
// and this kernel is bound by VALU issue).  A record whose slots pass the key
// capacity gets the all-ones sentinel key (past every tile) on its slots
// below the capacity.
// ---------------------------------------------------------------------------
template <typename KeyT>
__global__ void __launch_bounds__(256) keygen_kernel(
    uint64_t m, uint64_t n, const uint32_t* __restrict__ perm,
    const uint32_t* __restrict__ cnt_sorted, const uint64_t* __restrict__ offsets,
    uint32_t* __restrict__ keyoff, const uint2* __restrict__ trect_sorted,
    const FrameDesc* __restrict__ frames, uint64_t capacity, KeyT* __restrict__ keys,
    uint32_t* __restrict__ vals, uint32_t* __restrict__ overflow) {
  // per record: (first tile id or sentinel, rect width | grid width << 16,
  // value, first slot relative to the wave's first); per slot of a round:
  // the round's number where a record starts there.  Each wave uses its own
  // rows.
  __shared__ uint4 s_rec[4][kWave];
  __shared__ uint32_t s_mark[4][kWave];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint64_t i0 = ((uint64_t)blockIdx.x * 4 + w) * kWave;
  const uint64_t i = i0 + lane;
  uint32_t cnt = 0;
  uint64_t off = 0;
  if (i < m) {
    cnt = cnt_sorted[i];
    off = offsets[i];
    if (cnt) {
      const uint32_t r = perm[i];
      const uint2 tr = trect_sorted[i];
      const FrameDesc fr = frames[r / (uint32_t)n];
      const uint32_t tx0 = tr.x & 0xffffu, tx1 = tr.x >> 16, ty0 = tr.y & 0xffffu;
      const bool ovf = off + cnt > capacity;
      keyoff[r] = ovf ? 0xffffffffu : (uint32_t)off;
      if (ovf) atomicOr(overflow, 1u);
      s_rec[w][lane] =
          make_uint4(ovf ? 0xffffffffu : (uint32_t)fr.tile_offset + ty0 * (uint32_t)fr.grid_x + tx0,
                     (tx1 - tx0 + 1u) | ((uint32_t)fr.grid_x << 16), ovf ? 0u : r, 0u);
    }
  }
  // contiguous slot range [lo, hi) of the wave's records
  const uint64_t lo = __shfl(off, 0, kWave);
  uint64_t hi = i < m ? off + cnt : 0;
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t h2 = __shfl_xor(hi, o, kWave);
    hi = h2 > hi ? h2 : hi;
  }
  if (hi > capacity) hi = capacity;
  if (i0 >= m || hi <= lo) return;  // wave-uniform
  // records with a slot in the range have first slots below hi; the others
  // (culled, or past the capacity) never own a slot.  The starts of the
  // records with slots increase strictly along the lanes from 0.
  const uint32_t start = (i < m && cnt && off < hi) ? (uint32_t)(off - lo) : 0xffffffffu;
  s_rec[w][lane].w = start;
  s_mark[w][lane] = 0u;
  const uint32_t span = (uint32_t)(hi - lo);  // < 2^32: slots are 32-bit
  // the wave's output runs, from wave-uniform bases
  const uint64_t lo_s = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(lo >> 32)) << 32) |
                        __builtin_amdgcn_readfirstlane((uint32_t)lo);
  KeyT* __restrict__ kout = keys + lo_s;
  uint32_t* __restrict__ vout = vals + lo_s;
  uint32_t before = 0;  // records starting before the round
  uint32_t round = 0;
  for (uint32_t base = 0; base < span; base += kWave) {
    // owner of slot base + lane: the last record starting at or before it.
    // Records starting inside the window mark their slot with the round's
    // number (distinct slots, so no two lanes write one word); LDS ops of
    // one wave complete in issue order, so the marks are in place when the
    // lanes read them.
    ++round;
    if (start != 0xffffffffu && start - base < (uint32_t)kWave) s_mark[w][start - base] = round;
    __builtin_amdgcn_wave_barrier();
    const uint64_t sm = __ballot(s_mark[w][lane] == round);
    const uint32_t upto =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(sm >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)sm, 0u)) +
        (uint32_t)((sm >> lane) & 1ull);
    const uint32_t owner = (before + upto - 1u) & (kWave - 1);
    before += (uint32_t)__popcll(sm);
    const uint32_t o = base + (uint32_t)lane;
    const uint4 R = s_rec[w][owner];
    if (o < span) {
      uint32_t key = 0xffffffffu;
      if (R.x != 0xffffffffu) {
        uint32_t col;
        const uint32_t row = div_rem(o - R.w, R.y & 0xffffu, col);
        key = R.x + row * (R.y >> 16) + col;
      }
      kout[o] = (KeyT)key;  // the sentinel stays all ones
      vout[o] = R.z;
    }
  }
}

// [start, end) of every tile's run in the sorted keys, (0, 0) if it has none.
// A lane finds its tile's start (the number of keys below it) by binary
// search, and the next lane's start is its end; a wave covers 63 tiles.
template <typename KeyT>
__global__ void __launch_bounds__(256) ranges_kernel(const KeyT* __restrict__ keys,
                                                     const uint64_t* k_dev, uint64_t capacity,
                                                     uint2* __restrict__ ranges,
                                                     uint32_t n_tiles) {
  const uint32_t K = (uint32_t)(*k_dev < capacity ? *k_dev : capacity);
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t t = ((uint64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave) * (kWave - 1) +
                     lane;
  uint32_t lo = 0, len = K;
  while (len > 0) {  // uniform: len does not depend on the outcomes
    const uint32_t half = len / 2;
    // keys[lo + half] is inside [lo, lo + len)
    const bool right = (uint64_t)keys[lo + half] < t;
    lo = right ? lo + half + (len & 1 ? 1u : 0u) : lo;
    len = half;
  }
  const uint32_t end = __shfl_down(lo, 1, kWave);
  if (lane < kWave - 1 && t < n_tiles)
    ranges[t] = end > lo ? make_uint2(lo, end) : make_uint2(0u, 0u);
}

// Plain copy, one 16-byte element per thread: the reference for the
// achievable HBM bandwidth that the sort's fraction is taken against.
__global__ void __launch_bounds__(256) copy16_kernel(const uint4* __restrict__ a,
                                                     uint4* __restrict__ b, uint64_t n) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) b[i] = a[i];
}

void launch_copy16(hipStream_t st, const void* src, void* dst, uint64_t n16) {
  if (n16 == 0) return;
  hipLaunchKernelGGL(copy16_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, st,
                     static_cast<const uint4*>(src), static_cast<uint4*>(dst), n16);
}

// Frame descriptors passed by value as kernel arguments (at most 64 per
// launch: 3 KB of the 4 KB argument space), so that a captured graph keeps
// each forward's own table.
constexpr int kFramesPerLaunch = 64;
struct FrameBatch {
  FrameDesc f[kFramesPerLaunch];
};

__global__ void set_frames_kernel(FrameBatch b, int count, FrameDesc* __restrict__ dst) {
  const int i = threadIdx.x;
  if (i < count) dst[i] = b.f[i];
}

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, uint64_t n, uint32_t v) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// host-side launch sequences
// ---------------------------------------------------------------------------
static inline unsigned blocks_for(uint64_t n, uint64_t per) {
  return (unsigned)((n + per - 1) / per);
}

void launch_set_frames(hipStream_t st, const FrameDesc* host, int n, FrameDesc* dst) {
  for (int i0 = 0; i0 < n; i0 += kFramesPerLaunch) {
    FrameBatch b{};
    const int c = std::min(kFramesPerLaunch, n - i0);
    std::copy(host + i0, host + i0 + c, b.f);
    hipLaunchKernelGGL(set_frames_kernel, dim3(1), dim3(kFramesPerLaunch), 0, st, b, c,
                       dst + i0);
  }
}

void launch_fill_u32(hipStream_t st, uint32_t* p, uint64_t n, uint32_t v) {
  if (n == 0) return;
  hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, p, n, v);
}

// Digit widths of the tile passes: ceil(bits / kMaxDigitBits) passes of
// near-equal width, the narrower ones first (fewer digits make longer runs
// per block).
static int tile_pass_widths(int bits, int* widths) {
  const int passes = std::max(1, (bits + kMaxDigitBits - 1) / kMaxDigitBits);
  const int base = bits / passes, extra = bits % passes;
  for (int p = 0; p < passes; ++p) widths[p] = base + (p >= passes - extra ? 1 : 0);
  return passes;
}

static int max_digit_width(int bits) {
  int w[8];
  const int passes = tile_pass_widths(bits, w);
  int mx = 1;
  for (int p = 0; p < passes; ++p) mx = std::max(mx, w[p]);
  return mx;
}

// Up to this many counts, and this many read by all blocks together, every
// scatter block walks down the columns itself, which takes the three column
// kernels out of the pass.  The first bounds a block's own serial walk, the
// second what the walks of many blocks cost in all.  Scatter alone against
// column kernels + scatter (us; three launches saved are worth 6 more): 256
// digits, 32 blocks 10 / 8 + 8, 147 blocks 18 / 14 + 10, 244 blocks 25 / 14 +
// 12; 64 digits, 512 blocks 18 / 14 + 11, 1,024 blocks 36 / 14 + 16; 32 digits,
// 1,200 blocks 35 / 13 + 18, 1,536 blocks 43 / 11 + 20, 2,048 blocks 63 / 12 +
// 25; 8 digits, 2,048 blocks 38 / 14 + 26, 4,096 blocks 83 / 14 + 47.
constexpr uint64_t kFoldCounts = 1u << 16;
constexpr uint64_t kFoldReads = 3u << 24;

constexpr bool walk_columns(uint64_t nb, int width) {
  return (nb << width) <= kFoldCounts && ((nb * nb) << width) <= kFoldReads;
}

// Workspace bounds use the smallest block of a pass with column kernels (4
// waves, 4096 keys); the others have at most kFoldCounts counts.
size_t radix_hist_elems(uint64_t n_max, int bits) {
  const int wmax = bits > 0 ? max_digit_width(bits) : 8;
  const size_t blocks = blocks_for(n_max, RadixShape<4, kSortRounds>::kTile);
  return std::max<size_t>(kFoldCounts, blocks << std::max(wmax, 8));
}
// (not fewer for a larger count)
size_t scan_block_elems(uint64_t n_max) {
  return std::max(blocks_for(std::min(n_max, kGatherBig), kScanFew * kScanThreads),
                  blocks_for(n_max, kScanTile));
}
// u32 elements of the column scan's chunk sums for up to n_max keys (an upper
// bound for every smaller count as well)
size_t radix_scan_elems(uint64_t n_max, int bits) {
  const int wmax = bits > 0 ? max_digit_width(bits) : 8;
  const uint64_t nb = blocks_for(n_max, RadixShape<4, kSortRounds>::kTile);
  const uint64_t nc = std::min<uint64_t>(isqrt_ceil(nb), kColMaxChunks);
  return (size_t)(nc + 1) << std::max(wmax, 8);
}

// Column scan of the block-major digit counts into per-block digit starts.
static void radix_offsets(hipStream_t st, uint32_t* hist, unsigned nb, int width,
                          uint32_t* scan_tmp) {
  const int bins = 1 << width;
  const unsigned rows = col_rows(nb);
  const unsigned nc = (nb + rows - 1) / rows;
  const unsigned thr = (unsigned)std::max(bins, kWave);
  hipLaunchKernelGGL(radix_colsum_kernel, dim3(nc), dim3(thr), 0, st, hist, nb, rows, bins,
                     scan_tmp);
  hipLaunchKernelGGL(radix_colspine_kernel, dim3(1), dim3(thr), 0, st, scan_tmp, nc, bins);
  hipLaunchKernelGGL(radix_coldown_kernel, dim3(nc), dim3(thr), 0, st, hist, nb, rows, bins,
                     scan_tmp, nc);
}

template <int BINS, int WAVES, int R, typename Load, typename Store>
static void radix_pass(hipStream_t st, Load in, Store out, const uint64_t* n_dev, uint64_t n_max,
                       int shift, int width, uint32_t* hist, uint32_t* scan_tmp) {
  const unsigned nb = blocks_for(n_max, RadixShape<WAVES, R>::kTile);
  const unsigned per = (nb + kXcds - 1) / kXcds;
  const dim3 grid(per * kXcds), block(RadixShape<WAVES, R>::kThreads);
  hipLaunchKernelGGL((radix_hist_kernel<BINS, WAVES, R, Load>), dim3(nb), dim3(256), 0, st, in,
                     n_dev, n_max, shift, width, hist);
  if (walk_columns(nb, width)) {
    hipLaunchKernelGGL((radix_scatter_kernel<BINS, WAVES, R, true, Load, Store>), grid, block, 0,
                       st, in, n_dev, n_max, shift, width, nb, per, hist, out);
    return;
  }
  radix_offsets(st, hist, nb, width, scan_tmp);
  hipLaunchKernelGGL((radix_scatter_kernel<BINS, WAVES, R, false, Load, Store>), grid, block, 0, st,
                     in, n_dev, n_max, shift, width, nb, per, hist, out);
}

// Large passes take 8-wave blocks (longer digit runs per block); small ones
// and 10-bit digits (LDS) take 4-wave blocks.
constexpr uint64_t kBigPass = 1ull << 24;
// Few keys: half the rounds, and so of a block's serial chain, and twice the
// blocks.  The depth order of 20000 records takes 51 us (68 with 16 rounds, 49
// with 4), 50000: 56 (68, 57), 100000: 66 (71, 71), 260000: 83 (80, 109; the
// column walks have grown past the gain).
constexpr int kFewRounds = 8;
constexpr uint64_t kFewPass = 1u << 17;
static_assert(walk_columns(kFewPass / RadixShape<4, kFewRounds>::kTile, 8), "columns walked");

template <typename Load, typename Store>
static void radix_pass_any(hipStream_t st, Load in, Store out, const uint64_t* n_dev,
                           uint64_t n_max, int shift, int width, uint32_t* hist,
                           uint32_t* scan_tmp) {
  if (width > 8)
    radix_pass<kMaxBins, 4, kSortRounds>(st, in, out, n_dev, n_max, shift, width, hist, scan_tmp);
  else if (n_max >= kBigPass)
    radix_pass<256, 8, kSortRounds>(st, in, out, n_dev, n_max, shift, width, hist, scan_tmp);
  else if (n_max <= kFewPass)
    radix_pass<256, 4, kFewRounds>(st, in, out, n_dev, n_max, shift, width, hist, scan_tmp);
  else
    radix_pass<256, 4, kSortRounds>(st, in, out, n_dev, n_max, shift, width, hist, scan_tmp);
}

// Up to here the order comes from counting pairs.  Its time grows with the
// square of the count, that of the passes hardly at all below 10^5.  Measured
// (us of kernel time, counting against the two-launch passes; each launch
// saved is worth 2 to 5 us more): records (with the offsets) 1000: 10 (2
// launches) / 37 (10), 8000: 23 / 48, 16000: 40 / 53, 32000: 86 / 60; tile
// keys of two passes, 8000: 10 / 17 (4 launches); size classes 4000: 10 / 13 (2
// launches), 8000: 17 / 11.
constexpr uint64_t kRankRecords = 16384;
constexpr uint64_t kRankKeys = 8192;
constexpr uint64_t kRankClasses = 4096;

// Stable sort of the records (keys, vals) by their 32 depth bits, 8-bit
// digits, then launch_offsets_scan over the sorted records.  Ends in
// (keys_a, vals_a).
void launch_depth_sort(hipStream_t st, uint32_t* keys_a, uint32_t* vals_a, uint32_t* keys_b,
                       uint32_t* vals_b, uint64_t m, uint32_t* hist, uint32_t* scan_tmp) {
  if (m == 0) return;
  for (int shift = 0; shift < 32; shift += 16) {
    radix_pass_any(st, StoredPairs<uint32_t>{keys_a, vals_a},
                   StorePairs<uint32_t>{keys_b, vals_b}, nullptr, m, shift, 8, hist, scan_tmp);
    radix_pass_any(st, StoredPairs<uint32_t>{keys_b, vals_b},
                   StorePairs<uint32_t>{keys_a, vals_a}, nullptr, m, shift + 8, 8, hist,
                   scan_tmp);
  }
}

bool rank_records(uint64_t m) { return m > 0 && m <= kRankRecords; }

void launch_rank_records(hipStream_t st, const uint32_t* keys, const uint32_t* vals, uint64_t m,
                         const uint2* trect, uint32_t* keys_out, uint32_t* vals_out,
                         uint32_t* cnt_sorted, uint2* trect_sorted) {
  hipLaunchKernelGGL(rank_records_kernel, dim3(blocks_for(m, kWave)), dim3(kRankWaves * kWave), 0,
                     st, keys, vals, (uint32_t)m, trect, keys_out, vals_out, cnt_sorted,
                     trect_sorted);
}

void launch_ranked_scan(hipStream_t st, const uint32_t* cnt_sorted, uint64_t m, uint64_t* offsets,
                        uint64_t* total, uint64_t* mailbox) {
  hipLaunchKernelGGL(scan_few_kernel, dim3(1), dim3(kScanFewThreads), 0, st, cnt_sorted,
                     (uint32_t)m, offsets, total, mailbox);
}

// The records in ascending order of size class; *first (unless NULL)
// receives the position of the first record of class `mark` or above, m if
// there is none.
void launch_class_order(hipStream_t st, uint64_t m, const uint32_t* ntiles, uint32_t* order,
                        uint32_t mark, uint32_t* first, uint32_t* hist, uint32_t* scan_tmp) {
  if (m == 0) {
    if (first) launch_fill_u32(st, first, 1, 0u);
    return;
  }
  const StoreOrder out{order, mark, first};
  if (m <= kRankClasses)
    hipLaunchKernelGGL(rank_classes_kernel, dim3(blocks_for(m + 1, kWave)),
                       dim3(kRankWaves * kWave), 0, st, ntiles, (uint32_t)m, out);
  else
    radix_pass_any(st, SizeClasses{ntiles}, out, nullptr, m, 0, kClassBits, hist, scan_tmp);
}

bool tile_keys_16bit(int bits) { return bits <= 16; }

void launch_keygen(hipStream_t st, uint64_t m, uint64_t n, const uint32_t* perm,
                   const uint32_t* cnt_sorted, const uint64_t* offsets, uint32_t* keyoff,
                   const uint2* trect_sorted, const FrameDesc* frames, uint64_t capacity,
                   int bits, void* keys, uint32_t* vals, uint32_t* overflow) {
  if (m == 0) return;
  if (tile_keys_16bit(bits))
    hipLaunchKernelGGL(keygen_kernel<uint16_t>, dim3(blocks_for(m, 256)), dim3(256), 0, st, m,
                       n, perm, cnt_sorted, offsets, keyoff, trect_sorted, frames, capacity,
                       static_cast<uint16_t*>(keys), vals, overflow);
  else
    hipLaunchKernelGGL(keygen_kernel<uint32_t>, dim3(blocks_for(m, 256)), dim3(256), 0, st, m,
                       n, perm, cnt_sorted, offsets, keyoff, trect_sorted, frames, capacity,
                       static_cast<uint32_t*>(keys), vals, overflow);
}

template <typename KeyT>
static bool tile_sort_t(hipStream_t st, KeyT* keys_a, uint32_t* vals_a, KeyT* keys_b,
                        uint32_t* vals_b, const uint64_t* k_dev, uint64_t k_max, int bits,
                        uint32_t* hist, uint32_t* scan_tmp) {
  if (k_max <= kRankKeys) {
    hipLaunchKernelGGL(rank_pairs_kernel<KeyT>, dim3(blocks_for(k_max, kWave)),
                       dim3(kRankWaves * kWave), 0, st, keys_a, vals_a, k_dev, (uint32_t)k_max,
                       keys_b, vals_b);
    return true;
  }
  int widths[8];
  const int passes = tile_pass_widths(bits, widths);
  bool in_b = false;
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    radix_pass_any(st, StoredPairs<KeyT>{in_b ? keys_b : keys_a, in_b ? vals_b : vals_a},
                   StorePairs<KeyT>{in_b ? keys_a : keys_b, in_b ? vals_a : vals_b}, k_dev, k_max,
                   shift, widths[p], hist, scan_tmp);
    in_b = !in_b;
    shift += widths[p];
  }
  return in_b;
}

// Stable sort of the tile keys by the tile-id bits [0, bits) in passes of
// near-equal width; 16-bit keys when bits <= 16.  Returns true if the result
// is in (keys_b, vals_b).
bool launch_tile_sort(hipStream_t st, void* keys_a, uint32_t* vals_a, void* keys_b,
                      uint32_t* vals_b, const uint64_t* k_dev, uint64_t k_max, int bits,
                      uint32_t* hist, uint32_t* scan_tmp) {
  if (k_max == 0) return false;
  if (tile_keys_16bit(bits))
    return tile_sort_t<uint16_t>(st, static_cast<uint16_t*>(keys_a), vals_a,
                                 static_cast<uint16_t*>(keys_b), vals_b, k_dev, k_max, bits,
                                 hist, scan_tmp);
  return tile_sort_t<uint32_t>(st, static_cast<uint32_t*>(keys_a), vals_a,
                               static_cast<uint32_t*>(keys_b), vals_b, k_dev, k_max, bits, hist,
                               scan_tmp);
}

// Beyond this many scan blocks the sums in front of them come from a kernel of
// their own: adding them up in every block grows with the square of the count.
// Without / with it (us, the scan, and with it the sums' kernel too): 1,280
// blocks 19 / 19 + 5, 4,096 (17M records) 66 / 54 + 8, 8,192 160 / 138 + 15,
// 32,768 (134M) 988 / 525 + 60.
constexpr unsigned kSpineBlocks = 4096;
static_assert(kSpineBlocks >= kGatherBig / kScanTile, "one sum per scan block");

// Exclusive scan of the depth-ordered records' tile counts into offsets
// (u64), total into *total; cnt_sorted[i] and trect_sorted[i] receive the
// count and the tile rect of record perm[i] (zero for a culled record).
void launch_offsets_scan(hipStream_t st, const uint32_t* skey, const uint32_t* perm,
                         const uint2* trect, uint64_t m, uint32_t* cnt_sorted,
                         uint2* trect_sorted, uint64_t* offsets, uint64_t* block_tmp,
                         uint64_t* total, uint64_t* mailbox) {
  if (m == 0) {
    launch_fill_u32(st, (uint32_t*)total, 2, 0u);
    return;
  }
  const bool big = m > kGatherBig;
  const unsigned items = big ? 16 : kScanFew;
  const dim3 grid(blocks_for(m, items * kScanThreads)), block(kScanThreads);
  if (big)
    hipLaunchKernelGGL(gather_counts_kernel<16>, grid, block, 0, st, m, skey, perm, trect,
                       cnt_sorted, trect_sorted, block_tmp);
  else
    hipLaunchKernelGGL(gather_counts_kernel<kScanFew>, grid, block, 0, st, m, skey, perm, trect,
                       cnt_sorted, trect_sorted, block_tmp);
  const unsigned nb = blocks_for(m, kScanTile);
  const bool spine = nb > kSpineBlocks;
  if (spine)
    hipLaunchKernelGGL(scan_spine_kernel, dim3(1), dim3(kSpineThreads), 0, st, block_tmp, nb);
  hipLaunchKernelGGL(scan_down_kernel, dim3(nb), block, 0, st, cnt_sorted, m, block_tmp,
                     spine ? 0u : kScanItems / items, offsets, total, mailbox);
}

void launch_ranges(hipStream_t st, const void* keys, int bits, const uint64_t* k_dev,
                   uint64_t k_max, uint64_t capacity, uint2* ranges, uint64_t n_tiles) {
  if (n_tiles == 0) return;
  const dim3 grid(blocks_for(n_tiles, 256 / kWave * (kWave - 1)));
  if (tile_keys_16bit(bits))
    hipLaunchKernelGGL(ranges_kernel<uint16_t>, grid, dim3(256), 0, st,
                       static_cast<const uint16_t*>(keys), k_dev, capacity, ranges,
                       (uint32_t)n_tiles);
  else
    hipLaunchKernelGGL(ranges_kernel<uint32_t>, grid, dim3(256), 0, st,
                       static_cast<const uint32_t*>(keys), k_dev, capacity, ranges,
                       (uint32_t)n_tiles);
}

}  // namespace gsr

