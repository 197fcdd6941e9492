// ssim.hip -- the mapper's rendering loss with its SSIM term, forward and
// backward (DROID-Splat eqn rnd_loss, Sec. 3.3; lambda2 = 0.2 in
// supplementary S1.2).  Per frame f of the batch,
//   L_f = l1 [ (1 - l2) mean|I - I*| + l2 (1 - SSIM(I, I*)) ]
//       + (1 - l1) mean_{Z* > 0} |Z - Z*|,
// SSIM being Wang et al.'s index with an 11 x 11 Gaussian window
// (sigma 1.5, weights summing to 1), C1 = 0.01^2, C2 = 0.03^2, window sums
// taken with zero padding, averaged over the 3 channels and all pixels.
//
// Launches:
//  - ssim_kernel computes the window sums w*x, w*y, w*(x^2 + y^2), w*xy, the
//    SSIM map with its derivatives A = dS/dmu_x, B = dS/d(w*x^2),
//    C = dS/d(w*xy), and, the window being symmetric, the adjoint
//    d(sum S)/dx = w*A + 2 x (w*B) + y (w*C), so that only the images are
//    read and only g_rgb is written; it also sums S, |x - y| and (channel 0)
//    the depth terms of its block;
//  - ssim_frame_kernel sums each frame's block records in a fixed order
//    into the frame's loss term and its depth gradient's scale;
//  - ssim_depth_kernel writes the depth gradients, whose scale is known only
//    then, and the total loss.
//
// ssim_kernel works down the columns of one colour plane in pairs of waves, a
// block each.  The first wave owns 128 adjacent columns of the map, two per
// lane: input rows are staged one at a time in LDS (x, y, x^2 + y^2 and xy),
// the horizontal 11-tap sums read 12 staged values for two columns, and the
// vertical sums accumulate in a ring of 11 output rows held in registers
// (slot = output row mod 11, static because the row loop is unrolled by 11).
// Each finished row of sums goes through LDS to the second wave, one row
// behind, which evaluates the map and does the same with the adjoint over the
// 118 columns whose windows lie inside the 128.  Neither the map nor its
// derivatives leave the CU.
//
// What bounds it: FP64 VALU issue, about 240 instructions per colour value of
// 128 columns and row, and on top the columns (128 / 118) and the rows
// ((segment + 22) / segment) that two pairs compute.  At 5.0 Mpixel in four
// frames it takes 274 us (the issue alone, at the measured 4.5 to 5.4 clocks
// per dependent pair of multiply-adds, about 200) and the depth pass 15; a
// kernel for the map, one column per lane, that left the derivatives in memory
// (24 bytes written and read per colour value) and one for the adjoint took
// 393.  Four pairs to a block, whose barrier then couples all of them, took
// 545 us, and a ring in the first wave beside the map (256 registers and
// spills whose reloads wait for the rows in flight) 690.
//
// The window sums and the map are evaluated in FP64: E[x^2] - mu^2 and the
// adjoint's sum of +-(2 x B + y C) terms cancel by up to three orders of
// magnitude where the image is flat (B, C ~ 1/C2), which FP32 would turn
// into errors of 1e-4 relative to the gradient.  Inputs and outputs are FP32.
#include <algorithm>
#include <cmath>

#include "launch.h"

namespace gsr {

namespace {

constexpr int kR = 5;                  // window radius (11 x 11)
constexpr int kTaps = 2 * kR + 1;
constexpr int kMapCols = 128;          // map columns per pair, two per lane
constexpr int kOutCols = kMapCols - 2 * kR;  // 118 output columns
constexpr int kInCols = kMapCols + 2 * kR;   // 138 staged columns
constexpr int kRow = kInCols + 2;      // (reads of unused lanes stay inside)
constexpr int kThreads = 2 * 64;       // one pair per block
// Segments: a pair runs 11 chunks iterations; the adjoint finishes output row
// i in iteration i + kLag.
constexpr int kLag = 4 * kR + 2;
constexpr int kMinChunks = 3, kMaxChunks = 16;
// rows whose global loads are in flight while a row is processed
constexpr int kAhead = 1;
// window sums: w*x, w*y, w*(x^2 + y^2), w*xy (the two second moments enter
// the map only through var_x + var_y)
constexpr int kMaps = 4;
constexpr double kC1 = 0.01 * 0.01;
constexpr double kC2 = 0.03 * 0.03;

struct Window {
  double g[kTaps];
};

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sums N values per thread over the block; thread 0 gets the totals.
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*red)[N]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) red[wv][k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
#pragma unroll
      for (int k = 0; k < N; ++k) v[k] += red[w][k];
}

__device__ __forceinline__ double sgn(double d) { return d > 0.0 ? 1.0 : (d < 0.0 ? -1.0 : 0.0); }

// Geometry of one pair's work: plane, output columns [x0, x0 + kOutCols),
// output rows [y0, y0 + seg), both clipped to the image.
struct Unit {
  int W, H, x0, y0;
  int64_t po;        // first value of the colour plane
  int64_t pix0;      // first pixel of the frame
  bool valid;
};

__device__ __forceinline__ Unit unit_of(const FrameDesc* frames, int seg) {
  const FrameDesc fr = frames[blockIdx.z];
  Unit w;
  w.W = fr.width;
  w.H = fr.height;
  const int ntx = (w.W + kOutCols - 1) / kOutCols, nty = (w.H + seg - 1) / seg;
  const int t = blockIdx.x;
  w.valid = t < ntx * nty;
  w.x0 = __builtin_amdgcn_readfirstlane(t / nty * kOutCols);
  w.y0 = __builtin_amdgcn_readfirstlane(t % nty * seg);
  w.po = 3 * fr.pixel_offset + (int64_t)blockIdx.y * w.W * w.H;
  w.pix0 = fr.pixel_offset;
  return w;
}

// Two adjacent columns of both images.  The rows are read through buffer
// descriptors of their own extent (none for a row outside the image), and a
// column outside has an offset past any row, so that the loads need no
// branches and what lies outside reads as zero (zero padding).
struct Px2 {
  float x[2], y[2];
};
constexpr uint32_t kOutside = 0xfffffffcu;
constexpr int kRawBuffer = 0x00027000;  // 32-bit data, no swizzle

__device__ __forceinline__ uint32_t col_offset(const Unit& w, int gx, bool use) {
  return use && gx >= 0 && gx < w.W ? 4u * (uint32_t)gx : kOutside;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_of(const Unit& w, const float* plane,
                                                         int gy) {
  const bool in = gy >= 0 && gy < w.H;
  const uint64_t at = (uint64_t)(plane + (in ? (int64_t)gy * w.W : 0));
  const uint64_t base =
      (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(at >> 32)) << 32 |
      (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)at);
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, in ? 4 * w.W : 0, kRawBuffer);
}

__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t row, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row, off, 0, 0));
}

__device__ __forceinline__ Px2 load2(__amdgpu_buffer_rsrc_t a, __amdgpu_buffer_rsrc_t b,
                                     const uint32_t (&off)[2]) {
  return Px2{{load1(a, off[0]), load1(a, off[1])}, {load1(b, off[0]), load1(b, off[1])}};
}

// Staged row: x, y, x^2 + y^2, xy.
struct alignas(16) Stage {
  double v[kMaps][kRow];
  uint4 off[64];  // the lanes' column offsets
};
struct alignas(16) SumRow {
  double v[kMaps][kMapCols];  // window sums
};
struct alignas(16) MapRow {
  double v[3][kRow];  // A, B, C
};

// Element i (0 or 1) of a pair of rows, by its byte offset: i alternates from
// one unrolled row to the next, and so does the parity of a chunk, so the
// address is formed per row instead of being held (and spilled) for both.
template <typename T>
__device__ __forceinline__ T& nth(T (&rows)[2], uint32_t i) {
  return *reinterpret_cast<T*>(reinterpret_cast<char*>(rows) + i * (uint32_t)sizeof(T));
}
// The other row's index, opaque to the compiler.
__device__ __forceinline__ uint32_t other(uint32_t i) {
  i ^= 1u;
  asm volatile("" : "+s"(i));
  return i;
}

__device__ __forceinline__ void stage2(Stage& s, int col, const Px2& v) {
  const double x0 = v.x[0], y0 = v.y[0], x1 = v.x[1], y1 = v.y[1];
  auto put = [&](int m, double a, double b) {
    *reinterpret_cast<double2*>(s.v[m] + col) = make_double2(a, b);
  };
  put(0, x0, x1);
  put(1, y0, y1);
  put(2, fma(y0, y0, x0 * x0), fma(y1, y1, x1 * x1));
  put(3, x0 * y0, x1 * y1);
}

// Adds the staged values v0, v1 of columns 2 i, 2 i + 1 (from the lane's
// first) to the window sums of the lane's two columns.
template <int I>
__device__ __forceinline__ void taps(const Window& win, double v0, double v1, double (&h)[2]) {
  if constexpr (I == 0) {
    h[0] = win.g[0] * v0;
    h[1] = win.g[0] * v1;
  } else {
    h[0] = fma(win.g[2 * I], v0, h[0]);
    h[1] = fma(win.g[2 * I - 1], v0, h[1]);
    h[1] = fma(win.g[2 * I], v1, h[1]);
  }
  if constexpr (2 * I + 1 < kTaps) h[0] = fma(win.g[2 * I + 1], v1, h[0]);
}
static_assert(kTaps == 11, "six column pairs cover two windows");

struct Taps12 {
  double2 v[6];
};
__device__ __forceinline__ Taps12 load_taps(const double* p) {
  Taps12 r;
#pragma unroll
  for (int i = 0; i < 6; ++i) r.v[i] = reinterpret_cast<const double2*>(p)[i];
  return r;
}

__device__ __forceinline__ void window2(const Window& win, const Taps12& t, double (&h)[2]) {
  taps<0>(win, t.v[0].x, t.v[0].y, h);
  taps<1>(win, t.v[1].x, t.v[1].y, h);
  taps<2>(win, t.v[2].x, t.v[2].y, h);
  taps<3>(win, t.v[3].x, t.v[3].y, h);
  taps<4>(win, t.v[4].x, t.v[4].y, h);
  taps<5>(win, t.v[5].x, t.v[5].y, h);
}

// Adds the row sums h of map m, row number u mod 11, to the ring; its first term
// (t = 0) assigns, so slots need no clearing.  The row that started ten rows
// ago is then complete, in slot (u + 1) mod 11.
template <int N>
__device__ __forceinline__ void ring_add(const Window& win, int u, int m, const double (&h)[2],
                                         double (&ring)[kTaps][N][2]) {
#pragma unroll
  for (int t = 0; t < kTaps; ++t) {
    const int s = (u - t + kTaps) % kTaps;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      ring[s][m][j] = t == 0 ? win.g[0] * h[j] : fma(win.g[t], h[j], ring[s][m][j]);
  }
}

// The map and its derivatives, in terms of the differences d = mu_x - mu_y and
// t = var(x - y), kept apart from the sums they would cancel in, so that
// equal images give S = 1 and A = 0, C = -2 B exactly:
//   S = (l_num / l_den) (c_num / c_den) = (1 - d^2 / l_den) (1 - t / c_den).
__device__ __forceinline__ double map_value(const double (&r)[kMaps][2], int j, double (&abc)[3]) {
  const double mx = r[0][j], my = r[1][j], mxy = mx * my, d = mx - my;
  const double l_num = fma(2.0, mxy, kC1), l_den = fma(d, d, l_num);
  const double t = fma(-d, d, fma(-2.0, r[3][j], r[2][j]));
  const double c_num = fma(2.0, r[3][j] - mxy, kC2), c_den = c_num + t;
  const double rinv = 1.0 / (l_den * c_den);
  const double inv_l = c_den * rinv, inv_c = l_den * rinv;
  const double u = l_num * rinv, k = t * inv_c;
  const double dS_dmu = 2.0 * d * (c_num * rinv) * inv_l * fma(my, d, -l_num);
  const double dS_dcov = 2.0 * u;
  abc[0] = fma(dS_dcov, fma(-mx, k, d), dS_dmu);
  abc[1] = fma(u, k, -u);  // dS/dvar
  abc[2] = dS_dcov;
  return fma(-d * inv_l, d, 1.0) * (1.0 - k);
}

// The first wave of a pair.  Iteration r adds staged row r, image row
// y0 - 10 + r, and finishes the window sums of map row y0 - 15 + r (r >= 10).
__device__ __forceinline__ void sums_wave(const Unit& w, int chunks, const Window& win,
                                          const float* __restrict__ rgb,
                                          const float* __restrict__ t_rgb, Stage (&st)[2],
                                          SumRow (&out)[2]) {
  const int lane = threadIdx.x & 63;
  const int col = 2 * lane;                 // map column and first staged column
  const int gx = w.x0 - 2 * kR + col;       // image column of the staged column
  const bool halo = lane < kR;
  const float *pa = rgb + w.po, *pb = t_rgb + w.po;
  // the lane's column offsets wait in LDS, beside the row that it reads: the
  // ring leaves no registers, and a spill's reload would wait for the rows in
  // flight
  st[0].off[lane] = st[1].off[lane] = make_uint4(
      col_offset(w, gx, true), col_offset(w, gx + 1, true), col_offset(w, gx + kMapCols, halo),
      col_offset(w, gx + kMapCols + 1, halo));
  Px2 main[kAhead], edge[kAhead];
  auto fetch = [&](const Stage& s, int gy, Px2& m, Px2& e) {
    const __amdgpu_buffer_rsrc_t a = row_of(w, pa, gy), b = row_of(w, pb, gy);
    const uint4 o = s.off[lane];
    m = load2(a, b, {o.x, o.y});
    e = load2(a, b, {o.z, o.w});
  };
  {
    const int gy = w.y0 - 2 * kR;
    Px2 m, e;
    fetch(st[0], gy, m, e);
    stage2(st[0], col, m);
    if (halo) stage2(st[0], kMapCols + col, e);
#pragma unroll
    for (int a = 0; a < kAhead; ++a) fetch(st[0], gy + 1 + a, main[a], edge[a]);
  }
  double ring[kTaps][kMaps][2];
  uint32_t cur = 0;  // r & 1
  __syncthreads();
  for (int k = 0; k < chunks; ++k) {
#pragma unroll
    for (int u = 0; u < kTaps; ++u) {
      const int r = k * kTaps + u;
      const Px2 px = main[0], px_h = edge[0];
#pragma unroll
      for (int a = 0; a + 1 < kAhead; ++a) main[a] = main[a + 1], edge[a] = edge[a + 1];
      const Stage& s = nth(st, cur);
      fetch(s, w.y0 - 2 * kR + r + 1 + kAhead, main[kAhead - 1], edge[kAhead - 1]);
      // map by map (the barriers keep the scheduler from collecting all the
      // loads in front, which does not fit the registers)
      Taps12 next = load_taps(s.v[0] + col);
#pragma unroll
      for (int m = 0; m < kMaps; ++m) {
        const Taps12 t = next;
        if (m + 1 < kMaps) next = load_taps(s.v[m + 1] + col);
        __builtin_amdgcn_sched_barrier(0);
        double h[2];
        window2(win, t, h);
        ring_add<kMaps>(win, u, m, h, ring);
      }
#pragma unroll
      for (int m = 0; m < kMaps; ++m)
        *reinterpret_cast<double2*>(nth(out, cur).v[m] + col) =
            make_double2(ring[(u + 1) % kTaps][m][0], ring[(u + 1) % kTaps][m][1]);
      cur = other(cur);
      stage2(nth(st, cur), col, px);
      if (halo) stage2(nth(st, cur), kMapCols + col, px_h);
      __syncthreads();
    }
  }
}

// The second wave.  Iteration r (>= 11) evaluates map row y0 - 16 + r from
// the sums of iteration r - 1, adds the map row before it to the adjoint and
// finishes output row y0 + r - 22.  acc: sum S over the output rows and
// columns, sum |x - y|, sum |z - z*|, valid depths.
__device__ __forceinline__ void adjoint_wave(const Unit& w, int chunks, const Window& win,
                                             double s_l1, double s_ss,
                                             const float* __restrict__ rgb,
                                             const float* __restrict__ t_rgb,
                                             const float* __restrict__ depth,
                                             const float* __restrict__ t_depth,
                                             const SumRow (&in)[2], MapRow (&rows)[2],
                                             float* __restrict__ g_rgb,
                                             double (&acc)[4]) {
  const int lane = threadIdx.x & 63;
  const int seg = kTaps * chunks - kLag;
  const int col = 2 * lane;  // output column and map column (kR further left)
  bool in_map[2], own[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int x = w.x0 - kR + col + j;
    in_map[j] = x >= 0 && x < w.W;
    own[j] = in_map[j] && col + j >= kR && col + j < kR + kOutCols;
  }
  const int gx = w.x0 + col;
  const bool used = col < kOutCols;
  const uint32_t off[2] = {col_offset(w, gx, used), col_offset(w, gx + 1, used)};
  const float *pa = rgb + w.po, *pb = t_rgb + w.po;
  const bool with_depth = blockIdx.y == 0;
  // the output rows' pixels: colours, and depth and target depth
  Px2 px[kAhead], dz[kAhead];
  auto fetch = [&](int gy, Px2& c, Px2& z) {
    c = load2(row_of(w, pa, gy), row_of(w, pb, gy), off);
    const int gz = with_depth ? gy : -1;
    z = load2(row_of(w, depth + w.pix0, gz), row_of(w, t_depth + w.pix0, gz), off);
  };
#pragma unroll
  for (int a = 0; a < kAhead; ++a) px[a] = dz[a] = Px2{{0.0f, 0.0f}, {0.0f, 0.0f}};
  double ring[kTaps][3][2];
  __syncthreads();
  for (int k = 0; k < chunks; ++k) {
#pragma unroll
    for (int u = 0; u < kTaps; ++u) {
      const int r = k * kTaps + u;
      if (k > 0) {
        const int gy = w.y0 + r - kLag;
        const Px2 v = px[0], z = dz[0];
#pragma unroll
        for (int a = 0; a + 1 < kAhead; ++a) px[a] = px[a + 1], dz[a] = dz[a + 1];
        // (rows above the segment are not used)
        fetch(gy + kAhead, px[kAhead - 1], dz[kAhead - 1]);
        // (the first row of all holds no map row yet: its ring slots are
        // assigned again before an output row reads them)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          double h[2];
          window2(win, load_taps(rows[(r & 1) ^ 1].v[m] + col), h);
          ring_add<3>(win, u, m, h, ring);
        }
        {
          const int my = w.y0 - 3 * kR - 1 + r;  // map row
          const bool row_in = my >= 0 && my < w.H;
          const bool row_own = my >= w.y0 && my < w.y0 + seg;
          double sum[kMaps][2], abc[2][3];
#pragma unroll
          for (int m = 0; m < kMaps; ++m) {
            const double2 v = *reinterpret_cast<const double2*>(in[(r & 1) ^ 1].v[m] + col);
            sum[m][0] = v.x;
            sum[m][1] = v.y;
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const double S = map_value(sum, j, abc[j]);
            const bool use = row_in && in_map[j];
#pragma unroll
            for (int m = 0; m < 3; ++m) abc[j][m] = use ? abc[j][m] : 0.0;
            acc[0] += row_in && row_own && own[j] ? S : 0.0;
          }
#pragma unroll
          for (int m = 0; m < 3; ++m)
            *reinterpret_cast<double2*>(rows[r & 1].v[m] + col) =
                make_double2(abc[0][m], abc[1][m]);
        }
        if (r >= kLag && gy < w.H) {
          const __amdgpu_buffer_rsrc_t row = row_of(w, g_rgb + w.po, gy);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const double(&d)[3][2] = ring[(u + 1) % kTaps];
            const double x = v.x[j], y = v.y[j];
            const double dssim = d[0][j] + fma(x, fma(2.0, d[1][j], d[2][j]), (y - x) * d[2][j]);
            const float g = (float)(s_l1 * sgn(x - y) - s_ss * dssim);
            // (a column outside is not written, and its x, y, z and z* are 0)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(g), row, off[j], 0, 0);
            acc[1] += fabs(x - y);
            const bool valid = z.y[j] > 0.0f;
            acc[2] += valid ? fabs((double)z.x[j] - (double)z.y[j]) : 0.0;
            acc[3] += valid ? 1.0 : 0.0;
          }
        }
      }
      __syncthreads();
    }
  }
}

__global__ void __launch_bounds__(kThreads, 2) ssim_kernel(
    const FrameDesc* __restrict__ frames, int units, int chunks, Window win, double lambda1,
    double lambda2, const float* __restrict__ rgb, const float* __restrict__ t_rgb,
    const float* __restrict__ depth, const float* __restrict__ t_depth,
    float* __restrict__ g_rgb, double* __restrict__ tile_sums /* [F][3][units][4] */) {
  __shared__ Stage stage[2];
  __shared__ SumRow sums[2];
  __shared__ MapRow rows[2];
  __shared__ double red[2][4];
  const Unit w = unit_of(frames, kTaps * chunks - kLag);
  double* out = tile_sums +
                (((int64_t)blockIdx.z * 3 + blockIdx.y) * units + blockIdx.x) * 4;
  if (!w.valid) {
    if (threadIdx.x < 4) out[threadIdx.x] = 0.0;
    return;
  }
  double acc[4] = {0.0, 0.0, 0.0, 0.0};  // sum S, sum |x - y|, sum |z - z*|, valid depths
  if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) {
    sums_wave(w, chunks, win, rgb, t_rgb, stage, sums);
  } else {
    const double n3 = 3.0 * (double)w.W * (double)w.H;
    adjoint_wave(w, chunks, win, lambda1 * (1.0 - lambda2) / n3, lambda1 * lambda2 / n3, rgb,
                 t_rgb, depth, t_depth, sums, rows, g_rgb, acc);
  }
  block_sums<4>(acc, red);
  if (threadIdx.x == 0)
    for (int k = 0; k < 4; ++k) out[k] = acc[k];
}

// One block per frame: its block records in a fixed order -> the frame's
// loss term, SSIM and depth gradient scale: fs[f] = ((1-l1) / |m|, L_f).
__global__ void __launch_bounds__(256) ssim_frame_kernel(
    const FrameDesc* __restrict__ frames, int units, const double* __restrict__ tile_sums,
    double lambda1, double lambda2, float* __restrict__ ssim, double* __restrict__ fs) {
  __shared__ double red[4][4];
  const int f = blockIdx.x;
  const int per_frame = 3 * units;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < per_frame; b += blockDim.x)
    for (int k = 0; k < 4; ++k) s[k] += tile_sums[((int64_t)f * per_frame + b) * 4 + k];
  block_sums<4>(s, red);
  if (threadIdx.x == 0) {
    const double n3 = 3.0 * (double)frames[f].width * (double)frames[f].height;
    const double ss = s[0] / n3;
    if (ssim) ssim[f] = (float)ss;
    fs[2 * f] = s[3] > 0.0 ? (1.0 - lambda1) / s[3] : 0.0;
    fs[2 * f + 1] = lambda1 * ((1.0 - lambda2) * s[1] / n3 + lambda2 * (1.0 - ss)) +
                    (s[3] > 0.0 ? (1.0 - lambda1) * s[2] / s[3] : 0.0);
  }
}

// The depth gradients of frame blockIdx.y, and (first thread of all) the sum
// of the frame terms in frame order.
__global__ void __launch_bounds__(256) ssim_depth_kernel(
    const FrameDesc* __restrict__ frames, int n_frames, const double* __restrict__ fs,
    const float* __restrict__ depth, const float* __restrict__ t_depth,
    float* __restrict__ g_depth, float* __restrict__ g_alpha, float* __restrict__ loss) {
  const int f = blockIdx.y;
  const FrameDesc fr = frames[f];
  const int64_t n = (int64_t)fr.width * fr.height;
  const double s_d = fs[2 * f];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t q = fr.pixel_offset + i;
    const float z = depth[q], tz = t_depth[q];
    g_depth[q] = tz > 0.0f ? (float)(s_d * sgn((double)z - (double)tz)) : 0.0f;
    g_alpha[q] = 0.0f;
  }
  if (blockIdx.x == 0 && f == 0 && threadIdx.x == 0) {
    double total = 0.0;
    for (int k = 0; k < n_frames; ++k) total += fs[2 * k + 1];
    *loss = (float)total;
  }
}

Window make_window() {
  Window w;
  double s = 0.0;
  for (int d = 0; d < kTaps; ++d) {
    const double k = d - kR;
    w.g[d] = std::exp(-(k * k) / (2.0 * 1.5 * 1.5));
    s += w.g[d];
  }
  for (int d = 0; d < kTaps; ++d) w.g[d] /= s;
  return w;
}

}  // namespace

// The chunks are the ones with the least work on the busiest SIMD: a launch
// runs as rounds of one pair per SIMD (two waves of 256 registers), of 11
// chunks rows each.  More rows per pair waste fewer on the 22 rows around a
// segment, fewer fill the last round better.
SsimPlan ssim_plan(const FrameDesc* frames, int F) {
  constexpr int64_t kSimds = 1024;
  constexpr int kMinSeg = kTaps * kMinChunks - kLag;
  SsimPlan best{0, 0, 0, 0};
  int64_t cost = 0;
  int max_w = 1, max_h = 1;
  for (int f = 0; f < F; ++f) {
    max_w = std::max(max_w, (int)frames[f].width);
    max_h = std::max(max_h, (int)frames[f].height);
  }
  const int64_t units_max =
      (int64_t)((max_w / (double)kOutCols + 1.0) * (max_h / (double)kMinSeg + 1.0));
  for (int c = kMinChunks; c <= kMaxChunks; ++c) {
    const int seg = kTaps * c - kLag;
    int64_t pairs = 0, most = 0, px = 0;
    for (int f = 0; f < F; ++f) {
      const int64_t units = (int64_t)((frames[f].width + kOutCols - 1) / kOutCols) *
                            ((frames[f].height + seg - 1) / seg);
      pairs += 3 * units;
      most = std::max(most, units);
      px = std::max(px, (int64_t)frames[f].width * frames[f].height);
    }
    const int64_t rounds = (pairs + kSimds - 1) / kSimds;
    if (best.chunks == 0 || rounds * c <= cost) {
      cost = rounds * c;
      best = SsimPlan{c, (int)most, px, units_max};
    }
  }
  return best;
}

void launch_loss_render(hipStream_t st, int F, const SsimPlan& plan, const FrameDesc* frames,
                        const float* rgb, const float* depth, const float* t_rgb,
                        const float* t_depth, float lambda1, float lambda2, double* tile_sums,
                        double* frame_sums, float* loss, float* ssim, float* g_rgb,
                        float* g_depth, float* g_alpha) {
  static const Window win = make_window();
  hipLaunchKernelGGL(ssim_kernel, dim3((unsigned)plan.units, 3u, (unsigned)F), dim3(kThreads),
                     0, st, frames, plan.units, plan.chunks, win, (double)lambda1,
                     (double)lambda2, rgb, t_rgb, depth, t_depth, g_rgb, tile_sums);
  hipLaunchKernelGGL(ssim_frame_kernel, dim3((unsigned)F), dim3(256), 0, st, frames,
                     plan.units, tile_sums, (double)lambda1, (double)lambda2, ssim,
                     frame_sums);
  const unsigned bx = (unsigned)std::min<int64_t>((plan.max_px + 1023) / 1024, 4096);
  hipLaunchKernelGGL(ssim_depth_kernel, dim3(std::max(bx, 1u), (unsigned)F), dim3(256), 0, st,
                     frames, F, frame_sums, depth, t_depth, g_depth, g_alpha, loss);
}

}  // namespace gsr
