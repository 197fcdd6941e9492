// surfel.hip -- the 2D Gaussian surfel (2DGS) variant of the rasterizer
// (DROID-Splat Sec. 3.3 compares 2D surfels with its 3D Gaussians in
// tab:renderer; the 2DGS method it cites).  The key, sort and range stages
// (A2-A5) and the batching are those of the 3D path; the preprocess and the
// compositing differ.
//
// A surfel is a flat disk: mean mu, two scales (s_u, s_v), rotation q whose
// first two axes t_u, t_v span it and whose third t_w is its normal, opacity
// and SH colour.  With the frame's world->camera [R_f | t_f] and intrinsics K,
//   M = K [s_u R_f t_u | s_v R_f t_v | R_f mu + t_f]     (rows M0, M1, M2)
// maps disk coordinates (u, v, 1) to homogeneous pixels, and the ray through
// pixel (x, y) meets the disk at (u, v) = (p0/p2, p1/p2), p = h_u x h_v,
// h_u = x M2 - M0, h_v = y M2 - M1, at depth M2 . (u, v, 1).  The record
// holds M2 and k_u = c_x M2 - M0, k_v = c_y M2 - M1 (c the projected centre,
// whose third components vanish), so that a pixel forms
//   h_u = (x - c_x) M2 + k_u,   h_v = (y - c_y) M2 + k_v
// from its small offset to the centre, which FP32 keeps exact to rounding;
// the centre is stored as FP32 hi/lo pairs.  Per pixel:
//   G = exp(-(u^2 + v^2)/2), G_lp = exp(-|(x, y) - c|^2), G' = max(G, G_lp),
//   alpha = min(0.99, sigma G'), depth = M2 . (u, v, 1) (c's depth where
//   G_lp wins), normal = t_w in the camera frame, turned to face the camera;
// compositing thresholds and order as in the 3D path.  The depth distortion
// of a pixel is the sum over pairs i < j of blended entries of
// w_i w_j (z_i - z_j)^2; the forward adds w_j (A z_j^2 - 2 z_j D_1 + D_2) per
// entry, A, D_1, D_2 the sums of w, w z, w z^2 in front of it, with every z
// taken relative to the pixel's first blended entry so that the FP32 sums
// stay near the spread of the depths rather than their size.  A surfel covers
// the bounding box of the image of the disk |(u, v)| <= sqrt(2 ln(255 sigma))
// (exact, from the disk's dual conic) united with the square of half width
// sqrt(ln(255 sigma)) around c, and is culled unless the disk lies beyond the
// near plane; the box's integer bounds are taken in FP64.
#include <algorithm>
#include <cstddef>

#include "launch.h"
#include "sh_device.h"
#include "wave_util.h"

namespace gsr {

namespace {

struct alignas(16) Surfel {  // 96 bytes: six 16-byte loads
  float m2x, m2y, zc, kux;  // M2 = (m2x, m2y, zc); k_u = (kux, kuy, 0)
  float kuy, kvx, kvy, cxh;  // k_v = (kvx, kvy, 0); centre x hi
  float cxl, cyh, cyl, opacity;
  float c0, c1, c2, n0;      // colour, normal
  float n1, n2;
  uint32_t sqx, sqy;         // pixel box, lo | hi << 16
  // where alpha can reach 1/255: |(e1 dx + e2 dy, e3 dy)| <= 1 (the disk's
  // image, widened to be centred on c; zeros: the whole box) or within the
  // low-pass radius, squared
  float e1, e2, e3, low;
};
static_assert(sizeof(Surfel) == 96, "surfel record layout");

template <int DEG>
__global__ void __launch_bounds__(256) surfel_preprocess_kernel(
    int64_t n, int n_frames, const FrameDesc* __restrict__ frames,
    const float* __restrict__ poses, const float* __restrict__ means,
    const float* __restrict__ log_scales /* [n,2] */, const float* __restrict__ quats,
    const float* __restrict__ opac, const float* __restrict__ sh, int tile_w, int tile_h,
    Surfel* __restrict__ rec, uint2* __restrict__ trect, uint32_t* __restrict__ depth_key,
    uint32_t* __restrict__ rec_id, uint32_t* __restrict__ ntiles) {
#pragma clang fp contract(off)
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const double su = exp((double)log_scales[2 * g]), sv = exp((double)log_scales[2 * g + 1]);
  double q[4];
  for (int a = 0; a < 4; ++a) q[a] = quats[4 * g + a];
  const double qn = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
  const double w = q[0] / qn, x = q[1] / qn, y = q[2] / qn, z = q[3] / qn;
  const double Rg[9] = {1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y - w * z), 2.0 * (x * z + w * y),
                        2.0 * (x * y + w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z - w * x),
                        2.0 * (x * z - w * y), 2.0 * (y * z + w * x), 1.0 - 2.0 * (x * x + y * y)};
  const double o = 1.0 / (1.0 + exp(-(double)opac[g]));
  const double mu[3] = {means[3 * g], means[3 * g + 1], means[3 * g + 2]};
  constexpr int nb = (DEG + 1) * (DEG + 1);
  const double amin = (double)kAlphaMin;
  // a surfel with a non-finite parameter is culled in every frame: the 9
  // geometric values here, the SH coefficients through the FP64 colour sum of
  // a kept record (finite exactly when every coefficient is, as for the 3D
  // Gaussians)
  bool finite = isfinite(opac[g]) && isfinite(log_scales[2 * g]) && isfinite(log_scales[2 * g + 1]);
  for (int a = 0; a < 3; ++a) finite = finite && isfinite(means[3 * g + a]);
  for (int a = 0; a < 4; ++a) finite = finite && isfinite(quats[4 * g + a]);
  for (int f = (int)blockIdx.y; f < n_frames; f += (int)gridDim.y) {
    const int64_t r = (int64_t)f * n + g;
    const FrameDesc fr = frames[f];
    double W[9], tf[3];
    load_pose(poses, f, W, tf);
    rec_id[r] = (uint32_t)r;
    depth_key[r] = 0xffffffffu;
    ntiles[r] = 0;
    double mc[3], T[9];  // T = R_f R_g: columns t_u, t_v, t_w in the camera frame
    for (int i = 0; i < 3; ++i) {
      mc[i] = W[i * 3 + 0] * mu[0] + W[i * 3 + 1] * mu[1] + W[i * 3 + 2] * mu[2] + tf[i];
      for (int j = 0; j < 3; ++j)
        T[i * 3 + j] = W[i * 3 + 0] * Rg[0 * 3 + j] + W[i * 3 + 1] * Rg[1 * 3 + j] +
                       W[i * 3 + 2] * Rg[2 * 3 + j];
    }
    const double near = fr.near_z;
    if (!finite || !(o > amin) || !(mc[2] > near)) continue;
    const double fx = fr.fx, fy = fr.fy, cx = fr.cx, cy = fr.cy;
    // columns a = s_u t_u, b = s_v t_v, c = mc; rows of M = K [a | b | c]
    const double A[3] = {su * T[0], su * T[3], su * T[6]};
    const double B[3] = {sv * T[1], sv * T[4], sv * T[7]};
    const double M0[3] = {fx * A[0] + cx * A[2], fx * B[0] + cx * B[2], fx * mc[0] + cx * mc[2]};
    const double M1[3] = {fy * A[1] + cy * A[2], fy * B[1] + cy * B[2], fy * mc[1] + cy * mc[2]};
    const double M2[3] = {A[2], B[2], mc[2]};
    const double ccx = M0[2] / M2[2], ccy = M1[2] / M2[2];
    const double r2 = 2.0 * log(o / amin);  // r_a^2
    const double ra = sqrt(r2), rl = sqrt(log(o / amin));
    // the disk's nearest point to the camera plane must be beyond the near plane
    if (!(M2[2] - ra * sqrt(M2[0] * M2[0] + M2[1] * M2[1]) > near)) continue;
    // bounding box of the image of the circle |(u, v)| = r_a: the dual conic
    // C* = M diag(r_a^2, r_a^2, -1) M^T has the vertical tangents x = x0 with
    // C*_00 - 2 x0 C*_02 + x0^2 C*_22 = 0 (and likewise in y)
    const double c22 = r2 * (M2[0] * M2[0] + M2[1] * M2[1]) - M2[2] * M2[2];
    const double c02 = r2 * (M0[0] * M2[0] + M0[1] * M2[1]) - M0[2] * M2[2];
    const double c00 = r2 * (M0[0] * M0[0] + M0[1] * M0[1]) - M0[2] * M0[2];
    const double c12 = r2 * (M1[0] * M2[0] + M1[1] * M2[1]) - M1[2] * M2[2];
    const double c11 = r2 * (M1[0] * M1[0] + M1[1] * M1[1]) - M1[2] * M1[2];
    const double dx = c02 * c02 - c00 * c22, dy = c12 * c12 - c11 * c22;
    const double sx = sqrt(dx > 0.0 ? dx : 0.0), sy = sqrt(dy > 0.0 ? dy : 0.0);
    const double xa = (c02 + sx) / c22, xb = (c02 - sx) / c22;
    const double ya = (c12 + sy) / c22, yb = (c12 - sy) / c22;
    double lox = xa < xb ? xa : xb, hix = xa < xb ? xb : xa;
    double loy = ya < yb ? ya : yb, hiy = ya < yb ? yb : ya;
    lox = ccx - rl < lox ? ccx - rl : lox;
    hix = ccx + rl > hix ? ccx + rl : hix;
    loy = ccy - rl < loy ? ccy - rl : loy;
    hiy = ccy + rl > hiy ? ccy + rl : hiy;
    const double xl = ceil(lox), xh = floor(hix), yl = ceil(loy), yh = floor(hiy);
    const int x_lo = xl > 0.0 ? (int)xl : 0;
    const int y_lo = yl > 0.0 ? (int)yl : 0;
    const int x_hi = xh < (double)(fr.width - 1) ? (int)xh : fr.width - 1;
    const int y_hi = yh < (double)(fr.height - 1) ? (int)yh : fr.height - 1;
    if (!(x_lo <= x_hi && y_lo <= y_hi)) continue;
    double dir[3];
    view_dir(W, tf, mu, dir);
    double Y[16];
    sh_basis<DEG>(dir[0], dir[1], dir[2], Y);
    double raw[3] = {0.0, 0.0, 0.0};
    const float* shg = sh + g * nb * 3;
    for (int k = 0; k < nb; ++k)
      for (int c = 0; c < 3; ++c) raw[c] += (double)shg[k * 3 + c] * Y[k];
    if (!isfinite(raw[0] + raw[1] + raw[2])) continue;
    const int tx0 = x_lo / tile_w, tx1 = x_hi / tile_w;
    const int ty0 = y_lo / tile_h, ty1 = y_hi / tile_h;
    ntiles[r] = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
    trect[r] = make_uint2((uint32_t)tx0 | ((uint32_t)tx1 << 16),
                          (uint32_t)ty0 | ((uint32_t)ty1 << 16));
    const float zf = (float)mc[2];
    depth_key[r] = __float_as_uint(zf);
    // normal turned to face the camera
    const double tw[3] = {T[2], T[5], T[8]};
    const double sgn = (tw[0] * mc[0] + tw[1] * mc[1] + tw[2] * mc[2]) < 0.0 ? 1.0 : -1.0;
    Surfel s;
    s.m2x = (float)M2[0];
    s.m2y = (float)M2[1];
    s.zc = zf;
    s.kux = (float)(ccx * M2[0] - M0[0]);
    s.kuy = (float)(ccx * M2[1] - M0[1]);
    s.kvx = (float)(ccy * M2[0] - M1[0]);
    s.kvy = (float)(ccy * M2[1] - M1[1]);
    s.cxh = (float)ccx;
    s.cxl = (float)(ccx - (double)s.cxh);
    s.cyh = (float)ccy;
    s.cyl = (float)(ccy - (double)s.cyh);
    s.opacity = (float)o;
    const double c0 = raw[0] + 0.5, c1 = raw[1] + 0.5, c2 = raw[2] + 0.5;
    s.c0 = (float)(c0 > 0.0 ? c0 : 0.0);
    s.c1 = (float)(c1 > 0.0 ? c1 : 0.0);
    s.c2 = (float)(c2 > 0.0 ? c2 : 0.0);
    s.n0 = (float)(sgn * tw[0]);
    s.n1 = (float)(sgn * tw[1]);
    s.n2 = (float)(sgn * tw[2]);
    s.sqx = (uint32_t)x_lo | ((uint32_t)x_hi << 16);
    s.sqy = (uint32_t)y_lo | ((uint32_t)y_hi << 16);
    s.e1 = s.e2 = s.e3 = 0.0f;
    s.low = (float)(0.5 * r2) * 1.0001f + 1e-3f;
    {
      // The disk's image {x : (x - x_e)^T S^-1 (x - x_e) <= 1} from the dual
      // conic, taken around c instead: |L^T (x - c)| <= 1 + |L^T (x_e - c)|
      // holds inside it (S^-1 = L L^T).  Only where the per-pixel FP32
      // intersection resolves the boundary to well under the 2 % the block
      // test adds: the boundary maps to disk coordinates with a stretch of at
      // most ((1 + h)/(1 - h))^2 for h = r_a |(M2_0, M2_1)| / M2_2 <= 1/2, and
      // an error of ~16 ulps of the largest products over p2 (which is linear
      // in the pixel) and r_a stays below 1e-4.
      const double c01 = r2 * (M0[0] * M1[0] + M0[1] * M1[1]) - M0[2] * M1[2];
      const double i22 = 1.0 / c22;
      const double sxx = dx * i22 * i22, syy = dy * i22 * i22;
      const double sxy = (c02 * c12 - c01 * c22) * i22 * i22;
      const double det = sxx * syy - sxy * sxy;
      const double kux = ccx * M2[0] - M0[0], kuy = ccx * M2[1] - M0[1];
      const double kvx = ccy * M2[0] - M1[0], kvy = ccy * M2[1] - M1[1];
      const double X = fmax(ccx - lox, hix - ccx) + 1.0, Y = fmax(ccy - loy, hiy - ccy) + 1.0;
      const double hux = X * fabs(M2[0]) + fabs(kux), huy = X * fabs(M2[1]) + fabs(kuy);
      const double hvx = Y * fabs(M2[0]) + fabs(kvx), hvy = Y * fabs(M2[1]) + fabs(kvy);
      const double p2 = fabs(kux * kvy - kuy * kvx) - X * fabs(M2[0] * kvy - M2[1] * kvx) -
                        Y * fabs(kux * M2[1] - kuy * M2[0]);
      const double big = hux * hvy + huy * hvx +
                         M2[2] * (huy * Y + X * hvy + hux * Y + X * hvx) / ra;
      if (det > 1e-6 * sxx * syy && p2 > 0.0 && big < 100.0 * p2 &&
          ra * sqrt(M2[0] * M2[0] + M2[1] * M2[1]) < 0.5 * M2[2]) {
        const double a1 = sqrt(syy / det), a2 = -sxy / sqrt(syy * det), a3 = 1.0 / sqrt(syy);
        const double ox = c02 * i22 - ccx, oy = c12 * i22 - ccy;
        const double m = a1 * ox + a2 * oy, b = a3 * oy;
        const double w = 1.0 / (1.0 + sqrt(m * m + b * b));
        s.e1 = (float)(a1 * w);
        s.e2 = (float)(a2 * w);
        s.e3 = (float)(a3 * w);
      }
    }
    rec[r] = s;
  }
}

// One pixel's view of one surfel: G', alpha before the clamp, depth.
struct SurfelHit {
  float Gh, z;
  bool obj;       // the disk term (not the low-pass) is the larger
  float u, v, hux, huy, huz, hvx, hvy, hvz, ex, ey;  // kept for the backward
};

// ln 255 rounded up: beyond this squared distance from the centre the
// low-pass term is below 1/255, so alpha = sigma G_lp < 1/255 there and it
// can never be blended; skipping its exp leaves every decision unchanged
// (where G >= G_lp the disk term is taken either way, and where G < G_lp
// alpha < 1/255 either way).
constexpr float kLowpassReach = 5.6f;

// The fields of an entry that a pixel's row reads, and the part of the
// intersection fixed by the lane's pixel column (h_u = (x - c_x) M2 + k_u
// does not depend on the row).
struct SurfelEntry {
  float cyh, cyl, m2x, m2y, kvx, kvy, zc, opacity;  // the record's row fields
  float ex, hux, huy, huz;                          // the column's part
};

__device__ __forceinline__ SurfelEntry surfel_entry(const Surfel& S, int px) {
#pragma clang fp contract(off)
  SurfelEntry e;
  e.cyh = S.cyh; e.cyl = S.cyl; e.m2x = S.m2x; e.m2y = S.m2y;
  e.kvx = S.kvx; e.kvy = S.kvy; e.zc = S.zc; e.opacity = S.opacity;
  asm volatile("" : "+v"(e.cyh), "+v"(e.cyl), "+v"(e.m2x), "+v"(e.m2y), "+v"(e.kvx),
               "+v"(e.kvy), "+v"(e.zc), "+v"(e.opacity));
  e.ex = -dx_of(S.cxh, S.cxl, px);  // x - c_x
  e.hux = e.ex * e.m2x + S.kux;
  e.huy = e.ex * e.m2y + S.kuy;
  e.huz = e.ex * e.zc;
  return e;
}

__device__ __forceinline__ SurfelHit surfel_eval(const SurfelEntry& e, int py) {
#pragma clang fp contract(off)
  SurfelHit h;
  h.ex = e.ex;
  h.ey = -dx_of(e.cyh, e.cyl, py);
  h.hux = e.hux;
  h.huy = e.huy;
  h.huz = e.huz;
  h.hvx = h.ey * e.m2x + e.kvx;
  h.hvy = h.ey * e.m2y + e.kvy;
  h.hvz = h.ey * e.zc;
  const float p0 = h.huy * h.hvz - h.huz * h.hvy;
  const float p1 = h.huz * h.hvx - h.hux * h.hvz;
  const float p2 = h.hux * h.hvy - h.huy * h.hvx;
  // reciprocal with one Newton step (within an ulp or so of 1/p2); a ray in the
  // disk's plane (p2 = 0) leaves the low-pass alone: with G = 0, alpha is set by
  // the low-pass or is 0, and u, v are not used
  const float r0 = __builtin_amdgcn_rcpf(p2);
  const float ip2 = __builtin_fmaf(__builtin_fmaf(-p2, r0, 1.0f), r0, r0);
  h.u = p0 * ip2;
  h.v = p1 * ip2;
  const float G = p2 != 0.0f ? gauss_of(h.u * h.u + h.v * h.v) : 0.0f;
  const float d2 = h.ex * h.ex + h.ey * h.ey;
  const float Glp = d2 < kLowpassReach ? gauss_of(2.0f * d2) : 0.0f;
  h.obj = G >= Glp;
  h.Gh = h.obj ? G : Glp;
  h.z = h.obj ? (e.m2x * h.u + e.m2y * h.v + e.zc) : e.zc;
  return h;
}

// The pixels of the 8 x 8 block at (bx, by) inside the surfel's box, one bit per
// lane; 0 where the block's part of the box cannot reach alpha >= 1/255.  ALL:
// the box alone.
template <bool ALL>
__device__ __forceinline__ uint64_t block_pixels(const Surfel& S, int bx, int by) {
  const BlockPart b = block_part(S.sqx, S.sqy, bx, by);
  if (b.empty()) return 0;
  if (!ALL) {
    float big;
    const float q = least_q(S.e1, S.e2, S.e3, S.cxh, S.cxl, S.cyh, S.cyl, b, big);
    const float r = 1.02f + 4e-6f * big;
    const float nx = __builtin_amdgcn_fmed3f(0.0f, dx_of(S.cxh, S.cxl, b.xhi),
                                             dx_of(S.cxh, S.cxl, b.xlo));
    const float ny = __builtin_amdgcn_fmed3f(0.0f, dx_of(S.cyh, S.cyl, b.yhi),
                                             dx_of(S.cyh, S.cyl, b.ylo));
    if (q > r * r && nx * nx + ny * ny > S.low) return 0;
  }
  return block_lanes(b, bx, by);
}

// A surfel staged in LDS for the forward: the record's fields up to the normal,
// then the block's pixels inside the box and one past the list position.
// (Assigned field by field: a copy of the whole record would go through scratch
// memory.)
struct alignas(16) FwdSurfel {
  float4 v0, v1, v2, v3;  // as Surfel
  float n1, n2;
  uint32_t px_lo, px_hi, pos;
  __device__ __forceinline__ void set(const Surfel& S, uint64_t in, uint32_t at) {
    v0 = make_float4(S.m2x, S.m2y, S.zc, S.kux);
    v1 = make_float4(S.kuy, S.kvx, S.kvy, S.cxh);
    v2 = make_float4(S.cxl, S.cyh, S.cyl, S.opacity);
    v3 = make_float4(S.c0, S.c1, S.c2, S.n0);
    n1 = S.n1;
    n2 = S.n2;
    px_lo = (uint32_t)in;
    px_hi = (uint32_t)(in >> 32);
    pos = at;
  }
  __device__ __forceinline__ uint64_t lanes() const {
    return ((uint64_t)__builtin_amdgcn_readfirstlane(px_hi) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane(px_lo);
  }
  __device__ __forceinline__ Surfel record() const {
    Surfel S;
    S.m2x = v0.x; S.m2y = v0.y; S.zc = v0.z; S.kux = v0.w;
    S.kuy = v1.x; S.kvx = v1.y; S.kvy = v1.z; S.cxh = v1.w;
    S.cxl = v2.x; S.cyh = v2.y; S.cyl = v2.z; S.opacity = v2.w;
    S.c0 = v3.x; S.c1 = v3.y; S.c2 = v3.z; S.n0 = v3.w;
    S.n1 = n1; S.n2 = n2;
    return S;
  }
};

// One wave composites one 8 x 8 block, a pixel per lane, as the 3D forward
// does: each lane culls its own record of a batch of 64 against the block
// (records loaded while the batch before them is composited) and the ones that
// reach it are packed into LDS in list order.  What bounds it: VALU issue; one
// wave per 16 x 16 tile took 1383 us on 250k surfels over 4 x 1200x680 and 526
// us on 20k over one 321x243 frame, this takes 976 and 87 us.  COUNT: also count the evaluated
// (pixel, entry) pairs, those whose box test passes before the pixel stops
// (one atomic add per block).
template <int TW, int TH, bool COUNT>
__global__ void __launch_bounds__(kWave) surfel_fwd_kernel(
    int first, int n_tiles, int groups, const uint32_t* __restrict__ order,
    uint32_t* __restrict__ tile_nproc, unsigned long long* __restrict__ pair_count,
    int n_frames, const FrameDesc* __restrict__ frames, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ vals, const Surfel* __restrict__ rec, float bg0, float bg1,
    float bg2, float* __restrict__ rgb, float* __restrict__ depth, float* __restrict__ alpha,
    float* __restrict__ normal, float* __restrict__ dist, float* __restrict__ t_final,
    int32_t* __restrict__ n_last, float* __restrict__ dist_aux /* [P][4]: z_ref, A, D_1, D_2 */) {
  using TB = TileBlocks<TW, TH>;
  __shared__ FwdSurfel sm[kWave + 2];
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
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, D = 0.0f, N0 = 0.0f, N1 = 0.0f, N2 = 0.0f;
  // distortion sums in FP64: the backward's weights e_i = A z_i^2 -
  // 2 z_i D_1 + D_2 and z_i A - D_1 cancel where the entries lie at one
  // depth, which FP32 sums over hundreds of entries cannot resolve
  float ZR = 0.0f;
  double SA = 0.0, S1 = 0.0, S2 = 0.0, DS = 0.0;
  uint32_t last = 0;
  uint64_t open = __ballot(px < fr.width && py < fr.height);  // pixels that have not stopped
  uint64_t hits = 0;
  const auto blend = [&](const FwdSurfel& F) {
    const Surfel S = F.record();
    const uint64_t lanes = F.lanes() & open;
    if (COUNT) hits += __popcll(lanes);
    const SurfelEntry en = surfel_entry(S, px);
    const SurfelHit h = surfel_eval(en, py);
    const float a = fminf(kAlphaMax, en.opacity * h.Gh);
    const float Tn = T * (1.0f - a);
    uint64_t act = __ballot(!(a < kAlphaMin)) & lanes;
    const uint64_t stop = __ballot(Tn < kTMin) & act;
    open &= ~stop;
    act &= ~stop;
    if (__builtin_amdgcn_inverse_ballot_w64(act)) {
      const float w = a * T;
      C0 += S.c0 * w;
      C1 += S.c1 * w;
      C2 += S.c2 * w;
      D += h.z * w;
      N0 += S.n0 * w;
      N1 += S.n1 * w;
      N2 += S.n2 * w;
      if (last == 0) ZR = h.z;
      const double zp = h.z - ZR, wd = w;
      DS += wd * (SA * zp * zp - 2.0 * zp * S1 + S2);
      SA += wd;
      S1 += wd * zp;
      S2 += wd * zp * zp;
      T = Tn;
      last = F.pos;
    }
  };
  // the batch's record in registers and the next batch's list entry; lanes past
  // the list's end read the list's first entry again
  const auto entry = [&](uint32_t e) { return e < rg.y ? vals[e] : vals[rg.x]; };
  Surfel R;
  uint32_t v_next = 0;
  if (rg.x < rg.y) {
    R = rec[entry(rg.x + lane)];
    v_next = entry(rg.x + kWave + lane);
  }
  for (uint32_t b = rg.x; b < rg.y && open; b += kWave) {
    uint64_t in = 0;
    if (b + lane < rg.y) in = block_pixels<COUNT>(R, bx, by);
    const uint64_t mk = __ballot(in != 0);
    const int n = __popcll(mk);
    const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u));
    if (in) sm[at].set(R, in, b + lane + 1 - rg.x);
    if (lane < 2) sm[n + lane].px_lo = sm[n + lane].px_hi = 0u;  // (entries are taken in pairs)
    R = rec[v_next];
    v_next = entry(b + 2 * kWave + lane);
    __syncthreads();
    FwdSurfel E0 = sm[0];
    for (int i = 0; i < n && open; i += 2) {
      const FwdSurfel E1 = sm[i + 1];
      blend(E0);
      E0 = sm[i + 2];
      blend(E1);
    }
    __syncthreads();
  }
  // the tile's walk length for the backward and the next schedule: the
  // largest list position any of its pixels blended
  int most = (int)last;
  for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, kWave));
  if (lane == 0) {
    if (TB::kN == 1) tile_nproc[tile] = (uint32_t)most;
    else if (most > 0) atomicMax(&tile_nproc[tile], (uint32_t)most);  // cleared by the order kernel
  }
  if (COUNT && lane == 0) atomicAdd(pair_count, (unsigned long long)hits);
  if (px < fr.width && py < fr.height) {
    const int64_t plane = (int64_t)fr.width * fr.height;
    const int64_t p = (int64_t)py * fr.width + px;
    float* img = rgb + 3 * fr.pixel_offset;
    img[p] = C0 + T * bg0;
    img[plane + p] = C1 + T * bg1;
    img[2 * plane + p] = C2 + T * bg2;
    float* nm = normal + 3 * fr.pixel_offset;
    nm[p] = N0;
    nm[plane + p] = N1;
    nm[2 * plane + p] = N2;
    depth[fr.pixel_offset + p] = D;
    alpha[fr.pixel_offset + p] = 1.0f - T;
    t_final[fr.pixel_offset + p] = T;
    n_last[fr.pixel_offset + p] = (int32_t)last;
    dist[fr.pixel_offset + p] = (float)DS;
    float4* ax = reinterpret_cast<float4*>(dist_aux) + (fr.pixel_offset + p);
    *ax = make_float4(ZR, (float)SA, (float)S1, (float)S2);
  }
}

// Per key (one surfel in one tile), the values the backward reduces: the
// gradients of the columns A = s_u t_u, B = s_v t_v and mc of
// M = K [A | B | mc], as sums the chain rule only scales.  With h_u =
// x M2 - M0, h_v = y M2 - M1 and (o_x, o_y) = (x - c_x^K, y - c_y^K) the
// pixel's offset from the principal point, column j's gradient is
//   (-f_x S_u[j], -f_y S_v[j], R[j]),  S_u = sum dL/dh_u, S_v = sum dL/dh_v,
//   R[j] = sum o_x dL/dh_u[j] + o_y dL/dh_v[j] + dL/dz (u, v, 1)[j],
// so no large product of a pixel position with a sum is left to cancel in
// the chain rule.  The low-pass term's gradient of the centre c =
// (M0_z, M1_z) / M2_z folds into column 2.  Order: S_u[3], S_v[3], R[3],
// opacity, colour[3], normal[3].
constexpr int kSG = 16;

//
// A workgroup takes a tile with WAVES waves of PIX 8 x 8 blocks each, as the 3D
// backward does; the 16 values are summed over a wave's lanes by FP64 matrix
// products (v_mfma_f64_4x4x4, whose operand and result lanes raster.hip
// states): four values at a time over lane bits 5 and 4 into the columns of
// one result, the four results over lane bits 1 and 0 into the columns of
// another, two row rotations for the remaining bits.  What bounds it: VALU
// issue (~190 instructions a visit, half of them FP64).  One wave per tile and
// a reduction through LDS took 3810 us on 250k surfels over 4 x 1200x680 and
// 843 us on 20k over one 321x243 frame; this takes 3340 and 319, the latter 207
// us in eight segments (both launches).
constexpr int kBatchB = 64;          // list entries per batch
constexpr int kBwdMinWaves = 4096;  // four waves on each of the 1,024 SIMDs

template <int WAVES>
struct BwdLds {
  Surfel sm[WAVES > 1 ? 2 : 1][kBatchB];
  uint32_t slot[WAVES > 1 ? 2 : 1][kBatchB];
  double tot[WAVES > 1 ? WAVES : 1][WAVES > 1 ? kBatchB : 1][kSG];
  uint64_t summed[WAVES];  // the batch's entries the wave has sums for
};

template <int TW, int TH, int PIX, BwdPass PASS>
__global__ void __launch_bounds__(TW* TH / PIX) surfel_bwd_kernel(
    double2* __restrict__ maps, int n_tiles, int groups, const uint32_t* __restrict__ order,
    const uint32_t* __restrict__ tile_nproc,
    int n_frames, const FrameDesc* __restrict__ frames, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ vals, const Surfel* __restrict__ rec,
    const uint32_t* __restrict__ keyoff, float bg0, float bg1,
    float bg2, const float* __restrict__ g_rgb, const float* __restrict__ g_depth,
    const float* __restrict__ g_alpha, const float* __restrict__ g_normal,
    const float* __restrict__ g_dist, const float* __restrict__ t_final,
    const int32_t* __restrict__ n_last, const float* __restrict__ dist_aux,
    float* __restrict__ partial, uint32_t* __restrict__ stamp,
    const uint32_t* __restrict__ epoch_dev) {
  using TB = TileBlocks<TW, TH>;
  constexpr int WAVES = TB::kN / PIX;
  constexpr int kCols = PIX < TB::kX ? PIX : TB::kX;
  static_assert(TB::kX % kCols == 0, "blocks of a wave form a rectangle");
  __shared__ BwdLds<WAVES> L;
  const int tile = tile_of_block(blockIdx.x, n_tiles, groups, order);
  if (tile < 0) return;
  int nproc = (int)tile_nproc[tile];
  // the segment's entries, from now on positions 0 .. nproc of a list of its own
  int seg0 = 0;
  const int seg = PASS == kBwdMaps ? blockIdx.y + 1 : blockIdx.y;
  if (PASS != kBwdWhole) {
    const int len =
        (int)segment_len(nproc, kBatchB, PASS == kBwdMaps ? gridDim.y + 1 : gridDim.y);
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
  uint2 rg = ranges[tile];
  rg.x += seg0;
  // the maps of the tile's pixels, segment after segment from the second
  double2* my_maps = nullptr;
  if (PASS != kBwdWhole)
    my_maps = maps + (int64_t)tile * (PASS == kBwdMaps ? gridDim.y : gridDim.y - 1) * (TW * TH) +
              wave * kWave + lane;
  const int64_t plane = (int64_t)fr.width * fr.height;
  // per pixel: T_{i+1} and the totals of the distortion sums.  dL/da_i takes
  // the upstream-weighted difference G . (v_i - B_i) between the entry's
  // values (colour, depth, normal, distortion weight e, alpha 1) and those
  // seen behind it; it cancels where neighbouring surfels agree, so it is
  // formed in FP64.  G is fixed per pixel, so the recursion
  // B_i = B_{i+1} + a_i (v_i - B_{i+1}) carries over to the scalar
  // E = G . B - G_A, which the pixel keeps (FP64) together with G in FP64.
  float T[PIX], AT[PIX], ZR[PIX], S1[PIX], S2[PIX];
  double E[PIX], H0[PIX], H1[PIX], H2[PIX], HD[PIX], HN0[PIX], HN1[PIX], HN2[PIX], HE[PIX];
  int last[PIX];
  int most[PIX];     // the block's longest walk (wave-uniform)
#pragma unroll
  for (int k = 0; k < PIX; ++k) {
    const int px = bx0 + (k % kCols) * kBlk + (lane & 7);
    const int py = by0 + (k / kCols) * kBlk + (lane >> 3);
    // pixels outside read the nearest one inside, and its values are dropped:
    // the loads need no branch each, so that all are in flight together
    const bool valid = px < fr.width && py < fr.height;
    const int64_t p = (int64_t)min(py, fr.height - 1) * fr.width + min(px, fr.width - 1);
    const int64_t q = fr.pixel_offset + p;
    const int nl = n_last[q];
    const float tf = t_final[q];
    const float4 ax = reinterpret_cast<const float4*>(dist_aux)[q];
    const float* gi = g_rgb + 3 * fr.pixel_offset;
    const float* gn = g_normal + 3 * fr.pixel_offset;
    const float g0 = gi[p], g1 = gi[plane + p], g2 = gi[2 * plane + p];
    const float gn0 = gn[p], gn1 = gn[plane + p], gn2 = gn[2 * plane + p];
    const float gd = g_depth[q], ge = g_dist[q], ga = g_alpha[q];
    last[k] = valid ? nl - seg0 : 0;
    T[k] = valid ? tf : 1.0f;
    ZR[k] = valid ? ax.x : 0.0f;
    AT[k] = valid ? ax.y : 0.0f;
    S1[k] = valid ? ax.z : 0.0f;
    S2[k] = valid ? ax.w : 0.0f;
    H0[k] = valid ? g0 : 0.0f;
    H1[k] = valid ? g1 : 0.0f;
    H2[k] = valid ? g2 : 0.0f;
    HN0[k] = valid ? gn0 : 0.0f;
    HN1[k] = valid ? gn1 : 0.0f;
    HN2[k] = valid ? gn2 : 0.0f;
    HD[k] = valid ? gd : 0.0f;
    HE[k] = valid ? ge : 0.0f;
    const double ha = valid ? ga : 0.0f;
    // behind the last entry: the background colour, zero depth, normal, e and
    // alpha (less G_A, the share of every entry's alpha of 1 in G . v_i)
    E[k] = __builtin_fma(H2[k], (double)bg2,
                         __builtin_fma(H1[k], (double)bg1, H0[k] * (double)bg0)) -
           ha;
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
    most[k] = __builtin_amdgcn_readfirstlane(mx);
  }
  double through = 1.0;  // kBwdMaps: the product of 1 - alpha
  double unit[4];  // right operands: unit columns
#pragma unroll
  for (int c = 0; c < 4; ++c) unit[c] = (lane & 3) == c ? 1.0 : 0.0;
  // lane 16 c + g of the last product holds value 4 g + c
  const int out_v = lane & 12 ? -1 : 4 * (lane & 3) + (lane >> 4);
  // Per-entry sums over the lane's pixels, FP64.  A lane adds to them only past
  // the alpha test, so they are still zero after an entry no lane blended
  // and are reset only after an entry that was reduced (the empty asm keeps
  // the zeros from being rewritten on every branch of the first block).
  double acc[kSG];
#pragma unroll
  for (int i = 0; i < kSG; ++i) {
    acc[i] = 0.0;
    asm volatile("" : "+v"(acc[i]));
  }
  // Batches of list entries from the back: [hi - kBatchB, hi).  The batch's
  // list entry is loaded ahead.
  int hi = nproc, buf = 0;
  uint32_t r_cur = 0;
  if (lane < hi) r_cur = vals[rg.x + max(0, hi - kBatchB) + lane];
  for (; hi > 0; hi -= kBatchB, buf ^= WAVES > 1) {
    const int lo = max(0, hi - kBatchB);
    const bool has = lane < hi - lo;
    uint64_t mk[PIX], in[PIX], any = 0;
    {
      const Surfel R = rec[r_cur];  // (lanes past the batch: a record all the same)
#pragma unroll
      for (int k = 0; k < PIX; ++k) {
        in[k] = 0;
        if (has && lo + lane < most[k])
          in[k] = block_pixels<false>(R, bx0 + (k % kCols) * kBlk, by0 + (k / kCols) * kBlk);
        mk[k] = __ballot(in[k] != 0);
        any |= mk[k];
      }
      if (WAVES == 1 ? (any >> lane) & 1 : has && (lane & (WAVES - 1)) == wave) {
        L.sm[buf][lane] = R;
        // the record's tile rect, from its pixel bounds
        const int rx0 = (int)(R.sqx & 0xffff) / TW, rx1 = (int)(R.sqx >> 16) / TW;
        const int ry0 = (int)(R.sqy & 0xffff) / TH;
        L.slot[buf][lane] = keyoff[r_cur] + (uint32_t)((ty - ry0) * (rx1 - rx0 + 1) + (tx - rx0));
      }
    }
    if (lane < lo) r_cur = vals[rg.x + max(0, lo - kBatchB) + lane];
    __syncthreads();  // (also: the previous batch's sums have been read)
    uint64_t summed = 0;
    while (any) {
      const int j = 63 - __builtin_clzll(any);
      any &= ~(1ull << j);
      const int pos = lo + j;
      const Surfel& S = L.sm[buf][j];
      uint64_t hit = 0;
#pragma unroll
      for (int k = 0; k < PIX; ++k) {
        if (PIX > 1 && !((mk[k] >> j) & 1)) continue;  // block missed (uniform)
        const int px = bx0 + (k % kCols) * kBlk + (lane & 7);
        const int py = by0 + (k / kCols) * kBlk + (lane >> 3);
        const SurfelEntry en = surfel_entry(S, px);
        const SurfelHit h = surfel_eval(en, py);
        const float sg = en.opacity * h.Gh;
        const float a = fminf(kAlphaMax, sg);
        const uint64_t act = __ballot(!(a < kAlphaMin)) & __ballot(pos < last[k]) &
                             readlane64(in[k], j);
        hit |= act;
        if (!__builtin_amdgcn_inverse_ballot_w64(act)) continue;
        const float om = 1.0f - a;
        const double zp = h.z - ZR[k];
        // dDist/dw_i: sum over the other entries m of w_m (z_i - z_m)^2
        const double e = AT[k] * zp * zp - 2.0 * zp * S1[k] + S2[k];
        // G . (v_i - B_i) = G . v_i - E
        double diff = __builtin_fma(H0[k], (double)S.c0, -E[k]);
        diff = __builtin_fma(H1[k], (double)S.c1, diff);
        diff = __builtin_fma(H2[k], (double)S.c2, diff);
        diff = __builtin_fma(HD[k], (double)h.z, diff);
        diff = __builtin_fma(HN0[k], (double)S.n0, diff);
        diff = __builtin_fma(HN1[k], (double)S.n1, diff);
        diff = __builtin_fma(HN2[k], (double)S.n2, diff);
        diff = __builtin_fma(HE[k], e, diff);
        E[k] = __builtin_fma((double)a, diff, E[k]);
        if (PASS == kBwdMaps) {
          through *= (double)om;
          continue;
        }
        const float inv = __builtin_amdgcn_rcpf(om);
        float Ti = T[k] * inv;
        Ti = __builtin_fmaf(__builtin_fmaf(-Ti, om, T[k]), inv, Ti);  // Newton step
        const float w = a * Ti;
        const double wd = w;
        T[k] = Ti;
        const float dLda = Ti * (float)diff;
        acc[10] = __builtin_fma(H0[k], wd, acc[10]);
        acc[11] = __builtin_fma(H1[k], wd, acc[11]);
        acc[12] = __builtin_fma(H2[k], wd, acc[12]);
        acc[13] = __builtin_fma(HN0[k], wd, acc[13]);
        acc[14] = __builtin_fma(HN1[k], wd, acc[14]);
        acc[15] = __builtin_fma(HN2[k], wd, acc[15]);
        // dL/dz_i: the depth map and the distortion, 2 w_i sum_m w_m (z_i - z_m)
        const double dzd = wd * (HD[k] + 2.0 * HE[k] * (zp * AT[k] - S1[k]));
        const bool clamped = sg > kAlphaMax;  // clamped: alpha does not move
        const float dGh = clamped ? 0.0f : dLda * en.opacity;
        acc[9] += clamped ? 0.0f : dLda * h.Gh;
        if (h.obj) {
          // z = M2 . (u, v, 1), G = exp(-(u^2 + v^2)/2), (u, v) = (p0, p1) / p2.
          // The chain through the intersection runs in FP64: its FP32
          // rounding is amplified by the conditioning 1/sin of the two
          // planes, squared for a derivative, and a tilted surfel's
          // per-pixel terms cancel in its rotation gradient.  h_u, h_v are
          // rebuilt from the stored FP32 values (the products are exact in
          // FP64); G and the decisions are the forward's.
          const double ex = h.ex, ey = h.ey;
          const double hux = ex * en.m2x + S.kux, huy = ex * en.m2y + S.kuy, huz = ex * en.zc;
          const double hvx = ey * en.m2x + en.kvx, hvy = ey * en.m2y + en.kvy, hvz = ey * en.zc;
          const double p0 = huy * hvz - huz * hvy, p1 = huz * hvx - hux * hvz;
          // 1/p2: hardware reciprocal and two Newton steps (FP64 accuracy;
          // p2 != 0 where the disk term was blended)
          const double p2 = hux * hvy - huy * hvx;
          double ip = __builtin_amdgcn_rcp(p2);
          ip = __builtin_fma(__builtin_fma(-p2, ip, 1.0), ip, ip);
          ip = __builtin_fma(__builtin_fma(-p2, ip, 1.0), ip, ip);
          const double u = p0 * ip, v = p1 * ip;
          const double gGd = (double)h.Gh * dGh;
          const double gu = -u * gGd + dzd * en.m2x;
          const double gv = -v * gGd + dzd * en.m2y;
          const double ox = (double)px - fr.cx, oy = (double)py - fr.cy;
          const double dp0 = gu * ip, dp1 = gv * ip, dp2 = -(gu * u + gv * v) * ip;
          // p = h_u x h_v: dL/dh_u = h_v x dL/dp, dL/dh_v = dL/dp x h_u
          const double a0 = hvy * dp2 - hvz * dp1, a1 = hvz * dp0 - hvx * dp2,
                       a2 = hvx * dp1 - hvy * dp0;
          const double b0 = dp1 * huz - dp2 * huy, b1 = dp2 * hux - dp0 * huz,
                       b2 = dp0 * huy - dp1 * hux;
          acc[0] += a0;
          acc[1] += a1;
          acc[2] += a2;
          acc[3] += b0;
          acc[4] += b1;
          acc[5] += b2;
          acc[6] += ox * a0 + oy * b0 + u * dzd;
          acc[7] += ox * a1 + oy * b1 + v * dzd;
          acc[8] += ox * a2 + oy * b2 + dzd;
        } else {
          // the low-pass: z = z_c, G_lp = exp(-|(x, y) - c|^2); its gradient
          // of c reaches M0_z, M1_z (S_u[2], S_v[2]) and, with the principal
          // point's share, R[2]
          const float t = 2.0f * h.Gh * dGh / en.zc;
          const float gx = t * h.ex, gy = t * h.ey;
          acc[2] -= gx;
          acc[5] -= gy;
          const float ocx = (S.cxh - fr.cx) + S.cxl, ocy = (S.cyh - fr.cy) + S.cyl;
          acc[8] += dzd - (gx * ocx + gy * ocy);
        }
      }
      if (PASS == kBwdMaps || hit == 0) continue;
      double tot = 0.0;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        double d = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          d = __builtin_amdgcn_mfma_f64_4x4x4f64(acc[4 * g + c], unit[c], d, 0, 0, 0);
        tot = __builtin_amdgcn_mfma_f64_4x4x4f64(d, unit[g], tot, 0, 0, 0);
      }
      if (__builtin_expect(__ballot(!isfinite(tot)) != 0, 0)) {
        // a value that is not finite has met the zeros of the others' columns:
        // sum each value by itself and select
        const int col = lane & 3;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          double d = 0.0;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const double s = __builtin_amdgcn_mfma_f64_4x4x4f64(acc[4 * g + c], 1.0, 0.0, 0, 0, 0);
            if (col == c) d = s;
          }
          d = __builtin_amdgcn_mfma_f64_4x4x4f64(d, 1.0, 0.0, 0, 0, 0);
          if (col == g) tot = d;
        }
      }
#pragma unroll
      for (int i = 0; i < kSG; ++i) {
        acc[i] = 0.0;
        asm volatile("" : "+v"(acc[i]));
      }
      tot += dpp<kDppRowRor8>(tot);
      tot += dpp<kDppRowRor4>(tot);
      if constexpr (WAVES == 1) {
        const uint32_t sl = L.slot[buf][j];
        if (out_v >= 0) partial[(size_t)sl * kSG + out_v] = (float)tot;
        if (lane == 4) stamp[sl] = epoch;
      } else {
        if (out_v >= 0) L.tot[wave][j][out_v] = tot;
        summed |= 1ull << j;
      }
    }
    if constexpr (PASS == kBwdMaps) {
      __syncthreads();
    } else if constexpr (WAVES > 1) {
      if (lane == 0) L.summed[wave] = summed;
      __syncthreads();
      uint64_t sw[WAVES], all = 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) all |= sw[w] = L.summed[w];
      // 16 threads per entry, the waves' totals in wave order
      const int v = threadIdx.x % kSG;
      for (int j = threadIdx.x / kSG; j < kBatchB; j += WAVES * kWave / kSG) {
        if (!((all >> j) & 1)) continue;
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w)
          if ((sw[w] >> j) & 1) t += L.tot[w][j][v];
        const uint32_t sl = L.slot[buf][j];
        partial[(size_t)sl * kSG + v] = (float)t;
        if (v == 0) stamp[sl] = epoch;
      }
    } else {
      __syncthreads();
    }
  }
  if (PASS == kBwdMaps) my_maps[(seg - 1) * (TW * TH)] = make_double2(through, E[0]);
}

// Per record (surfel, frame): the sum of its keys' partials that this
// backward stamped, FP64.  A group of kSlotGroup lanes shares a record; the
// records come in order of tile count, so the groups of one wave walk lists
// of similar length.
constexpr int kSlotGroup = 8;

__global__ void __launch_bounds__(256) surfel_slot_reduce_kernel(
    uint64_t m, const uint32_t* __restrict__ order, const uint32_t* __restrict__ keyoff,
    const uint32_t* __restrict__ ntiles, const float* __restrict__ partial,
    const uint32_t* __restrict__ stamp, const uint32_t* __restrict__ epoch_dev,
    uint64_t key_capacity, double* __restrict__ sgrad /* [m][kSG] */) {
  const uint32_t epoch = *epoch_dev;
  const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t k = gid / kSlotGroup;
  const int sub = threadIdx.x & (kSlotGroup - 1);
  const bool active = k < m;
  const uint64_t r = active ? order[k] : 0;
  uint32_t cnt = active ? ntiles[r] : 0u;
  const uint32_t off = cnt ? keyoff[r] : 0u;
  if (cnt && (uint64_t)off + cnt > key_capacity) cnt = 0;  // overflowed the key capacity
  double acc[kSG];
#pragma unroll
  for (int j = 0; j < kSG; ++j) acc[j] = 0.0;
  for (uint32_t s = sub; s < cnt; s += kSlotGroup) {
    if (stamp[off + s] != epoch) continue;
    const float* pp = partial + (size_t)(off + s) * kSG;
#pragma unroll
    for (int j = 0; j < kSG; ++j) acc[j] += pp[j];
  }
  // sum over the group's 8 lanes by DPP moves (no LDS round trips): the
  // half-row mirror (partner 7 - l) leaves the group symmetric, then the
  // quad permutes l ^ 2 and l ^ 1 finish; all 8 lanes end with the same
  // total (each add is commutative, so mirrored lanes agree bitwise)
  static_assert(kSlotGroup == 8, "the group reduction is a half-row of DPP lanes");
#pragma unroll
  for (int j = 0; j < kSG; ++j) acc[j] += dpp<kDppHalfMirror>(acc[j]);
#pragma unroll
  for (int j = 0; j < kSG; ++j) acc[j] += dpp<kDppQuadXor2>(acc[j]);
#pragma unroll
  for (int j = 0; j < kSG; ++j) acc[j] += dpp<kDppQuadXor1>(acc[j]);
  if (!active || !ntiles[r]) return;
#pragma unroll
  for (int j0 = 0; j0 < kSG; j0 += kSlotGroup) {
    double v = acc[j0];
#pragma unroll
    for (int j = j0 + 1; j < j0 + kSlotGroup && j < kSG; ++j) v = sub == j - j0 ? acc[j] : v;
    if (j0 + sub < kSG) sgrad[r * kSG + j0 + sub] = v;
  }
}

// Chain rule from the per-key sums to the parameters (FP64), per surfel and
// frame: the record's sum of its key partials gives the gradients of the
// columns of M = K [A | B | mc]: A = s_u t_u, B = s_v t_v,
// mc = R_f mu + t_f, t_u, t_v, t_w the camera-frame axes R_f R_g.  The pose
// twist (rho, phi) moves every camera-frame vector y by phi x y and mc by
// rho as well, so dL/dphi = sum y x dL/dy.
template <int DEG>
__global__ void __launch_bounds__(256) surfel_preprocess_bwd_kernel(
    int64_t n, int n_frames, const FrameDesc* __restrict__ frames,
    const float* __restrict__ poses, const float* __restrict__ means,
    const float* __restrict__ log_scales, const float* __restrict__ quats,
    const float* __restrict__ opac, const float* __restrict__ sh,
    const uint32_t* __restrict__ ntiles, const uint32_t* __restrict__ keyoff,
    const double* __restrict__ sgrad, uint64_t key_capacity, float* __restrict__ g_means,
    float* __restrict__ g_log_scales, float* __restrict__ g_quats, float* __restrict__ g_opac,
    float* __restrict__ g_sh, double* __restrict__ twist_partial /* [F][n_waves][6] */) {
#pragma clang fp contract(off)
  const int64_t g0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = g0 < n;
  const int64_t g = active ? g0 : 0;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) / kWave;
  const int64_t wave_id = g0 / kWave;
  constexpr int nb = (DEG + 1) * (DEG + 1);
  const double su = active ? exp((double)log_scales[2 * g]) : 1.0;
  const double sv = active ? exp((double)log_scales[2 * g + 1]) : 1.0;
  double qh[4];
  for (int a = 0; a < 4; ++a) qh[a] = active ? quats[4 * g + a] : (a == 0 ? 1.0 : 0.0);
  const double qn = sqrt(qh[0] * qh[0] + qh[1] * qh[1] + qh[2] * qh[2] + qh[3] * qh[3]);
  for (int a = 0; a < 4; ++a) qh[a] /= qn;
  const double w = qh[0], x = qh[1], y = qh[2], z = qh[3];
  const double Rg[9] = {1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y - w * z), 2.0 * (x * z + w * y),
                        2.0 * (x * y + w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z - w * x),
                        2.0 * (x * z - w * y), 2.0 * (y * z + w * x), 1.0 - 2.0 * (x * x + y * y)};
  const double o = active ? 1.0 / (1.0 + exp(-(double)opac[g])) : 0.0;
  const double mu[3] = {active ? (double)means[3 * g] : 0.0,
                        active ? (double)means[3 * g + 1] : 0.0,
                        active ? (double)means[3 * g + 2] : 0.0};
  const float* shg = sh + g * nb * 3;
  double dmu[3] = {0, 0, 0}, dR[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, dls[2] = {0, 0}, dop = 0.0;
  float dsh[nb * 3];
  for (int i = 0; i < nb * 3; ++i) dsh[i] = 0.0f;
  bool kept = false;
  for (int f = 0; f < n_frames; ++f) {
    double tw[6] = {0, 0, 0, 0, 0, 0};
    const int64_t r = (int64_t)f * n + g;
    uint32_t cnt = active ? ntiles[r] : 0u;
    kept = kept || cnt > 0;
    const uint32_t off = cnt ? keyoff[r] : 0u;
    if (cnt && (uint64_t)off + cnt > key_capacity) cnt = 0;  // overflowed the key capacity
    if (cnt > 0) {
      double K[kSG];
      for (int i = 0; i < kSG; ++i) K[i] = sgrad[r * kSG + i];
      const FrameDesc fr = frames[f];
      double W[9], tf[3];
      load_pose(poses, f, W, tf);
      double mc[3], T[9];
      for (int i = 0; i < 3; ++i) {
        mc[i] = W[i * 3 + 0] * mu[0] + W[i * 3 + 1] * mu[1] + W[i * 3 + 2] * mu[2] + tf[i];
        for (int j = 0; j < 3; ++j)
          T[i * 3 + j] = W[i * 3 + 0] * Rg[0 * 3 + j] + W[i * 3 + 1] * Rg[1 * 3 + j] +
                         W[i * 3 + 2] * Rg[2 * 3 + j];
      }
      const double fx = fr.fx, fy = fr.fy;
      // gradients of the columns A, B, mc of M = K [A | B | mc]
      double dcol[3][3];
      for (int j = 0; j < 3; ++j) {
        dcol[j][0] = -fx * K[j];
        dcol[j][1] = -fy * K[3 + j];
        dcol[j][2] = K[6 + j];
      }
      const double tu[3] = {T[0], T[3], T[6]}, tv[3] = {T[1], T[4], T[7]};
      const double tn[3] = {T[2], T[5], T[8]};
      const double sgn = (tn[0] * mc[0] + tn[1] * mc[1] + tn[2] * mc[2]) < 0.0 ? 1.0 : -1.0;
      double dT[3][3];  // dT[j] = dL/d(column j of T)
      for (int i = 0; i < 3; ++i) {
        dT[0][i] = su * dcol[0][i];
        dT[1][i] = sv * dcol[1][i];
        dT[2][i] = sgn * K[13 + i];
      }
      dls[0] += su * (dcol[0][0] * tu[0] + dcol[0][1] * tu[1] + dcol[0][2] * tu[2]);
      dls[1] += sv * (dcol[1][0] * tv[0] + dcol[1][1] * tv[1] + dcol[1][2] * tv[2]);
      // T = R_f R_g
      for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
          dR[i * 3 + j] += W[0 * 3 + i] * dT[j][0] + W[1 * 3 + i] * dT[j][1] +
                           W[2 * 3 + i] * dT[j][2];
      dop += K[9];
      // colour: c = max(0, raw), raw = sum_k sh_k Y_k(dir) + 1/2
      double dir[3];
      const double dist = view_dir(W, tf, mu, dir);
      double Y[16];
      sh_basis<DEG>(dir[0], dir[1], dir[2], Y);
      double raw[3] = {0.0, 0.0, 0.0};
      for (int k = 0; k < nb; ++k)
        for (int c = 0; c < 3; ++c) raw[c] += (double)shg[k * 3 + c] * Y[k];
      double draw[3];
      for (int c = 0; c < 3; ++c) draw[c] = raw[c] + 0.5 > 0.0 ? K[10 + c] : 0.0;
      double wk[16];
      for (int k = 0; k < nb; ++k) {
        double acc = 0.0;
        for (int c = 0; c < 3; ++c) {
          dsh[k * 3 + c] += (float)(Y[k] * draw[c]);
          acc += (double)shg[k * 3 + c] * draw[c];
        }
        wk[k] = acc;
      }
      double ddir[3];
      sh_dir_grad<DEG>(dir[0], dir[1], dir[2], wk, ddir);
      const double pr = dir[0] * ddir[0] + dir[1] * ddir[1] + dir[2] * ddir[2];
      double dd[3];
      for (int a = 0; a < 3; ++a) dd[a] = (ddir[a] - dir[a] * pr) / dist;
      const double* dmc = dcol[2];
      for (int a = 0; a < 3; ++a)
        dmu[a] += W[0 * 3 + a] * dmc[0] + W[1 * 3 + a] * dmc[1] + W[2 * 3 + a] * dmc[2] + dd[a];
      // twist: the camera centre moves by -R_f^T rho, so the view direction
      // adds R_f dd to rho; mc and the three axes rotate with phi
      for (int a = 0; a < 3; ++a)
        tw[a] = dmc[a] + W[a * 3 + 0] * dd[0] + W[a * 3 + 1] * dd[1] + W[a * 3 + 2] * dd[2];
      const double* ys[4] = {mc, tu, tv, tn};
      const double* gs[4] = {dmc, dT[0], dT[1], dT[2]};
      for (int m = 0; m < 4; ++m) {
        const double* Yv = ys[m];
        const double* Gv = gs[m];
        tw[3] += Yv[1] * Gv[2] - Yv[2] * Gv[1];
        tw[4] += Yv[2] * Gv[0] - Yv[0] * Gv[2];
        tw[5] += Yv[0] * Gv[1] - Yv[1] * Gv[0];
      }
    }
    {
      // the wave's six twist sums by the transposing VALU reduction
      int idx;
      bool writer;
      const double s = wave_transpose_sum<6>(tw, threadIdx.x & (kWave - 1), idx, writer);
      if (writer) twist_partial[((int64_t)f * n_waves + wave_id) * 6 + idx] = s;
    }
  }
  if (!active) return;
  if (!kept) {  // no frame sees it (culled, or a non-finite parameter)
    for (int a = 0; a < 3; ++a) g_means[g * 3 + a] = 0.0f;
    for (int a = 0; a < 4; ++a) g_quats[g * 4 + a] = 0.0f;
    g_log_scales[2 * g] = g_log_scales[2 * g + 1] = 0.0f;
    g_opac[g] = 0.0f;
    for (int i = 0; i < nb * 3; ++i) g_sh[g * nb * 3 + i] = 0.0f;
    return;
  }
  g_log_scales[2 * g] = (float)dls[0];
  g_log_scales[2 * g + 1] = (float)dls[1];
  quat_grad(qh, qn, dR, g_quats + g * 4);
  for (int a = 0; a < 3; ++a) g_means[g * 3 + a] = (float)dmu[a];
  g_opac[g] = (float)(dop * o * (1.0 - o));
  float* gsh = g_sh + g * nb * 3;
  for (int i = 0; i < nb * 3; ++i) gsh[i] = dsh[i];
}

}  // namespace

size_t surfel_record_bytes() { return sizeof(Surfel); }
size_t surfel_square_offset() { return offsetof(Surfel, sqx); }
int surfel_grad_values() { return kSG; }
int64_t surfel_preprocess_bwd_waves(int64_t n) { return ((n + 255) / 256) * 4; }

void launch_surfel_preprocess(hipStream_t st, int64_t n, int F, const FrameDesc* frames,
                              const float* poses, const float* means, const float* log_scales,
                              const float* quats, const float* opac, const float* sh, int deg,
                              int tile_w, int tile_h, void* rec, uint2* trect,
                              uint32_t* depth_key, uint32_t* rec_id, uint32_t* ntiles) {
  if (n <= 0 || F <= 0) return;
  const dim3 grid((unsigned)((n + 255) / 256), (unsigned)std::min(F, 65535));
#define GSR_SURF_PRE(D)                                                                      \
  hipLaunchKernelGGL(surfel_preprocess_kernel<D>, grid, dim3(256), 0, st, n, F, frames,      \
                     poses, means, log_scales, quats, opac, sh, tile_w, tile_h,             \
                     (Surfel*)rec, trect, depth_key, rec_id, ntiles)
  switch (deg) {
    case 0: GSR_SURF_PRE(0); break;
    case 1: GSR_SURF_PRE(1); break;
    case 2: GSR_SURF_PRE(2); break;
    default: GSR_SURF_PRE(3); break;
  }
#undef GSR_SURF_PRE
}

void launch_surfel_fwd(hipStream_t st, int tw, int th, int n_tiles, int F,
                       const FrameDesc* frames, const uint2* ranges, const uint32_t* vals,
                       const void* rec, const float* bg, float* rgb, float* depth, float* alpha,
                       float* normal, float* dist, float* t_final, int32_t* n_last,
                       float* dist_aux, uint32_t* nproc, const uint32_t* prev_nproc,
                       uint32_t* order, bool xcd_groups, unsigned long long* pairs) {
  if (n_tiles <= 0) return;
  const int groups = tile_schedule_groups(xcd_groups);
  launch_tile_order(st, n_tiles, groups, prev_nproc, order, nproc);
#define GSR_SURF_FWD_C(W, H, C)                                                               \
  for_block_runs(n_tiles, groups, TileBlocks<W, H>::kN, [&](int first, unsigned blocks) {     \
    hipLaunchKernelGGL((surfel_fwd_kernel<W, H, C>), dim3(blocks), dim3(kWave), 0, st, first, \
                       n_tiles, groups, order, nproc, pairs, F, frames, ranges, vals,         \
                       (const Surfel*)rec, bg[0], bg[1], bg[2], rgb, depth, alpha, normal,    \
                       dist, t_final, n_last, dist_aux);                                      \
  })
#define GSR_SURF_FWD(W, H)                 \
  if (pairs) GSR_SURF_FWD_C(W, H, true);   \
  else GSR_SURF_FWD_C(W, H, false)
  if (tw == 16 && th == 16) GSR_SURF_FWD(16, 16);
  else if (tw == 8 && th == 8) GSR_SURF_FWD(8, 8);
  else if (tw == 32 && th == 8) GSR_SURF_FWD(32, 8);
  else if (tw == 16 && th == 8) GSR_SURF_FWD(16, 8);
  else if (tw == 32 && th == 16) GSR_SURF_FWD(32, 16);
#undef GSR_SURF_FWD
#undef GSR_SURF_FWD_C
}

template <int TW, int TH, int PIX>
static void launch_bwd_t(hipStream_t st, int pix, int n_tiles, int groups, const uint32_t* order,
                         int F, const FrameDesc* frames, const uint2* ranges,
                         const uint32_t* vals, const Surfel* rec, const uint32_t* keyoff,
                         const float* bg, const float* g_rgb, const float* g_depth,
                         const float* g_alpha, const float* g_normal, const float* g_dist,
                         const float* t_final, const int32_t* n_last, const float* dist_aux,
                         float* partial, uint32_t* stamp, const uint32_t* epoch,
                         const uint32_t* nproc, int segments, double2* maps) {
  if constexpr (PIX > 1) {
    if (pix < PIX) {
      launch_bwd_t<TW, TH, PIX / 2>(st, pix, n_tiles, groups, order, F, frames, ranges, vals, rec,
                                    keyoff, bg, g_rgb, g_depth, g_alpha, g_normal, g_dist,
                                    t_final, n_last, dist_aux, partial, stamp, epoch, nproc,
                                    segments, maps);
      return;
    }
  }
  const auto go = [&](auto* k, int parts) {
    hipLaunchKernelGGL(k, dim3(tile_schedule_grid(n_tiles, groups), (unsigned)parts),
                       dim3(TW * TH / PIX), 0, st, maps, n_tiles, groups, order, nproc, F, frames,
                       ranges, vals, rec, keyoff, bg[0], bg[1], bg[2], g_rgb, g_depth, g_alpha,
                       g_normal, g_dist, t_final, n_last, dist_aux, partial, stamp, epoch);
  };
  if constexpr (PIX == 1) {
    if (segments > 1) {
      go(surfel_bwd_kernel<TW, TH, 1, kBwdMaps>, segments - 1);
      go(surfel_bwd_kernel<TW, TH, 1, kBwdSegments>, segments);
      return;
    }
  }
  go(surfel_bwd_kernel<TW, TH, PIX, kBwdWhole>, 1);
}

void launch_surfel_bwd(hipStream_t st, int tw, int th, int n_tiles, int F,
                       const FrameDesc* frames, const uint2* ranges, const uint32_t* vals,
                       const void* rec, const uint32_t* keyoff,
                       const float* bg, const float* g_rgb, const float* g_depth,
                       const float* g_alpha, const float* g_normal, const float* g_dist,
                       const float* t_final, const int32_t* n_last, const float* dist_aux,
                       float* partial, uint32_t* stamp, const uint32_t* epoch,
                       const uint32_t* nproc, uint32_t* order, bool xcd_groups, int segments,
                       double2* maps) {
  if (n_tiles <= 0) return;
  const int groups = tile_schedule_groups(xcd_groups);
  launch_tile_order(st, n_tiles, groups, nproc, order);
  // Blocks per wave: as many as leave kBwdMinWaves waves, as in the 3D
  // backward.  Measured with 1 / 2 / 4 blocks (us): 4 x 1200x680 (12,900 tiles
  // of 16x16) 4417 / 4079 / 3325; 1 x 321x243 (336 tiles) 319 / 455 / 713.
  const int blocks = tw * th / kWave;
  int pix = 4;
  while (pix > 1 && (int64_t)n_tiles * blocks / pix < kBwdMinWaves) pix /= 2;
#define GSR_SURF_BWD(W, H)                                                                    \
  launch_bwd_t<W, H, std::min(4, TileBlocks<W, H>::kN)>(                                      \
      st, pix, n_tiles, groups, order, F, frames, ranges, vals, (const Surfel*)rec, keyoff, bg, \
      g_rgb, g_depth, g_alpha, g_normal, g_dist, t_final, n_last, dist_aux, partial, stamp,    \
      epoch, nproc, segments, maps)
  if (tw == 16 && th == 16) GSR_SURF_BWD(16, 16);
  else if (tw == 8 && th == 8) GSR_SURF_BWD(8, 8);
  else if (tw == 32 && th == 8) GSR_SURF_BWD(32, 8);
  else if (tw == 16 && th == 8) GSR_SURF_BWD(16, 8);
  else if (tw == 32 && th == 16) GSR_SURF_BWD(32, 16);
#undef GSR_SURF_BWD
}

void launch_surfel_slot_reduce(hipStream_t st, uint64_t m, const uint32_t* order,
                               const uint32_t* keyoff, const uint32_t* ntiles,
                               const float* partial, const uint32_t* stamp,
                               const uint32_t* epoch, uint64_t key_capacity, double* sgrad) {
  if (m == 0) return;
  const uint64_t threads = m * kSlotGroup;
  hipLaunchKernelGGL(surfel_slot_reduce_kernel, dim3((unsigned)((threads + 255) / 256)),
                     dim3(256), 0, st, m, order, keyoff, ntiles, partial, stamp, epoch,
                     key_capacity, sgrad);
}

void launch_surfel_preprocess_bwd(hipStream_t st, int64_t n, int F, const FrameDesc* frames,
                                  const float* poses, const float* means,
                                  const float* log_scales, const float* quats,
                                  const float* opac, const float* sh, int deg,
                                  const uint32_t* ntiles, const uint32_t* keyoff,
                                  const double* sgrad, uint64_t key_capacity, float* g_means,
                                  float* g_log_scales, float* g_quats, float* g_opac,
                                  float* g_sh, double* twist_partial, float* g_twist) {
  if (n > 0) {
    const dim3 grid((unsigned)((n + 255) / 256));
#define GSR_SURF_PRE_BWD(D)                                                                   \
  hipLaunchKernelGGL(surfel_preprocess_bwd_kernel<D>, grid, dim3(256), 0, st, n, F, frames,  \
                     poses, means, log_scales, quats, opac, sh, ntiles, keyoff, sgrad,         \
                     key_capacity, g_means, g_log_scales, g_quats, g_opac, g_sh, twist_partial)
    switch (deg) {
      case 0: GSR_SURF_PRE_BWD(0); break;
      case 1: GSR_SURF_PRE_BWD(1); break;
      case 2: GSR_SURF_PRE_BWD(2); break;
      default: GSR_SURF_PRE_BWD(3); break;
    }
#undef GSR_SURF_PRE_BWD
  }
  launch_twist_reduce(st, F, twist_partial, n > 0 ? surfel_preprocess_bwd_waves(n) : 0, g_twist);
}

}  // namespace gsr
