// adam.hip -- fused optimiser step of the mapping loop (A13).
//
// The mapper runs a fixed number of optimisation iterations per call
// (DROID-Splat supplementary S1.2: 100 iterations, positional learning rate
// annealed, other parameters as in MonoGS), optimising the Gaussians and,
// when pose refinement is on, the keyframe poses (Sec. 3.3, S1.3).  One
// launch updates the three groups the workload optimises:
//   means      (lr_means)   Adam
//   SH colours (lr_sh)      Adam
//   pose twist (lr_pose)    Adam on xi in se(3), then T_f <- Exp(xi) T_f and
//                           xi <- 0 (the twist is always evaluated at zero)
// with bias-corrected moments m, v and an iteration counter held in device
// memory (incremented by the kernel, so a captured iteration advances it on
// every replay).  The pose fold is FP64.
#include <algorithm>

#include "launch.h"

namespace gsr {

struct AdamHyper {
  float lr_means, lr_sh, lr_pose, beta1, beta2, eps;
};

__device__ __forceinline__ float adam_delta(float g, float& m, float& v, float b1, float b2,
                                            float c1, float c2, float eps) {
  // (the fused forms are spelled out: every caller rounds alike)
  m = fmaf(b1, m, (1.0f - b1) * g);
  v = fmaf(b2, v, (1.0f - b2) * g * g);
  const float mh = m / c1;
  const float vh = v / c2;
  return mh / (sqrtf(vh) + eps);
}

// One group of parameters: p, its gradient and moments.
struct AdamGroup {
  float* __restrict__ p;
  const float* __restrict__ g;
  float* __restrict__ m;
  float* __restrict__ v;
};

__device__ __forceinline__ void adam_one(const AdamGroup& a, uint64_t i, float lr,
                                         const AdamHyper& h, float c1, float c2) {
  float m = a.m[i], v = a.v[i];
  a.p[i] = fmaf(-lr, adam_delta(a.g[i], m, v, h.beta1, h.beta2, c1, c2, h.eps), a.p[i]);
  a.m[i] = m;
  a.v[i] = v;
}

// Gaussians: n3 means and nsh SH coefficients, V at a time (4 where every
// array is 16-byte aligned) and one by one at the end of each group.  Bound by
// memory, 28 bytes per element: at 500k Gaussians of degree 3 (25.5M elements)
// one element per thread took 147 us, four take 132 (5.4 TB/s).
template <int V>
__global__ void __launch_bounds__(256) adam_gauss_kernel(uint64_t n3, uint64_t nsh,
                                                         AdamGroup means, AdamGroup sh,
                                                         AdamHyper h,
                                                         const int32_t* __restrict__ step) {
  const int t = *step + 1;  // the pose kernel of the same launch sequence bumps it
  const float c1 = 1.0f - powf(h.beta1, (float)t);
  const float c2 = 1.0f - powf(h.beta2, (float)t);
  const uint64_t first = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t v3 = n3 / V, vsh = nsh / V;
  for (uint64_t i = first; i < v3 + vsh; i += stride) {
    const bool is_mean = i < v3;
    if constexpr (V == 4) {
      const AdamGroup& a = is_mean ? means : sh;
      const float lr = is_mean ? h.lr_means : h.lr_sh;
      const uint64_t j = is_mean ? i : i - v3;
      float4 p = reinterpret_cast<float4*>(a.p)[j];
      const float4 g = reinterpret_cast<const float4*>(a.g)[j];
      float4 m = reinterpret_cast<float4*>(a.m)[j], v = reinterpret_cast<float4*>(a.v)[j];
      p.x = fmaf(-lr, adam_delta(g.x, m.x, v.x, h.beta1, h.beta2, c1, c2, h.eps), p.x);
      p.y = fmaf(-lr, adam_delta(g.y, m.y, v.y, h.beta1, h.beta2, c1, c2, h.eps), p.y);
      p.z = fmaf(-lr, adam_delta(g.z, m.z, v.z, h.beta1, h.beta2, c1, c2, h.eps), p.z);
      p.w = fmaf(-lr, adam_delta(g.w, m.w, v.w, h.beta1, h.beta2, c1, c2, h.eps), p.w);
      reinterpret_cast<float4*>(a.p)[j] = p;
      reinterpret_cast<float4*>(a.m)[j] = m;
      reinterpret_cast<float4*>(a.v)[j] = v;
    } else if (is_mean) {  // (a branch: addresses by selection take a seventh longer here)
      adam_one(means, i, h.lr_means, h, c1, c2);
    } else {
      adam_one(sh, i - v3, h.lr_sh, h, c1, c2);
    }
  }
  if (first < n3 % V) adam_one(means, n3 - 1 - first, h.lr_means, h, c1, c2);
  if (first < nsh % V) adam_one(sh, nsh - 1 - first, h.lr_sh, h, c1, c2);
}

// One thread per frame: Adam on the twist, then T <- Exp(xi) T with
// Exp(rho, phi) = [R(phi), V(phi) rho], R by Rodrigues, V the SE(3) left
// Jacobian; the last thread advances the iteration counter.
__global__ void adam_pose_kernel(int n_frames, float* __restrict__ poses,
                                 const float* __restrict__ g_twist, float* __restrict__ m_tw,
                                 float* __restrict__ v_tw, AdamHyper h,
                                 int32_t* __restrict__ step) {
  const int f = threadIdx.x;
  const int t = *step + 1;
  if (f < n_frames) {
    const float c1 = 1.0f - powf(h.beta1, (float)t);
    const float c2 = 1.0f - powf(h.beta2, (float)t);
    double xi[6];
    for (int k = 0; k < 6; ++k) {
      float m = m_tw[f * 6 + k], v = v_tw[f * 6 + k];
      xi[k] = -(double)h.lr_pose *
              (double)adam_delta(g_twist[f * 6 + k], m, v, h.beta1, h.beta2, c1, c2, h.eps);
      m_tw[f * 6 + k] = m;
      v_tw[f * 6 + k] = v;
    }
    const double* rho = xi;
    const double* phi = xi + 3;
    const double th2 = phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2];
    const double th = sqrt(th2);
    double A, B, Cc;  // sin(th)/th, (1-cos)/th^2, (th - sin)/th^3
    if (th < 1e-5) {
      A = 1.0 - th2 / 6.0;
      B = 0.5 - th2 / 24.0;
      Cc = 1.0 / 6.0 - th2 / 120.0;
    } else {
      A = sin(th) / th;
      B = (1.0 - cos(th)) / th2;
      Cc = (th - sin(th)) / (th2 * th);
    }
    const double K[9] = {0, -phi[2], phi[1], phi[2], 0, -phi[0], -phi[1], phi[0], 0};
    double K2[9];
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) {
        double acc = 0.0;
        for (int l = 0; l < 3; ++l) acc += K[i * 3 + l] * K[l * 3 + j];
        K2[i * 3 + j] = acc;
      }
    double R[9], V[9];
    for (int i = 0; i < 9; ++i) {
      const double id = (i % 4 == 0) ? 1.0 : 0.0;
      R[i] = id + A * K[i] + B * K2[i];
      V[i] = id + B * K[i] + Cc * K2[i];
    }
    double tr[3];
    for (int i = 0; i < 3; ++i)
      tr[i] = V[i * 3 + 0] * rho[0] + V[i * 3 + 1] * rho[1] + V[i * 3 + 2] * rho[2];
    float* P = poses + f * 12;
    double Rf[9], tf[3];
    for (int i = 0; i < 3; ++i) {
      for (int j = 0; j < 3; ++j) Rf[i * 3 + j] = P[i * 4 + j];
      tf[i] = P[i * 4 + 3];
    }
    for (int i = 0; i < 3; ++i) {
      for (int j = 0; j < 3; ++j)
        P[i * 4 + j] = (float)(R[i * 3 + 0] * Rf[0 * 3 + j] + R[i * 3 + 1] * Rf[1 * 3 + j] +
                               R[i * 3 + 2] * Rf[2 * 3 + j]);
      P[i * 4 + 3] = (float)(R[i * 3 + 0] * tf[0] + R[i * 3 + 1] * tf[1] + R[i * 3 + 2] * tf[2] +
                             tr[i]);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) *step = t;
}

void launch_adam(hipStream_t st, uint64_t n3, uint64_t nsh, float* means, const float* g_means,
                 float* m_means, float* v_means, float* sh, const float* g_sh, float* m_sh,
                 float* v_sh, int n_frames, float* poses, const float* g_twist, float* m_tw,
                 float* v_tw, float lr_means, float lr_sh, float lr_pose, float beta1,
                 float beta2, float eps, int32_t* step) {
  const AdamHyper h{lr_means, lr_sh, lr_pose, beta1, beta2, eps};
  const uint64_t total = n3 + nsh;
  if (total > 0) {
    const AdamGroup a{means, g_means, m_means, v_means}, c{sh, g_sh, m_sh, v_sh};
    uintptr_t bits = 0;
    for (const void* p : {(const void*)means, (const void*)g_means, (const void*)m_means,
                          (const void*)v_means, (const void*)sh, (const void*)g_sh,
                          (const void*)m_sh, (const void*)v_sh})
      bits |= (uintptr_t)p;
    const bool wide = (bits & 15u) == 0;
    const uint64_t per = wide ? 4 : 1;
    const unsigned blocks =
        (unsigned)std::min<uint64_t>((total + 256 * per - 1) / (256 * per), 65536);
    if (wide)
      hipLaunchKernelGGL(adam_gauss_kernel<4>, dim3(blocks), dim3(256), 0, st, n3, nsh, a, c, h,
                         step);
    else
      hipLaunchKernelGGL(adam_gauss_kernel<1>, dim3(blocks), dim3(256), 0, st, n3, nsh, a, c, h,
                         step);
  }
  const int threads = n_frames > 0 ? ((n_frames + 63) / 64) * 64 : 64;
  hipLaunchKernelGGL(adam_pose_kernel, dim3(1), dim3(threads), 0, st, n_frames, poses, g_twist,
                     m_tw, v_tw, h, step);
}

}  // namespace gsr
