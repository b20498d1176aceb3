// y = K : p of one voxel from the stored form of the tangent (material.hip):
// D (6x6, dS2_I = D_IJ e_J with engineering shears e, order 11, 22, 33, 23,
// 13, 12), S2 and H = F - 1:  y = p S2 + F (D : sym(F^T p)).  H and not F: at
// the strains of a metal its rounding is hundreds of times smaller, and the
// products with the unit matrix are exact (a particle's K : p in single
// precision 8.4e-8 from FP64 with F, 5.1e-8 with H; 81 rounded entries 6.1e-8).
#pragma once

#include "kernels.hpp"

namespace rve {

constexpr int kKComp = 51;   // numbers of the stored tangent per voxel
constexpr int kKFull = 81;   // ... of one given as dP/dF (user materials)

// position of the pair (i, j) in the order 11, 22, 33, 23, 13, 12
__host__ __device__ constexpr int voigt(int i, int j) {
  return i == j ? i : 6 - i - j;
}

// engineering strains of sym(F^T p)
template <typename T>
__device__ __forceinline__ void kp_strain(const T* H, const T* p, T* e) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
    e[i] = p[4 * i] + (H[i] * p[i] + H[3 + i] * p[3 + i] + H[6 + i] * p[6 + i]);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = i + 1; j < 3; ++j)
      e[voigt(i, j)] = (p[3 * i + j] + p[3 * j + i]) +
                       (H[i] * p[j] + H[3 + i] * p[3 + j] + H[6 + i] * p[6 + j] +
                        H[j] * p[i] + H[3 + j] * p[3 + i] + H[6 + j] * p[6 + i]);
}

// y of all nine components, K[kKComp] in registers
template <typename T>
__device__ __forceinline__ void kp_apply(const T* K, const T* p, T* y) {
  const T* S = K + 36;
  const T* H = K + 42;
  T e[6], s[6];
  kp_strain(H, p, e);
#pragma unroll
  for (int I = 0; I < 6; ++I) {
    T acc = T(0);
#pragma unroll
    for (int J = 0; J < 6; ++J) acc += K[6 * I + J] * e[J];
    s[I] = acc;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      T acc = T(0);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        acc += p[3 * i + k] * S[voigt(k, j)] + H[3 * i + k] * s[voigt(k, j)];
      y[3 * i + j] = s[voigt(i, j)] + acc;
    }
}

// Material product of a CG direction (Sec. 2.1, Eqs. 15-16): y = K : p per
// voxel and the block's partial of p . y; one voxel per thread, K streamed
// once, coalesced per component.  FULL: K as 81 components of dP/dF (user
// materials); else the stored form of the crystal tangent (kp_apply.hpp).
// The stop flag of the run is tested once the voxel's loads are issued.
// Bound by HBM, at 64^3 by the last-level cache: 276 B per voxel in FP32 take
// 12.8 us at 64^3 (5.7 TB/s) and 116 us at 128^3 (5.0 TB/s); 81 components
// took 17.5 and 167 us.
template <typename T, bool FULL>
__device__ __forceinline__ double kp_voxel(const T* __restrict__ K,
                                           const T* __restrict__ p,
                                           T* __restrict__ y, int64_t v,
                                           int64_t cs, bool in,
                                           const int32_t* done) {
  const int32_t stopped =
      done ? __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  constexpr int NK = FULL ? kKFull : kKComp;
  T kv[NK], pd[9], yv[9];
#pragma unroll
  for (int d = 0; d < 9; ++d) pd[d] = p[d * cs + v];
#pragma unroll
  for (int i = 0; i < NK; ++i) kv[i] = K[i * cs + v];
  if (stopped || !in) return 0.0;
  if constexpr (FULL) {
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      yv[c] = T(0);
#pragma unroll
      for (int d = 0; d < 9; ++d) yv[c] += kv[9 * c + d] * pd[d];
    }
  } else {
    kp_apply(kv, pd, yv);
  }
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    y[c * cs + v] = yv[c];
    acc += double(pd[c]) * double(yv[c]);
  }
  return acc;
}

// The same over a batch arena: a block belongs to one RVE (every edge's voxel
// count is a multiple of the block size) and writes that RVE's partial.
template <typename T>
__device__ __forceinline__ void kp_batch_block(const BatchSpec<T>& b, int blk,
                                               double* red) {
  const int64_t v0 = (int64_t)blk * kBlock;
  const SpecItem<T>& it = b.items[b.vrve[v0]];
  if (it.sc->done) return;
  const double acc = kp_voxel<T, false>(b.K, b.p, b.y, v0 + threadIdx.x, b.cs,
                                        true, nullptr);
  const double t = block_sum_fixed(acc, red);
  if (threadIdx.x == 0) it.pkp[(v0 - it.off) / kBlock] = t;
}

}  // namespace rve
