// Device-side CG scalar logic (text after Eq. 16: alpha = r.z / p.Ap,
// beta = r_new.z_new / r.z, z the preconditioned residual, stop at
// ||r|| <= eta ||b|| or p.Ap <= 0; p.Ap is formed as p.(K:p), see
// cg_alpha_publish and cg_alpha_consume) and the fixed-order reductions of
// the per-block partial sums.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace rve {

// fixed-order reduction over the block (deterministic for a given block
// size)
__device__ __forceinline__ double cg_block_reduce(double v, double* red) {
  return block_sum_fixed(v, red);
}

// sum of partial[0 .. count) by one block: each thread sums a strided
// subset in index order, then the block tree
__device__ __forceinline__ double cg_sum_partials(const double* partial,
                                                  int count, double* red) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < count; i += blockDim.x) acc += partial[i];
  return cg_block_reduce(acc, red);
}

// The scalars at the start of a CG run (rr0 and rz0 are set)
__host__ __device__ inline void cg_start(Scalars* sc, int max_iters,
                                         double eta) {
  sc->max_iters = max_iters;
  sc->eta2 = eta * eta;
  sc->done = 0;
  sc->converged = 0;
  sc->breakdown = 0;
  sc->iters = 0;
  sc->fails = 0;
  sc->its[0] = 0;
  sc->its[1] = -1;  // iteration 0 has no previous update
  sc->halt[0] = sc->halt[1] = 0;
  sc->alphas[0] = sc->alphas[1] = 0.0;
  sc->xalpha = 0.0;
  sc->xvalid = 0;
}

// Copies the scalars into the host's coherent pinned buffer pub (plain
// vector stores, which reach host memory uncached and are complete when
// the kernel is; the host reads them after waiting for an event recorded
// behind the kernel).  Called by every thread of the block: the barrier
// orders the block's own writes to sc before the copy, which reads them
// back from L2 rather than from the scalar cache.
__device__ __forceinline__ void publish_scalars(const Scalars* sc,
                                                Scalars* pub) {
  static_assert(sizeof(Scalars) % 8 == 0, "Scalars copied in 8-byte words");
  constexpr int W = (int)(sizeof(Scalars) / 8);
  __syncthreads();
  const unsigned long long* src = reinterpret_cast<const unsigned long long*>(sc);
  unsigned long long* dst = reinterpret_cast<unsigned long long*>(pub);
  for (int i = threadIdx.x; i < W; i += blockDim.x)
    dst[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}

// ---- reductions consumed by the next kernel ----------------------------------
// Instead of a one-block reduction launch between two kernels, every block
// of the consuming kernel sums the producer's partials itself in a fixed
// order (every consumer of the same partials in the same order, so all get
// the same number) and takes the scalar decision locally; block 0 alone
// publishes the result.  Iteration k (parity p = k & 1) reads slot p ^ 1
// and publishes slot p, so no block reads what another block of the same
// launch writes.

struct BetaStep {
  bool first;   // iteration 0: the direction is r itself
  bool stop;    // converged, capped or non-finite: no further work
  double beta;
};

// The r.r and r.z partials of the last pencil pass are summed by every
// wavefront of the consumer on its own: lane l adds partial[l],
// partial[l + 64], ... in index order, then a butterfly over the wavefront
// (both lanes of a pair add the same two numbers), so every wavefront of
// every consuming kernel gets the same bits, with no barrier or LDS.  The
// first PU loads of each lane can be issued early (load), away from the sum.
template <int PU>
struct WavePartials {
  double v[PU];
  __device__ __forceinline__ void load(const double* __restrict__ partial,
                                       int count) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int i = l + 64 * u;
      v[u] = partial[i < count ? i : count - 1];  // clamped: no branch
    }
  }
  __device__ __forceinline__ double sum(const double* __restrict__ partial,
                                        int count) const {
    const int l = threadIdx.x & 63;
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < PU; ++u) acc += (l + 64 * u < count) ? v[u] : 0.0;
    for (int i = l + 64 * PU; i < count; i += 64) acc += partial[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    return acc;
  }
};

// The decision of the direction pass of parity p from the r.r and r.z sums
// of the last pencil pass (or, in iteration 0, prev < 0, from the start's).
// k = prev + 1 updates are complete; the thread with pub publishes.
__device__ __forceinline__ BetaStep cg_beta_step(Scalars* sc, int p, int prev,
                                                 double rr, double rz,
                                                 bool pub) {
  const int q = p ^ 1;
  const int k = prev + 1;
  const bool first = prev < 0;
  const double e2bb = first ? sc->eta2 * rr : sc->eta2bb;
  const bool conv = first ? rr == 0.0 : rr <= e2bb;
  BetaStep d{first, conv, 0.0};
  if (!first) d.stop = conv || k >= sc->max_iters || !isfinite(rr);
  if (!first && !d.stop) d.beta = rz / sc->rzs[q];
  if (pub) {
    sc->rrs[p] = rr;
    sc->rzs[p] = rz;
    sc->its[p] = k;
    sc->iters = k;
    sc->rr_new = rr;
    if (first) {
      sc->bb = rr;
      sc->eta2bb = e2bb;
    }
    if (conv) sc->converged = 1;
    if (d.stop) {
      sc->done = 1;
      sc->halt[p] = 1;
      if (first) sc->xalpha = 0.0;
    } else {
      sc->beta = d.beta;
      if (first) sc->xvalid = 1;
    }
  }
  return d;
}

// reduce the partials of the last pencil pass and take the decision (the
// chunk-closing kernel)
__device__ __forceinline__ BetaStep cg_beta_consume(const double* prr,
                                                    const double* prz,
                                                    int count, Scalars* sc,
                                                    int p) {
  const int prev = sc->its[p ^ 1];
  const bool pub = threadIdx.x == 0;
  if (prev < 0) return cg_beta_step(sc, p, prev, sc->rr0, sc->rz0, pub);
  WavePartials<8> a, b;
  a.load(prr, count);
  b.load(prz, count);
  return cg_beta_step(sc, p, prev, a.sum(prr, count), b.sum(prz, count), pub);
}

// alpha_k = r.z / p.(K:p), published by one thread.  Since p lies in the
// range of the projection G and G is an orthogonal projection,
// p.G(K:p) = p.(K:p): alpha is known before the transforms of K:p end, and
// the pencil pass applies r -= alpha G(K:p) as it forms G(K:p).
__device__ __forceinline__ void cg_alpha_set(double pAp, Scalars* sc, int p) {
  if (threadIdx.x != 0) return;
  sc->pAp = pAp;
  if (!(pAp > 0.0) || !isfinite(pAp)) {
    sc->breakdown = 1;
    sc->done = 1;
    sc->halt[p] = 1;
    sc->iters = sc->its[p] + 1;
    sc->xalpha = 0.0;
  } else {
    const double al = sc->rzs[p] / pAp;
    sc->alpha = al;
    sc->alphas[p] = al;
    sc->xalpha = al;
  }
}

// In block 0 of the forward pass of parity p: reduce the p.(K:p) partials of
// the K:p kernel and publish alpha
__device__ __forceinline__ void cg_alpha_publish(const double* partial,
                                                 int count, Scalars* sc,
                                                 int p, double* red) {
  cg_alpha_set(cg_sum_partials(partial, count, red), sc, p);
}

// The residual pass forms alpha itself from pass A's partials when K:p is
// folded into pass A: every block the same bits, the one with `pub`
// publishes.  False on a stopped run or a breakdown (no block touches the
// residual then); rzs[p] was published by an earlier pass.
template <typename T>
__device__ __forceinline__ bool cg_alpha_consume(const double* partial,
                                                 int count, Scalars* sc, int p,
                                                 bool pub, T& alpha) {
  if (sc->halt[p] || sc->done) return false;
  double pAp = 0.0;
  for (int i = threadIdx.x & 63; i < count; i += 64) pAp += partial[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) pAp += __shfl_xor(pAp, o, 64);
  const double rz = sc->rzs[p];
  if (pub) cg_alpha_set(pAp, sc, p);
  if (!(pAp > 0.0) || !isfinite(pAp)) return false;
  alpha = T(rz / pAp);
  return true;
}

}  // namespace rve
