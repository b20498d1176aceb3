// Elementwise and reduction kernels of the Newton-CG increment:
//   predictor F = F_prev + dFbar (Sec. 2.1, Eq. 12 with the homogeneous
//   first guess), CG vector updates with FP64-accumulated dot products and
//   fixed-order (deterministic) reductions (text after Eq. 16), the Newton
//   update F += dF, the commit of the increment with the fatigue indicators
//   of Sec. 3.3, Eqs. 23-24.
#include "cg_scalars.hpp"
#include "kernels.hpp"
#include "kp_apply.hpp"
#include "newton.hpp"

namespace rve {

namespace {

__device__ __forceinline__ double block_reduce(double v, double* red) {
  return block_sum_fixed(v, red);
}

}  // namespace

__global__ void predict_kernel(double* __restrict__ F,
                               const double* __restrict__ Fp, int64_t N,
                               double d0, double d1, double d2, double d3,
                               double d4, double d5, double d6, double d7,
                               double d8) {
  const double d[9] = {d0, d1, d2, d3, d4, d5, d6, d7, d8};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 9 * N;
       i += (int64_t)gridDim.x * blockDim.x)
    F[i] = Fp[i] + d[i / N];
}

void launch_predict(double* F, const double* Fprev, const double dFbar[9],
                    int64_t N, hipStream_t s) {
  hipLaunchKernelGGL(predict_kernel, dim3(2048), dim3(kBlock), 0, s, F, Fprev,
                     N, dFbar[0], dFbar[1], dFbar[2], dFbar[3], dFbar[4],
                     dFbar[5], dFbar[6], dFbar[7], dFbar[8]);
}

template <typename T, bool FULL>
__global__ __launch_bounds__(kBlock) void kp_kernel(
    const T* __restrict__ K, const T* __restrict__ p, T* __restrict__ y,
    const Scalars* __restrict__ sc, int64_t N, double* __restrict__ pkp) {
  __shared__ double red[kBlock / 64];
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double acc = kp_voxel<T, FULL>(K, p, y, v < N ? v : N - 1, N, v < N,
                                       &sc->done);
  const double t = block_reduce(acc, red);
  if (threadIdx.x == 0) pkp[blockIdx.x] = t;
}

int kp_blocks(int64_t N) { return (int)((N + kBlock - 1) / kBlock); }

template <typename T>
void launch_kp(const T* K, bool full, const T* p, T* y, const Scalars* sc,
               int64_t N, double* pkp, hipStream_t s) {
  const dim3 grid((unsigned)kp_blocks(N));
  if (full)
    launch((kp_kernel<T, true>), grid, dim3(kBlock), 0, s, K, p, y, sc, N, pkp);
  else
    launch((kp_kernel<T, false>), grid, dim3(kBlock), 0, s, K, p, y, sc, N, pkp);
}

template void launch_kp<float>(const float*, bool, const float*, float*,
                               const Scalars*, int64_t, double*, hipStream_t);
template void launch_kp<double>(const double*, bool, const double*, double*,
                                const Scalars*, int64_t, double*, hipStream_t);

template <typename T>
__global__ void convert_kernel(const double* __restrict__ in,
                               T* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = T(in[i]);
}

template <typename T>
void launch_convert(const double* in, T* out, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL((convert_kernel<T>), dim3(2048), dim3(kBlock), 0, s, in,
                     out, n);
}

// The scalars of an FP64 residual, fixed order: r.r and r.z of the CG start
// and ||G(P)||^2 from 3 x count partials, ||P||^2 and <P>.  One block, a
// wavefront per sum and no barrier between them (thirteen block sums one
// after the other took 10.9 us at 32^3, now 3.7).
constexpr int kRedThreads = 13 * 64;
__device__ __forceinline__ void reduce_residual_block(const RedItem& it,
                                                      Scalars* sc) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const double* src = w < 3    ? it.partial + w * it.count
                      : w == 3 ? it.psq
                               : it.psum + (w - 4) * it.nss;
  const int n = w < 3 ? it.count : w == 3 ? 9 * it.nss : it.nss;
  double v = 0.0;
#pragma unroll 4
  for (int i = l; i < n; i += 64) v += src[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if (l) return;
  if (w == 0) sc->rr0 = v;
  else if (w == 1) sc->rz0 = v;
  else if (w == 2) sc->res2 = v;
  else if (w == 3) sc->P2 = v;
  else sc->pbar[w - 4] = v * it.invN3;
}

__global__ __launch_bounds__(kRedThreads) void reduce_residual_kernel(
    RedItem it, Scalars* __restrict__ sc, Scalars* pub) {
  reduce_residual_block(it, sc);
  if (pub) publish_scalars(sc, pub);
}

// one block per RVE
__global__ __launch_bounds__(kRedThreads) void reduce_batch_kernel(
    const RedItem* __restrict__ items, Scalars* __restrict__ scs) {
  Scalars* sc = scs + blockIdx.x;
  if (!sc->inactive) reduce_residual_block(items[blockIdx.x], sc);
}

void launch_reduce_batch(const RedItem* items, int nitems, Scalars* scs,
                         hipStream_t s) {
  hipLaunchKernelGGL(reduce_batch_kernel, dim3(nitems), dim3(kRedThreads), 0, s,
                     items, scs);
}

// End of a CG chunk: the decision the direction pass of the next iteration
// (parity p) would take, published for the host; it writes only slot p,
// which that pass rewrites with the same values.
__global__ __launch_bounds__(kBlock) void cg_close_kernel(
    const double* __restrict__ prr, const double* __restrict__ prz, int count,
    Scalars* __restrict__ sc, int p, Scalars* pub) {
  if (!sc->done) (void)cg_beta_consume(prr, prz, count, sc, p);
  if (pub) publish_scalars(sc, pub);
}

void launch_cg_close(const double* prr, const double* prz, int count,
                     Scalars* sc, int parity, hipStream_t s, Scalars* pub) {
  hipLaunchKernelGGL(cg_close_kernel, dim3(1), dim3(kBlock), 0, s, prr, prz,
                     count, sc, parity, pub);
}

void launch_reduce_residual(const double* part, int count, const double* psum,
                            const double* psq, int nss, double invN3,
                            Scalars* sc, hipStream_t s, Scalars* pub) {
  hipLaunchKernelGGL(reduce_residual_kernel, dim3(1), dim3(kRedThreads), 0, s,
                     RedItem{part, count, psum, psq, nss, invN3}, sc, pub);
}

__global__ void init_scalars_kernel(Scalars* sc, int max_iters, double eta,
                                    double rr0, double rz0) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    sc->rr0 = rr0;
    sc->rz0 = rz0;
    cg_start(sc, max_iters, eta);
  }
}

__global__ void bench_scalars_kernel(Scalars* sc) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    // an iteration that leaves the residual unchanged (alpha = beta = 0)
    // and reads every vector
    sc->done = 0;
    sc->alpha = 0.0;
    sc->beta = 0.0;
    sc->alphas[0] = sc->alphas[1] = 0.0;
  }
}

void launch_bench_scalars(Scalars* sc, hipStream_t s) {
  hipLaunchKernelGGL(bench_scalars_kernel, dim3(1), dim3(64), 0, s, sc);
}

void launch_init_scalars(Scalars* sc, int max_iters, double eta, double rr0,
                         double rz0, hipStream_t s) {
  hipLaunchKernelGGL(init_scalars_kernel, dim3(1), dim3(64), 0, s, sc,
                     max_iters, eta, rr0, rz0);
}

// Commit: accumulate the indicator fields from the converged trial state.
//   dLp = sum_a dg_a s_a (x) m_a;  Pcyc += sqrt(2/3 dLp:dLp);
//   Pcyc_lit += dLp:dLp / dt;  W_a += tau_a dg_a.
__global__ __launch_bounds__(kBlock) void commit_kernel(CommitArgs A) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= A.N) return;
  const int64_t N = A.N;
  const double* __restrict__ tb = A.table + (int64_t)A.phase[v] * kTableStride;
  if (tb[0] != 0.0) return;  // elastic particles accumulate nothing
  double dLp[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  double dg[12];
#pragma unroll
  for (int al = 0; al < 12; ++al) {
    dg[al] = A.dg_t[al * N + v];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        dLp[3 * i + j] += dg[al] * tb[kTabS + 3 * al + i] * tb[kTabM + 3 * al + j];
  }
  double dd = 0.0;
#pragma unroll
  for (int i = 0; i < 9; ++i) dd += dLp[i] * dLp[i];
  A.pcyc[v] += sqrt(2.0 / 3.0 * dd);
  A.pcyc_lit[v] += dd / A.dt;
  // resolved shear stresses at the converged state
  double F[9], Fpi[9], Fe[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    F[c] = A.F[c * N + v];
    Fpi[c] = A.Fpi_t[c * N + v];
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      Fe[3 * i + j] = F[3 * i] * Fpi[j] + F[3 * i + 1] * Fpi[3 + j] +
                      F[3 * i + 2] * Fpi[6 + j];
  double C[9];
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int q = 0; q < 3; ++q)
      C[3 * p + q] = Fe[p] * Fe[q] + Fe[3 + p] * Fe[3 + q] + Fe[6 + p] * Fe[6 + q];
  const double E[6] = {0.5 * (C[0] - 1.0), 0.5 * (C[4] - 1.0),
                       0.5 * (C[8] - 1.0), 0.5 * C[5],
                       0.5 * C[2],         0.5 * C[1]};
  const double w[6] = {1, 1, 1, 2, 2, 2};
  double S[6];
#pragma unroll
  for (int I = 0; I < 6; ++I) {
    double acc = 0.0;
#pragma unroll
    for (int J = 0; J < 6; ++J) acc += tb[kTabC + 6 * I + J] * w[J] * E[J];
    S[I] = acc;
  }
#pragma unroll
  for (int al = 0; al < 12; ++al) {
    const double* s = tb + kTabS + 3 * al;
    const double* m = tb + kTabM + 3 * al;
    const double Sm0 = S[0] * m[0] + S[5] * m[1] + S[4] * m[2];
    const double Sm1 = S[5] * m[0] + S[1] * m[1] + S[3] * m[2];
    const double Sm2 = S[4] * m[0] + S[3] * m[1] + S[2] * m[2];
    const double tau = s[0] * Sm0 + s[1] * Sm1 + s[2] * Sm2;
    A.wcyc[al * N + v] += tau * dg[al];
  }
}

void launch_commit(const CommitArgs& a, hipStream_t s) {
  const int64_t grid = (a.N + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(commit_kernel, dim3((unsigned)grid), dim3(kBlock), 0, s, a);
}

__global__ void fill_i32_kernel(int32_t* p, int32_t v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}
__global__ void fill_f64_kernel(double* p, double v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  const int64_t g = (n + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)(g < 2048 ? (g > 0 ? g : 1) : 2048)),
                     dim3(kBlock), 0, s, p, v, n);
}
void launch_fill_f64(double* p, double v, int64_t n, hipStream_t s) {
  const int64_t g = (n + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(fill_f64_kernel, dim3((unsigned)(g < 2048 ? (g > 0 ? g : 1) : 2048)),
                     dim3(kBlock), 0, s, p, v, n);
}

// sigma = P F^T / det F
__global__ void cauchy_kernel(const double* __restrict__ F,
                              const double* __restrict__ P,
                              double* __restrict__ sig, int64_t N) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
  double f[9], p[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    f[c] = F[c * N + v];
    p[c] = P[c * N + v];
  }
  const double J = f[0] * (f[4] * f[8] - f[5] * f[7]) -
                   f[1] * (f[3] * f[8] - f[5] * f[6]) +
                   f[2] * (f[3] * f[7] - f[4] * f[6]);
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      sig[(3 * i + j) * N + v] =
          (p[3 * i] * f[3 * j] + p[3 * i + 1] * f[3 * j + 1] +
           p[3 * i + 2] * f[3 * j + 2]) / J;
}

void launch_cauchy(const double* F, const double* P, double* sig, int64_t N,
                   hipStream_t s) {
  const int64_t g = (N + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(cauchy_kernel, dim3((unsigned)g), dim3(kBlock), 0, s, F, P,
                     sig, N);
}

template void launch_convert<float>(const double*, float*, int64_t,
                                    hipStream_t);
template void launch_convert<double>(const double*, double*, int64_t,
                                     hipStream_t);


// ------------------------------------------------------------------ batch
__global__ void newton_control_batch_kernel(Scalars* __restrict__ scs,
                                            BatchLog* __restrict__ log,
                                            int nitems, int it, NewtonCtl ctl) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nitems) return;
  Scalars& sc = scs[b];
  BatchLog& L = log[b];
  if (L.status != 1) return;
  if (it > 0) {  // the linear solve of the previous iteration
    if (it - 1 < kBatchLog) L.cg_hist[it - 1] = sc.iters;
    L.cg_total += sc.iters;
    L.breakdowns += sc.breakdown ? 1 : 0;
  }
  const double res = sqrt(sc.res2), pn = sqrt(sc.P2);
  const double rel = pn > 0.0 ? res / pn : 0.0;
  if (it < kBatchLog) L.res_hist[it] = rel;
  if (it == 0) L.predictor_rel = rel;
  L.rel = rel;
  for (int c = 0; c < 9; ++c) L.pbar[c] = sc.pbar[c];
  L.newton_iters = it;
  int st = 1;
  if (sc.fails > 0) {
    L.fails = sc.fails;
    st = -5;   // RVE_ELOCAL
  } else if (res <= ctl.newton_tol * pn) {
    st = 0;    // RVE_OK
    sc.commit = 1;
  } else if (it >= ctl.newton_max) {
    st = -4;   // RVE_ENOTCONV
  }
  L.status = st;
  if (st != 1) {
    sc.inactive = 1;
    sc.done = 1;
    return;
  }
  const double eta = forcing_eta(ctl.forcing, ctl.cg_tol, ctl.newton_tol, rel);
  cg_start(&sc, ctl.cg_max, eta);
}

void launch_newton_control_batch(Scalars* scs, BatchLog* log, int nitems,
                                 int it, const NewtonCtl& ctl, hipStream_t s) {
  hipLaunchKernelGGL(newton_control_batch_kernel,
                     dim3((unsigned)((nitems + 63) / 64)), dim3(64), 0, s, scs,
                     log, nitems, it, ctl);
}

__global__ void predict_batch_kernel(double* __restrict__ F,
                                     const double* __restrict__ Fp,
                                     const uint8_t* __restrict__ vrve,
                                     const double* __restrict__ dF, int64_t N) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 9 * N;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = i / N;
    F[i] = Fp[i] + dF[9 * vrve[i - c * N] + c];
  }
}

void launch_predict_batch(double* F, const double* Fprev, const uint8_t* vrve,
                          const double* dF, int64_t N, hipStream_t s) {
  hipLaunchKernelGGL(predict_batch_kernel, dim3(2048), dim3(kBlock), 0, s, F,
                     Fprev, vrve, dF, N);
}

// commit of the RVEs flagged in their scalars: committed state <- trial,
// F_prev <- F, the fluctuation increment, and the indicator fields
__global__ __launch_bounds__(kBlock) void commit_batch_kernel(CommitBatchArgs A) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= A.N) return;
  const int b = A.vrve[v];
  if (!A.scs[b].commit) return;
  const int64_t N = A.N;
  double F[9], Fpi[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    F[c] = A.F[c * N + v];
    Fpi[c] = A.Fpi_t[c * N + v];
    A.dFt[c * N + v] = F[c] - A.Fprev[c * N + v] - A.dF[9 * b + c];
    A.Fprev[c * N + v] = F[c];
    A.Pc[c * N + v] = A.P[c * N + v];
    A.Fpi_c[c * N + v] = Fpi[c];
  }
  double dg[12];
#pragma unroll
  for (int al = 0; al < 12; ++al) {
    dg[al] = A.dg_t[al * N + v];
    A.dg_c[al * N + v] = dg[al];
    A.chi_c[al * N + v] = A.chi_t[al * N + v];
  }
  const double* __restrict__ tb = A.table + (int64_t)A.phase[v] * kTableStride;
  if (tb[0] != 0.0) return;
  double dLp[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int al = 0; al < 12; ++al)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        dLp[3 * i + j] += dg[al] * tb[kTabS + 3 * al + i] * tb[kTabM + 3 * al + j];
  double dd = 0.0;
#pragma unroll
  for (int i = 0; i < 9; ++i) dd += dLp[i] * dLp[i];
  A.pcyc[v] += sqrt(2.0 / 3.0 * dd);
  A.pcyc_lit[v] += dd / A.dt;
  double Fe[9];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      Fe[3 * i + j] = F[3 * i] * Fpi[j] + F[3 * i + 1] * Fpi[3 + j] +
                      F[3 * i + 2] * Fpi[6 + j];
  double C[9];
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int q = 0; q < 3; ++q)
      C[3 * p + q] = Fe[p] * Fe[q] + Fe[3 + p] * Fe[3 + q] + Fe[6 + p] * Fe[6 + q];
  const double E[6] = {0.5 * (C[0] - 1.0), 0.5 * (C[4] - 1.0),
                       0.5 * (C[8] - 1.0), 0.5 * C[5],
                       0.5 * C[2],         0.5 * C[1]};
  const double w[6] = {1, 1, 1, 2, 2, 2};
  double S[6];
#pragma unroll
  for (int I = 0; I < 6; ++I) {
    double acc = 0.0;
#pragma unroll
    for (int J = 0; J < 6; ++J) acc += tb[kTabC + 6 * I + J] * w[J] * E[J];
    S[I] = acc;
  }
#pragma unroll
  for (int al = 0; al < 12; ++al) {
    const double* s = tb + kTabS + 3 * al;
    const double* m = tb + kTabM + 3 * al;
    const double Sm0 = S[0] * m[0] + S[5] * m[1] + S[4] * m[2];
    const double Sm1 = S[5] * m[0] + S[1] * m[1] + S[3] * m[2];
    const double Sm2 = S[4] * m[0] + S[3] * m[1] + S[2] * m[2];
    A.wcyc[al * N + v] += (s[0] * Sm0 + s[1] * Sm1 + s[2] * Sm2) * dg[al];
  }
}

void launch_commit_batch(const CommitBatchArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(commit_batch_kernel, dim3((unsigned)((a.N + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, s, a);
}

}  // namespace rve
