// The linear map G(A) = F^-1{ Ghat : F(A) } of Sec. 2.1, Eqs. 10-11, and the
// CG iteration on G(K : p) of Eqs. 15-16 over a cubic grid of N^3 voxels:
//
//   forward slabs, pass A (one block per x-slab and component group): the
//     field, or K:p formed on the spot (SRC_KROW); rows y and y + N/2 packed
//     as one complex line, FFT along z, the two half spectra unpacked in
//     place (kz < N/2; the kz = N/2 Nyquist plane is zeroed by the operator,
//     so its slots hold the kz = 0 column's second half), FFT along y, the
//     spectrum stored as [c][x][ky][kz] (kz < N/2);
//   inverse slabs, pass C: the inverse, from two planes per tensor row;
//     writes the real field, or adds it to F at the end of a solve.
//   Between them, for a field (pencil_body, one block per ky, tile of kz and
//   tensor row): FFT along x, the projection Bhat_ij = v_j (sum_l Ahat_il
//   v_l) / |v|^2 (zero at the null frequency and wherever a component is
//   Nyquist; Sec. 2.2, Eqs. 18-21) with the 1/N^3 of the inverse transform,
//   inverse FFT along x.
//   A CG iteration, whose vectors stay in Fourier space, runs
//     direction pencils (pencil_inv_body: x += alpha p, p = z + beta p,
//     inverse FFT along x), inverse slabs (p), K:p, forward slabs, residual
//     pencils (pencil_fwd_body: FFT along x, r -= alpha G(K:p), r.r, r.z).
//
// Only the delta_ik structure of the operator is used: row i of the output
// depends on row i of the input.
#include "cg_scalars.hpp"
#include "common.hpp"
#include "fft.hpp"
#include "kernels.hpp"
#include "kp_apply.hpp"
#include "../../include/rve.h"

#include <type_traits>

namespace rve {

template <int N>
struct SlabGeom {
  static constexpr int H = N / 2;
  static constexpr int PITCH = N + 1;                 // LDS row pitch (complex)
  static constexpr int PLANE = H * PITCH;             // one packed plane
};

// rows of the packed plane: line = q*H + y', element = z
template <int N>
struct RowMap {
  __device__ __forceinline__ int operator()(int line, int e) const {
    const int q = line / SlabGeom<N>::H;
    const int yp = line - q * SlabGeom<N>::H;
    return q * SlabGeom<N>::PLANE + yp * SlabGeom<N>::PITCH + e;
  }
};

// spectral columns: line = q*H + kz, element = ky
template <int N>
struct ColMap {
  __device__ __forceinline__ int operator()(int line, int y) const {
    constexpr int H = SlabGeom<N>::H;
    const int q = line / H;
    const int kz = line - q * H;
    int row, col;
    if (y < H) {
      row = y;
      col = kz;
    } else {
      row = y - H;
      col = (kz == 0) ? H : N - kz;
    }
    return q * SlabGeom<N>::PLANE + row * SlabGeom<N>::PITCH + col;
  }
};

__device__ __forceinline__ int xcd_remap(int b, int nb) {
  // consecutive workgroups land on different XCDs (round robin over 8);
  // give neighbouring logical tiles the same XCD so they share its L2
  if (nb % 8) return b;
  return (b % 8) * (nb / 8) + b / 8;
}

__device__ __forceinline__ double block_sum(double v, double* red) {
  // fixed-order reduction over the block (deterministic)
  return block_sum_fixed(v, red);
}

// items whose global loads are issued together before their LDS stores:
// FP32 eight, or 32 on grids of 128 (whose slab planes leave two blocks per
// CU, so that the registers are there), which makes each pass's loads one
// chunk in flight at once; FP64 eight (pass A at 64^3 16.2 us one at a time,
// now 15.2; the FP64 forward slabs of a batch of 664 k voxels 44 and 40.7)
template <typename T, int N>
constexpr int kStage = sizeof(T) == 4 && N >= 128 ? 32 : 8;

// The twiddles of a body.  DEFER (an FP32 body whose data loads are one
// chunk per thread): loaded into a register at its start (one per thread,
// N <= kBlock) and written to LDS once the data loads are in flight, so
// that their latency overlaps that of the data; otherwise written to LDS
// at once (kept in a register across a loop of chunks, the value would be
// parked in scratch memory).
template <typename T, int N>
constexpr bool kDeferTw(int per) {
  return sizeof(T) == 4 && per <= kStage<T, N>;
}
template <typename T, int N, bool DEFER>
struct TwiddleStage {
  static_assert(N <= kBlock, "one twiddle per thread");
  cplx<T> v;
  __device__ __forceinline__ void load(const cplx<T>* __restrict__ g,
                                       cplx<T>* tw) {
    if constexpr (DEFER)
      v = g[(int)threadIdx.x < N ? (int)threadIdx.x : N - 1];  // no branch
    else if ((int)threadIdx.x < N)
      tw[threadIdx.x] = g[threadIdx.x];
  }
  __device__ __forceinline__ void store(cplx<T>* tw) const {
    if constexpr (DEFER)
      if ((int)threadIdx.x < N) tw[threadIdx.x] = v;
  }
};

// A run's stop flag, read when a body starts and consulted once its first
// data loads are issued (a stopped CG run's passes return without work).
// The relaxed atomic read makes it a vector load issued ahead of the data
// loads, whose in-order completion lets the check wait for it alone; a
// scalar load would be waited for together with the kernel arguments,
// before any data load is issued.
__device__ __forceinline__ int32_t stop_flag(const Scalars* gate) {
  return gate ? __hip_atomic_load(&gate->done, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT)
              : 0;
}
// The flag's first use: an empty statement that takes the register, so
// that the compiler neither tests the flag (and waits for its load) before
// this point nor moves the data loads above it.
__device__ __forceinline__ bool stopped_now(int32_t f) {
  asm volatile("" : "+v"(f));
  return f != 0;
}

// ------------------------------------------------------------------ pass A
// lb: logical block within this RVE's pass-A grid
// gate: the run's scalars when the pass must return at once on a stopped
// run (returns false then); with SRC_KROW the check precedes all work
template <typename T, int N, int CPB, int SRC, int NT = kBlock>
__device__ __forceinline__ bool slab_fwd_body(const SlabFwdArgs<T>& a, int lb,
                                              cplx<T>* lds, cplx<T>* tw,
                                              double* red,
                                              const Scalars* gate = nullptr) {
  constexpr int H = N / 2;
  constexpr int NG = 9 / CPB;
  const int64_t cs = a.cs;
  const int x = lb / NG;
  const int grp = lb - x * NG;
  const int32_t stopped = stop_flag(gate);
  if (SRC != SRC_FIELD && stopped_now(stopped)) return false;
  constexpr int PER0 = (H * N + NT - 1) / NT;
  TwiddleStage<T, N, SRC == SRC_FIELD && kDeferTw<T, N>(PER0)> tws;
  if (a.tw) tws.load(a.tw, tw);   // else the kernel has filled tw
  double ss[CPB], s1[CPB];
#pragma unroll
  for (int q = 0; q < CPB; ++q) ss[q] = s1[q] = 0.0;

  // build the real plane(s), packed: row y' holds y' (re) and y'+H (im);
  // each thread builds both rows of a (y', z) slot and stores one complex
  if constexpr (SRC == SRC_FIELD) {
    // the loads of a chunk of items are issued together, then the chunk is
    // written to LDS (same per-thread order of the sums as item by item)
    constexpr int PER = (H * N + NT - 1) / NT;
    constexpr int CH = PER < kStage<T, N> ? PER : kStage<T, N>;
    for (int c0 = 0; c0 < PER; c0 += CH) {
      T val[CH][2][CPB];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int t = threadIdx.x + (c0 + u) * NT;
        if (c0 + u < PER && t < H * N) {
          const int yp = t / N, z = t - (t / N) * N;
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const int64_t v = ((int64_t)x * N + yp + hh * H) * N + z;
#pragma unroll
            for (int q = 0; q < CPB; ++q)
              val[u][hh][q] = a.field[(grp * CPB + q) * cs + v];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int t = threadIdx.x + (c0 + u) * NT;
        if (c0 + u < PER && t < H * N) {
          const int yp = t / N, z = t - (t / N) * N;
#pragma unroll
          for (int q = 0; q < CPB; ++q) {
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
              ss[q] += double(val[u][hh][q]) * double(val[u][hh][q]);
              s1[q] += double(val[u][hh][q]);
            }
            lds[q * SlabGeom<N>::PLANE + yp * SlabGeom<N>::PITCH + z] =
                cplx<T>{val[u][0][q], val[u][1][q]};
          }
        }
      }
    }
  }
  if (a.tw) tws.store(tw);
  if (stopped_now(stopped)) return false;
  double kacc[CPB];  // p . (K:p) of each component over the slab
#pragma unroll
  for (int q = 0; q < CPB; ++q) kacc[q] = 0.0;
  for (int t = threadIdx.x; SRC == SRC_KROW && t < H * N; t += NT) {
    const int yp = t / N, z = t - (t / N) * N;
    T out[2][CPB];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int64_t v = ((int64_t)x * N + yp + hh * H) * N + z;
      T pd[9];
#pragma unroll
      for (int d = 0; d < 9; ++d) pd[d] = a.field[d * cs + v];
      if (a.kfull) {
#pragma unroll
        for (int q = 0; q < CPB; ++q) {
          const int c = grp * CPB + q;
          T acc = T(0);
#pragma unroll
          for (int d = 0; d < 9; ++d) acc += a.K[(9 * c + d) * cs + v] * pd[d];
          out[hh][q] = acc;
        }
      } else {
        // components of one tensor row i = grp (CPB 3) or c = 3 i + j
        T H[9], e[6];
#pragma unroll
        for (int d = 0; d < 9; ++d) H[d] = a.K[(42 + d) * cs + v];
        kp_strain(H, pd, e);
        auto row = [&](int i, int j) {
          T acc = T(0), sij = T(0);
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const int I = voigt(k, j);
            T s = T(0);
#pragma unroll
            for (int J = 0; J < 6; ++J) s += a.K[(6 * I + J) * cs + v] * e[J];
            if (k == i) sij = s;
            const T pk = i == 0 ? pd[k] : (i == 1 ? pd[3 + k] : pd[6 + k]);
            const T hk = i == 0 ? H[k] : (i == 1 ? H[3 + k] : H[6 + k]);
            acc += pk * a.K[(36 + I) * cs + v] + hk * s;
          }
          return sij + acc;
        };
        if constexpr (CPB == 3) {
#pragma unroll
          for (int q = 0; q < CPB; ++q) out[hh][q] = row(grp, q);
        } else {
          out[hh][0] = row(grp / 3, grp % 3);
        }
      }
#pragma unroll
      for (int q = 0; q < CPB; ++q) {
        const int c = grp * CPB + q;
        // the direction's component c, without an indexed register
        T pc = pd[0];
#pragma unroll
        for (int d = 1; d < 9; ++d) pc = (c == d) ? pd[d] : pc;
        kacc[q] += double(pc) * double(out[hh][q]);
      }
    }
#pragma unroll
    for (int q = 0; q < CPB; ++q)
      lds[q * SlabGeom<N>::PLANE + yp * SlabGeom<N>::PITCH + z] =
          cplx<T>{out[0][q], out[1][q]};
  }
  __syncthreads();

  // FFT along z of the packed rows
  fft_lines<N, -1>(lds, tw, CPB * H, RowMap<N>());

  // unpack the two real-row spectra in place
  for (int t = threadIdx.x; t < CPB * H * H; t += NT) {
    const int q = t / (H * H);
    const int rem = t - q * H * H;
    const int yp = rem / H, k = rem - (rem / H) * H;
    cplx<T>* row = &lds[q * SlabGeom<N>::PLANE + yp * SlabGeom<N>::PITCH];
    if (k == 0) {
      const cplx<T> z0 = row[0];
      row[0] = {z0.x, T(0)};  // A_0 (real)
      row[H] = {z0.y, T(0)};  // B_0 (real), kept in the Nyquist slot
    } else {
      const cplx<T> zk = row[k], zm = row[N - k];
      const cplx<T> A = {T(0.5) * (zk.x + zm.x), T(0.5) * (zk.y - zm.y)};
      const cplx<T> B = {T(0.5) * (zk.y + zm.y), T(0.5) * (zm.x - zk.x)};
      row[k] = A;
      row[N - k] = B;
    }
  }
  __syncthreads();

  // FFT along y of every kz column
  fft_lines<N, -1>(lds, tw, CPB * H, ColMap<N>());

  // store the spectrum [c][x][ky][kz]
  const ColMap<N> cm;
  for (int t = threadIdx.x; t < CPB * N * H; t += NT) {
    const int q = t / (N * H);
    const int rem = t - q * N * H;
    const int ky = rem / H, kz = rem - (rem / H) * H;
    const int c = grp * CPB + q;
    a.spec[((size_t)(c * N + x) * N + ky) * H + kz] = lds[cm(q * H + kz, ky)];
  }
  if (SRC == SRC_KROW && a.pkp_out) {
    // per component and slab: the same sums under every schedule
#pragma unroll
    for (int q = 0; q < CPB; ++q) {
      const double t1 = block_sum(kacc[q], red);
      if (threadIdx.x == 0) a.pkp_out[(grp * CPB + q) * N + x] = t1;
    }
  }
  if (a.psum) {
    // per-slab, per-component sum and sum of squares: [9][N]
#pragma unroll
    for (int q = 0; q < CPB; ++q) {
      const double t1 = block_sum(s1[q], red);
      const double t2 = block_sum(ss[q], red);
      if (threadIdx.x == 0) {
        const int c = grp * CPB + q;
        a.psum[c * N + x] = t1;
        a.psq[c * N + x] = t2;
      }
    }
  }
  return true;
}

// ------------------------------------------------------------------ pass B
// G of one tensor row i: FFT along x, the projection, and back.  Only two
// lines of a row are transformed each way: v_y and v_z do not depend on x, so
// y_0 and v_y y_1 + v_z y_2 go forward, and of the result s v (s the row's
// scalar per frequency) v_x s and s come back; the slab pass applies v_y and
// v_z to the latter.  In double precision this pass takes 13.3 us at 64^3
// (31 MB, 2.4 TB/s) and 8.9 us at 40^3; with three lines and three planes
// written it took 13.9 and 9.6 us.  The chain load, two transforms, store of
// a block bounds it, not the bytes.
template <typename T, int N, int TT>
struct ProjGeom {
  static constexpr int TP = TT + 1;        // LDS pitch of a kx row
  static constexpr int LS = N * TP + TT;   // LDS stride of a line group
  static constexpr int LDS = 2 * LS;
  static constexpr int NTILE = (N / 2 + TT - 1) / TT;
};

template <typename T, int N, int TT>
__device__ __forceinline__ void pencil_body(const PencilArgs<T>& a, int lb,
                                            cplx<T>* lds, cplx<T>* tw) {
  using G = ProjGeom<T, N, TT>;
  constexpr int H = N / 2, TP = G::TP, LS = G::LS;
  const int i = lb % 3, rest = lb / 3;
  const int tile = rest % G::NTILE, ky = rest / G::NTILE, kz0 = tile * TT;
  const int ncol = (H - kz0) < TT ? (H - kz0) : TT;
  auto plane = [&](int j, int x, int tt) {
    return ((size_t)((3 * i + j) * N + x) * N + ky) * H + kz0 + tt;
  };
  if (ky == H) {  // Nyquist ky: the projection is zero there
    for (int t = threadIdx.x; t < 2 * N * TT; t += kBlock) {
      const int j = t / (N * TT), rem = t - j * N * TT;
      const int x = rem / TT, tt = rem - (rem / TT) * TT;
      if (tt < ncol) a.spec[plane(j, x, tt)] = {T(0), T(0)};
    }
    return;
  }
  constexpr int PER = (N * TT + kBlock - 1) / kBlock;
  constexpr int CH = PER < 4 ? PER : 4;
  for (int t = threadIdx.x; t < N; t += kBlock) tw[t] = a.tw[t];
  const T v2 = a.vt[N + ky];
  for (int c0 = 0; c0 < PER; c0 += CH) {
    cplx<T> y[CH][3];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int t = threadIdx.x + (c0 + u) * kBlock;
      const int x = t / TT, tt = t - (t / TT) * TT;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        y[u][j] = {T(0), T(0)};
        if (c0 + u < PER && t < N * TT && tt < ncol) y[u][j] = a.spec[plane(j, x, tt)];
      }
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int t = threadIdx.x + (c0 + u) * kBlock;
      const int x = t / TT, tt = t - (t / TT) * TT;
      if (c0 + u < PER && t < N * TT) {
        const T v3 = a.vt[2 * N + (tt < ncol ? kz0 + tt : 0)];
        lds[x * TP + tt] = y[u][0];
        lds[LS + x * TP + tt] = {v2 * y[u][1].x + v3 * y[u][2].x,
                                 v2 * y[u][1].y + v3 * y[u][2].y};
      }
    }
  }
  __syncthreads();
  auto pm = [](int line, int kx) {
    const int j = line / TT;
    return j * LS + kx * TP + (line - j * TT);
  };
  fft_lines<N, -1>(lds, tw, 2 * TT, pm);
  for (int t = threadIdx.x; t < N * TT; t += kBlock) {
    const int kx = t / TT, tt = t - (t / TT) * TT, kz = kz0 + tt;
    const T v1 = a.vt[kx];
    const T v3 = a.vt[2 * N + (kz < H ? kz : 0)];
    const bool zero = kx == H || tt >= ncol || (kx == 0 && ky == 0 && kz == 0);
    const T inv = zero ? T(0) : a.invN3 / (v1 * v1 + v2 * v2 + v3 * v3);
    const cplx<T> y0 = lds[kx * TP + tt], y1 = lds[LS + kx * TP + tt];
    const cplx<T> q = {(y0.x * v1 + y1.x) * inv, (y0.y * v1 + y1.y) * inv};
    lds[kx * TP + tt] = {v1 * q.x, v1 * q.y};
    lds[LS + kx * TP + tt] = q;
  }
  __syncthreads();
  fft_lines<N, +1>(lds, tw, 2 * TT, pm);
  for (int t = threadIdx.x; t < 2 * N * TT; t += kBlock) {
    const int j = t / (N * TT), rem = t - j * N * TT;
    const int x = rem / TT, tt = rem - (rem / TT) * TT;
    if (tt < ncol) a.spec[plane(j, x, tt)] = lds[j * LS + x * TP + tt];
  }
}

// ------------------------------------- CG vectors in the x-transformed pencils
// The vectors of a CG run live in Fourier space.  A compatible field is
// A_ij = a_i v_j per frequency, so three half spectra hold the residual
// (rho_i = sum_j R_ij v_j of the unnormalised spectrum R), the direction
// (pi_i, p_ij = pi_i v_j with the 1/N^3 of the inverse transform) and the
// iterate (xi_i, the same), layout [i][ky][kx][kz].  G needs no tensor of its
// own: the projection of K:p is the contraction with v, so
//   pencil_fwd_body: FFT along x of K:p, rho -= alpha (K:p) v, and the norms
//     r.r = sum |rho|^2 / |v|^2 / N^3 and r.z (Parseval; every frequency of
//     one half space counts twice);
//   pencil_inv_body: z = M r, pi = z + beta pi, xi += alpha_prev pi_prev, and
//     the inverse FFT along x of the direction.
// M = I - prec n (x) n, n = v/|v|, is the Green operator of an isotropic
// medium up to a factor, prec = (lambda + mu)/(lambda + 2 mu): a plain CG for
// prec = 0.  Of row i only two lines are transformed each way: v_y and v_z
// are constant along x, so y_i2 and y_i3 are combined before the forward
// transform, and the inverse needs pi_i and v_x pi_i.
// In the plane kz = 0 both a frequency and its mirror are stored.  Their
// transforms round differently, and the part of rho that is not Hermitian
// would never be reduced (the real field does not contain it): the mirror
// half (mirrored) is left out of the norms, and the direction takes the
// other half's rho there.
// Bound by the latency of one load, six-line transform and store per block.
template <int N>
__device__ __forceinline__ bool mirrored(int kx, int ky, int kz) {
  return kz == 0 && (ky > N / 2 || (ky == 0 && kx > N / 2));
}

template <typename T, int N, int TT>
struct PencilGeom {
  static constexpr int H = N / 2;
  static constexpr int TP = TT + 1;          // LDS pitch of a kx row
  static constexpr int LS = N * TP + TT;     // LDS stride of a line group
  static constexpr int LDS = 6 * LS;
  static constexpr int NTILE = (H + TT - 1) / TT;
};

template <int N, int TT>
struct PencilMap {
  __device__ __forceinline__ int operator()(int line, int kx) const {
    const int j = line / TT;
    return j * PencilGeom<float, N, TT>::LS + kx * (TT + 1) + (line - j * TT);
  }
};

// the frequency of a pencil item, its wave vector, and 1/|v|^2 (zero where
// the operator is: the null frequency and the Nyquist ones)
template <typename T, int N>
struct Freq {
  T v1, v2, v3, inv;
  double wgt;
  __device__ __forceinline__ Freq(const T* __restrict__ vt, int kx, int ky,
                                  int kz, bool in) {
    constexpr int H = N / 2;
    const int kzc = kz < H ? kz : 0;
    v1 = vt[kx];
    v2 = vt[N + ky];
    v3 = vt[2 * N + kzc];
    const bool zero = !in || kx == H || ky == H || (kx == 0 && ky == 0 && kz == 0);
    const T n2 = v1 * v1 + v2 * v2 + v3 * v3;
    inv = zero ? T(0) : T(1) / n2;
    wgt = mirrored<N>(kx, ky, kz) ? 0.0 : 2.0;
  }
};

template <int N>
__device__ __forceinline__ size_t sv_index(int i, int ky, int kx, int kz) {
  return ((size_t)(i * N + ky) * N + kx) * (N / 2) + kz;
}

// RES: rho = -(P v) of the FP64 residual, rounded to TR, and ||G(P)||^2 in
// pres besides the norms of the rounded one; else rho -= alpha (K:p) v
template <typename T, typename TR, int N, int TT, int NT, bool RES>
__device__ __forceinline__ bool pencil_fwd_body(const PencilFwdArgs<T, TR>& a,
                                                int lb, cplx<T>* lds,
                                                cplx<T>* tw, double* red,
                                                T alpha,
                                                const Scalars* gate) {
  using G = PencilGeom<T, N, TT>;
  constexpr int H = G::H, TP = G::TP, LS = G::LS;
  const int tile = lb % G::NTILE, ky = lb / G::NTILE, kz0 = tile * TT;
  const int ncol = (H - kz0) < TT ? (H - kz0) : TT;
  const int32_t stopped = stop_flag(gate);
  for (int t = threadIdx.x; t < N; t += NT) tw[t] = a.tw[t];
  const T v2 = a.vt[N + ky];
  constexpr int PER = (3 * N * TT + NT - 1) / NT;
  constexpr int CH0 = sizeof(T) == 4 ? 4 : 2;
  constexpr int CH = PER < CH0 ? PER : CH0;
  // this thread's frequencies; their rho is loaded with the spectrum when it
  // is at most two items per thread
  constexpr int PP = (N * TT + NT - 1) / NT;
  constexpr bool kEarly = !RES && PP <= 2;
  cplx<TR> rv[kEarly ? PP : 1][3];
  if constexpr (kEarly) {
#pragma unroll
    for (int u = 0; u < PP; ++u) {
      const int t = threadIdx.x + u * NT;
      const int kx = t / TT, tt = t - (t / TT) * TT;
      if (t < N * TT && tt < ncol)
#pragma unroll
        for (int i = 0; i < 3; ++i) rv[u][i] = a.rho[sv_index<N>(i, ky, kx, kz0 + tt)];
    }
  }
  for (int c0 = 0; c0 < PER; c0 += CH) {
    cplx<T> y[CH][3];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int t = threadIdx.x + (c0 + u) * NT;
#pragma unroll
      for (int j = 0; j < 3; ++j) y[u][j] = {T(0), T(0)};
      if (c0 + u < PER && t < 3 * N * TT) {
        const int i = t / (N * TT), rem = t - i * N * TT;
        const int x = rem / TT, tt = rem - (rem / TT) * TT;
        if (tt < ncol)
#pragma unroll
          for (int j = 0; j < 3; ++j)
            y[u][j] = a.spec[((size_t)((3 * i + j) * N + x) * N + ky) * H + kz0 + tt];
      }
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int t = threadIdx.x + (c0 + u) * NT;
      if (c0 + u < PER && t < 3 * N * TT) {
        const int i = t / (N * TT), rem = t - i * N * TT;
        const int x = rem / TT, tt = rem - (rem / TT) * TT;
        const T v3 = a.vt[2 * N + (tt < ncol ? kz0 + tt : 0)];
        lds[2 * i * LS + x * TP + tt] = y[u][0];
        lds[(2 * i + 1) * LS + x * TP + tt] = {v2 * y[u][1].x + v3 * y[u][2].x,
                                               v2 * y[u][1].y + v3 * y[u][2].y};
      }
    }
  }
  if (stopped_now(stopped)) return false;
  __syncthreads();
  if (ky != H) fft_lines<N, -1>(lds, tw, 6 * TT, PencilMap<N, TT>());

  double srr = 0.0, srz = 0.0, sres = 0.0;
#pragma unroll
  for (int u = 0; u < PP; ++u) {
    const int t = threadIdx.x + u * NT;
    const int kx = t / TT, tt = t - (t / TT) * TT;
    if (t >= N * TT || tt >= ncol) continue;
    const Freq<T, N> f(a.vt, kx, ky, kz0 + tt, true);
    cplx<TR> r[3];
    double w2 = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const cplx<T> y0 = lds[2 * i * LS + kx * TP + tt];
      const cplx<T> y1 = lds[(2 * i + 1) * LS + kx * TP + tt];
      const cplx<T> w = {f.v1 * y0.x + y1.x, f.v1 * y0.y + y1.y};
      const size_t at = sv_index<N>(i, ky, kx, kz0 + tt);
      if constexpr (RES) {
        w2 += double(w.x) * double(w.x) + double(w.y) * double(w.y);
        r[i] = f.inv == T(0) ? cplx<TR>{TR(0), TR(0)} : cplx<TR>{TR(-w.x), TR(-w.y)};
      } else {
        if constexpr (kEarly) r[i] = rv[u][i]; else r[i] = a.rho[at];
        if (f.inv != T(0)) r[i] = {r[i].x - TR(alpha) * TR(w.x), r[i].y - TR(alpha) * TR(w.y)};
      }
      a.rho[at] = r[i];
    }
    double q = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      q += double(r[i].x) * double(r[i].x) + double(r[i].y) * double(r[i].y);
    const T dx = T(r[0].x) * f.v1 + T(r[1].x) * f.v2 + T(r[2].x) * f.v3;
    const T dy = T(r[0].y) * f.v1 + T(r[1].y) * f.v2 + T(r[2].y) * f.v3;
    const double in = f.wgt * double(f.inv);
    const double l = (double(dx) * double(dx) + double(dy) * double(dy)) * double(f.inv);
    srr += in * q;
    srz += in * (q - a.prec * l);
    sres += in * w2;
  }
  const double t1 = block_sum_fixed(srr, red);
  const double t2 = block_sum_fixed(srz, red);
  if (threadIdx.x == 0) {
    a.prr[lb] = t1 * a.invN3;
    a.prz[lb] = t2 * a.invN3;
  }
  if constexpr (RES) {
    const double t3 = block_sum_fixed(sres, red);
    if (threadIdx.x == 0) a.pres[lb] = t3 * a.invN3;
  }
  return true;
}

// FINAL: the inverse FFT along x of the iterate xi + xalpha pi (nothing is
// written but the spectrum); else the next direction and its inverse FFT
template <typename T, int N, int TT, int NT, bool FINAL>
__device__ __forceinline__ void pencil_inv_body(const PencilInvArgs<T>& a,
                                                int lb, cplx<T>* lds,
                                                cplx<T>* tw) {
  using G = PencilGeom<T, N, TT>;
  const bool pub = lb == 0 && threadIdx.x == 0;
  constexpr int H = G::H, TP = G::TP, LS = G::LS;
  const int tile = lb % G::NTILE, ky = lb / G::NTILE, kz0 = tile * TT;
  const int ncol = (H - kz0) < TT ? (H - kz0) : TT;
  // the loads of the vectors and partials are issued before the decision
  constexpr int PP = (N * TT + NT - 1) / NT;
  constexpr bool kEarly = PP <= (sizeof(T) == 4 ? 2 : 1);
  constexpr int PE = kEarly ? PP : 1;
  cplx<T> rv[PE][3], pv[PE][3], xv[PE][3];
  auto load = [&](int u, int w) {
    const int t = threadIdx.x + u * NT;
    const int kx = t / TT, tt = t - (t / TT) * TT;
    if (t < N * TT && tt < ncol)
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const size_t at = sv_index<N>(i, ky, kx, kz0 + tt);
        if (!FINAL) {
          const bool m = mirrored<N>(kx, ky, kz0 + tt);
          const cplx<T> r = a.rho[m ? sv_index<N>(i, (N - ky) % N, (N - kx) % N, 0) : at];
          rv[w][i] = {m ? -r.x : r.x, r.y};   // v is odd: rho(-k) = -conj
        }
        pv[w][i] = a.pi[at];
        xv[w][i] = a.xi[at];
      }
  };
  if constexpr (kEarly) {
#pragma unroll
    for (int u = 0; u < PP; ++u) load(u, u);
  }
  bool first = false;
  T beta = T(0), alpha = T(0);
  bool valid = true;
  Scalars* sc = a.scw;
  if constexpr (FINAL) {
    valid = sc->xvalid != 0;
    alpha = T(sc->xalpha);
  } else if (a.prr) {
    // every flag read here was written by an earlier pass: block 0 of
    // the RVE publishes slot `parity` (and done), which no block reads
    const int q = a.parity ^ 1;
    WavePartials<8> wr, wz;
    wr.load(a.prr, a.count);
    wz.load(a.prz, a.count);
    if (sc->halt[q]) {
      if (pub) sc->halt[a.parity] = 1;
      return;
    }
    const int prev = sc->its[q];
    const double rr = prev < 0 ? sc->rr0 : wr.sum(a.prr, a.count);
    const double rz = prev < 0 ? sc->rz0 : wz.sum(a.prz, a.count);
    const BetaStep d = cg_beta_step(sc, a.parity, prev, rr, rz, pub);
    if (d.stop) return;
    first = d.first;
    beta = T(d.beta);
    alpha = first ? T(0) : T(sc->alphas[q]);
  } else {  // timing: alpha = beta = 0
    beta = T(sc->beta);
    alpha = T(sc->alpha);
  }
  for (int t = threadIdx.x; t < N; t += NT) tw[t] = a.tw[t];
#pragma unroll
  for (int u = 0; u < PP; ++u) {
    const int w = kEarly ? u : 0;
    if constexpr (!kEarly) load(u, 0);
    const int t = threadIdx.x + u * NT;
    const int kx = t / TT, tt = t - (t / TT) * TT;
    if (t >= N * TT) continue;
    const bool in = tt < ncol;
    const Freq<T, N> f(a.vt, kx, ky, kz0 + tt, in);
    cplx<T> p[3];
    if constexpr (FINAL) {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        p[i] = (in && valid) ? xv[w][i] : cplx<T>{T(0), T(0)};
        // after a breakdown (alpha = 0) pi may be infinite or NaN
        if (in && valid && alpha != T(0))
          p[i] = {p[i].x + alpha * pv[w][i].x, p[i].y + alpha * pv[w][i].y};
      }
    } else if (in) {
      const cplx<T>* r = rv[w];
      const T g = a.prec * f.inv;
      const T dx = g * (r[0].x * f.v1 + r[1].x * f.v2 + r[2].x * f.v3);
      const T dy = g * (r[0].y * f.v1 + r[1].y * f.v2 + r[2].y * f.v3);
      const T sc3 = a.invN3 * f.inv;
      const T vv[3] = {f.v1, f.v2, f.v3};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        p[i] = {sc3 * (r[i].x - vv[i] * dx), sc3 * (r[i].y - vv[i] * dy)};
        cplx<T> x = {T(0), T(0)};
        if (!first) {
          p[i] = {p[i].x + beta * pv[w][i].x, p[i].y + beta * pv[w][i].y};
          x = {xv[w][i].x + alpha * pv[w][i].x, xv[w][i].y + alpha * pv[w][i].y};
        }
        const size_t at = sv_index<N>(i, ky, kx, kz0 + tt);
        a.pi[at] = p[i];
        a.xi[at] = x;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) p[i] = {T(0), T(0)};
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      lds[2 * i * LS + kx * TP + tt] = {f.v1 * p[i].x, f.v1 * p[i].y};
      lds[(2 * i + 1) * LS + kx * TP + tt] = p[i];
    }
  }
  __syncthreads();
  if (ky != H) fft_lines<N, +1>(lds, tw, 6 * TT, PencilMap<N, TT>());
  for (int t = threadIdx.x; t < 6 * N * TT; t += NT) {
    const int l = t / (N * TT), rem = t - l * N * TT;
    const int x = rem / TT, tt = rem - (rem / TT) * TT;
    if (tt < ncol)
      a.spec[((size_t)((3 * (l / 2) + (l & 1)) * N + x) * N + ky) * H + kz0 + tt] =
          lds[l * LS + x * TP + tt];
  }
}

// ------------------------------------------------------------------ pass C
// It reads the planes that pencil_body and pencil_inv_body write: component
// 3 i + j is v_j times a spectrum of row i, of which the planes 3 i (j = 0,
// with v_x applied) and 3 i + 1 are stored.
template <typename T, typename TO, int N, int CPB, int DST, int NT = kBlock>
__device__ __forceinline__ bool slab_inv_body(const SlabInvArgs<T, TO>& a,
                                              int lb, cplx<T>* lds,
                                              cplx<T>* tw, double* red,
                                              const Scalars* gate = nullptr) {
  constexpr int H = N / 2;
  constexpr int NG = 9 / CPB;
  const int64_t cs = a.cs;
  const int x = lb / NG;
  const int grp = lb - x * NG;
  const int32_t stopped = stop_flag(gate);
  constexpr int PER0 = (CPB * N * H + NT - 1) / NT;
  TwiddleStage<T, N, kDeferTw<T, N>(PER0)> tws;
  tws.load(a.tw, tw);
  const ColMap<N> cm;
  {
    constexpr int PER = PER0;
    constexpr int CH = PER < kStage<T, N> ? PER : kStage<T, N>;
    for (int c0 = 0; c0 < PER; c0 += CH) {
      cplx<T> val[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int t = threadIdx.x + (c0 + u) * NT;
        if (c0 + u < PER && t < CPB * N * H) {
          const int q = t / (N * H);
          const int rem = t - q * N * H;
          const int ky = rem / H, kz = rem - (rem / H) * H;
          const int c = grp * CPB + q;
          const int pl = c % 3 == 2 ? c - 1 : c;
          val[u] = a.spec[((size_t)(pl * N + x) * N + ky) * H + kz];
        }
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int t = threadIdx.x + (c0 + u) * NT;
        if (c0 + u < PER && t < CPB * N * H) {
          const int q = t / (N * H);
          const int rem = t - q * N * H;
          const int ky = rem / H, kz = rem - (rem / H) * H;
          const int j = (grp * CPB + q) % 3;
          if (j > 0) {
            const T f = a.vt[j == 1 ? N + ky : 2 * N + kz];
            val[u] = {f * val[u].x, f * val[u].y};
          }
          lds[cm(q * H + kz, ky)] = val[u];
        }
      }
    }
  }
  tws.store(tw);
  if (stopped_now(stopped)) return false;
  __syncthreads();
  fft_lines<N, +1>(lds, tw, CPB * H, ColMap<N>());

  // pack the two half spectra of rows y' and y'+H into one complex line
  for (int t = threadIdx.x; t < CPB * H * H; t += NT) {
    const int q = t / (H * H);
    const int rem = t - q * H * H;
    const int yp = rem / H, k = rem - (rem / H) * H;
    cplx<T>* row = &lds[q * SlabGeom<N>::PLANE + yp * SlabGeom<N>::PITCH];
    if (k == 0) {
      const T a0 = row[0].x, b0 = row[H].x;
      row[0] = {a0, b0};
      row[H] = {T(0), T(0)};
    } else {
      const cplx<T> A = row[k], B = row[N - k];
      row[k] = {A.x - B.y, A.y + B.x};        // A + i B
      row[N - k] = {A.x + B.y, B.x - A.y};    // conj(A) + i conj(B)
    }
  }
  __syncthreads();
  fft_lines<N, +1>(lds, tw, CPB * H, RowMap<N>());

  double acc = 0.0;
  for (int t = threadIdx.x; t < H * N; t += NT) {
    const int yp = t / N, z = t - (t / N) * N;
#pragma unroll
    for (int q = 0; q < CPB; ++q) {
      const int c = grp * CPB + q;
      const cplx<T> zz = lds[q * SlabGeom<N>::PLANE + yp * SlabGeom<N>::PITCH + z];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const int64_t v = ((int64_t)x * N + yp + hh * H) * N + z;
        const T val = hh ? zz.y : zz.x;
        if constexpr (DST == DST_ADDF)
          a.out[c * cs + v] += TO(val);
        else
          a.out[c * cs + v] = TO(val);
        if constexpr (DST == DST_NORM) acc += double(val) * double(val);
      }
    }
  }
  if (DST == DST_NORM && a.partial) {
    double tot = block_sum(acc, red);
    if (threadIdx.x == 0) a.partial[lb] = tot;
  }
  return true;
}

// The schedule of the passes that no handle tunes (G of a field, the FP64
// residual): one component per slab block and the tile of cg_tile.  Three
// components per block leave the chip short of blocks (forward slabs in
// double precision, three / one: 6.4 / 5.4 us at 32^3, 13.0 / 9.7 at 48^3).
template <int N>
constexpr int kTile = N < 64 ? 4 : 8;

// ---------------------------------------------------- single-RVE kernels
// Threads of a slab block: 512 where a radix pass of the plane has more than
// 256 butterflies (48^3: 384, 96^3: 1536, 128^3: 1024), so that 256 threads
// go through it in several barrier-separated chunks.  Passes A + C, 256 / 512
// threads: FP32 48^3 15.8 / 14.6 us, 96^3 59.4 / 54.9, 128^3 106.8 / 76.8;
// FP64 19.2 / 18.1, 101.7 / 90.1, 216.5 / 179.7.  At 64^3 (256 butterflies)
// half of 512 threads would idle: FP32 16.1 / 19.5, FP64 23.6 / 29.3; 1024
// threads lose at 96^3 and 128^3 (58.3, 109.9).
template <typename T, int N>
constexpr int kSlabThreads = N == 48 || N >= 96 ? 512 : kBlock;

template <typename T, int N, int CPB, int SRC>
__global__ __launch_bounds__((kSlabThreads<T, N>)) void slab_fwd_kernel(
    SlabFwdArgs<T> a) {
  constexpr int NT = kSlabThreads<T, N>;
  __shared__ cplx<T> lds[CPB * SlabGeom<N>::PLANE];
  __shared__ cplx<T> tw[N];
  __shared__ double red[NT / 64];
  // done comes from an earlier launch, except after a breakdown that block
  // 0 of this launch publishes at its end (cg_alpha_publish): blocks that
  // read done before that write and go on only fill the spectrum, which
  // the passes of a stopped run never read (they return on done).  The body
  // reads it and returns once its loads are issued.
  if (!slab_fwd_body<T, N, CPB, SRC, NT>(a, xcd_remap(blockIdx.x, gridDim.x),
                                         lds, tw, red, a.sc))
    return;
  if (a.pkp && blockIdx.x == 0)
    cg_alpha_publish(a.pkp, a.pkp_count, a.scw, a.parity, red);
}

template <typename T, int N, int TT>
__global__ __launch_bounds__(kBlock) void pencil_proj_kernel(PencilArgs<T> a) {
  __shared__ cplx<T> lds[ProjGeom<T, N, TT>::LDS];
  __shared__ cplx<T> tw[N];
  pencil_body<T, N, TT>(a, xcd_remap(blockIdx.x, gridDim.x), lds, tw);
}

// Pass A of a field for a caller without tables: every block computes the
// twiddles that it needs, block 0 also writes them and the wave vectors
// (Sec. 2.2, Eq. 18; continuous Eq. 19: v = q n / L, discrete Eqs. 20-21:
// v = tan(q / 2) n / L; the Nyquist entry is never used and is set to 0) for
// the passes that follow: three launches instead of four.
template <int N>
__global__ __launch_bounds__((kSlabThreads<double, N>)) void slab_fwd_tables_kernel(
    SlabFwdArgs<double> a, ProjTables p) {
  constexpr int NT = kSlabThreads<double, N>;
  __shared__ cplx<double> lds[SlabGeom<N>::PLANE];
  __shared__ cplx<double> tw[N];
  __shared__ double red[NT / 64];
  const int i = threadIdx.x;
  if (i < N) {
    double sn, cs;
    sincospi(-2.0 * (double)i / (double)N, &sn, &cs);
    tw[i] = {cs, sn};
    if (blockIdx.x == 0) p.tw[i] = {cs, sn};
  }
  if (blockIdx.x == 0)
    for (int t = i; t < 3 * N; t += NT) {
      const int d = t / N, idx = t - d * N;
      const int k = idx < N / 2 ? idx : idx - N;
      const double scale = (double)N / (d == 0 ? p.L0 : (d == 1 ? p.L1 : p.L2));
      p.vt[t] = idx == N / 2 ? 0.0
                : p.continuous ? 2.0 * M_PI * (double)k / (double)N * scale
                               : tan(M_PI * (double)k / (double)N) * scale;
    }
  slab_fwd_body<double, N, 1, SRC_FIELD, NT>(a, xcd_remap(blockIdx.x, gridDim.x),
                                             lds, tw, red);
}

// threads of a CG pencil block: 512 once a block has as many frequencies
// (64^3: one butterfly per thread and radix pass, nine loads in flight each)
template <int N, int TT>
constexpr int kPencilThreads = N * TT >= 512 ? 512 : 256;

template <typename T, typename TR, int N, int TT, bool RES>
__global__ __launch_bounds__((kPencilThreads<N, TT>)) void pencil_fwd_kernel(
    PencilFwdArgs<T, TR> a) {
  constexpr int NT = kPencilThreads<N, TT>;
  __shared__ cplx<T> lds[PencilGeom<T, N, TT>::LDS];
  __shared__ cplx<T> tw[N];
  __shared__ double red[NT / 64];
  T alpha = T(0);
  if constexpr (!RES) {
    if (a.pkp) {
      // K:p folded into pass A: every block forms alpha from its partials
      // (the same bits), block 0 publishes it; after a breakdown none of
      // them touches the residual
      if (!cg_alpha_consume(a.pkp, a.pkp_count, a.scw, a.parity,
                            blockIdx.x == 0, alpha))
        return;
    } else {
      alpha = T(a.sc->alphas[a.parity]);
    }
  }
  pencil_fwd_body<T, TR, N, TT, NT, RES>(a, xcd_remap(blockIdx.x, gridDim.x),
                                         lds, tw, red, alpha,
                                         RES || a.pkp ? nullptr : a.sc);
}

template <typename T, int N, int TT, bool FINAL>
__global__ __launch_bounds__((kPencilThreads<N, TT>)) void pencil_inv_kernel(
    PencilInvArgs<T> a) {
  __shared__ cplx<T> lds[PencilGeom<T, N, TT>::LDS];
  __shared__ cplx<T> tw[N];
  pencil_inv_body<T, N, TT, kPencilThreads<N, TT>, FINAL>(
      a, xcd_remap(blockIdx.x, gridDim.x), lds, tw);
}

template <typename T, typename TO, int N, int CPB, int DST>
__global__ __launch_bounds__((kSlabThreads<T, N>)) void slab_inv_kernel(
    SlabInvArgs<T, TO> a) {
  constexpr int NT = kSlabThreads<T, N>;
  __shared__ cplx<T> lds[CPB * SlabGeom<N>::PLANE];
  __shared__ cplx<T> tw[N];
  __shared__ double red[NT / 64];
  slab_inv_body<T, TO, N, CPB, DST, NT>(a, xcd_remap(blockIdx.x, gridDim.x), lds,
                                        tw, red, a.sc);
}

// The schedules that exist (rve_set_fft_schedule): three component planes per
// slab block up to 64 KiB of LDS, so that two blocks share a CU; sixteen kz
// columns per pencil block where three lines of them stay below 64 KiB, which
// gives the six of a CG pencil at most 107 KB of a CU's 160 (128^3 FP32).
template <typename T, int N>
constexpr bool cpb3_fits() {
  return 3 * SlabGeom<N>::PLANE * (int)sizeof(cplx<T>) <= 64 * 1024;
}
template <typename T, int N, int TT>
constexpr bool pencil_fits() {
  return (3 * (N * (TT + 1) + TT) + N) * (int)sizeof(cplx<T>) +
             kBlock * (int)sizeof(double) <= 64 * 1024;
}

// ------------------------------------------------------- batched kernels
// Every RVE of a batch in one launch: block -> (RVE, local block) through
// the descriptor table; the RVE's edge and schedule (components per slab
// block, kz columns per pencil block) select the compiled FFT plan.
// Converged or retired RVEs (Scalars::done for CG work, ::inactive for the
// residual) return at once.
#define RVE_BATCH_SIZES(X) X(16) X(24) X(32) X(40) X(48) X(64)

template <typename T>
__device__ __forceinline__ int batch_item(const BatchSpec<T>& b, int pass,
                                          int blk) {
  // first blocks ascend: a lane per RVE compares, one latency for up to 64
  int r = -1;
  for (int r0 = 0; r0 < b.nitems; r0 += 64) {
    const int l = r0 + (int)(threadIdx.x & 63);
    const bool le = l < b.nitems && b.items[l].blk[pass] <= blk;
    const int c = __popcll(__ballot(le));
    r += c;
    if (c < 64) break;
  }
  return __builtin_amdgcn_readfirstlane(r);
}

// Blocks of 256 threads at every edge, since one launch holds several: the
// 512 of a single RVE's slabs at 48^3 (kSlabThreads) are too many for its
// smaller neighbours; not timed in a batch of 48^3 alone.
// Each pass as a block body (blk: the block it plays, a launch's blockIdx.x
// or a virtual block of the persistent CG kernel) and a one-launch kernel.
// CPBS: the slab schedules compiled in (bit 0: one component per block,
// bit 1: three), so that a launch whose RVEs all use one of them does not
// carry the registers of the other.  A CG pass leaves an RVE whose run has
// stopped alone, the others one that is inactive.
template <typename T, int NN, int CPB>
__device__ __forceinline__ void slab_fwd_item(const SlabFwdArgs<T>& a, int lb,
                                              unsigned char* smem) {
  cplx<T>* lds = reinterpret_cast<cplx<T>*>(smem);
  cplx<T>* tw = lds + CPB * SlabGeom<NN>::PLANE;
  double* red = reinterpret_cast<double*>(tw + NN);
  slab_fwd_body<T, NN, CPB, SRC_FIELD>(a, lb, lds, tw, red);
}
template <typename T, typename TO, int NN, int CPB, int DST>
__device__ __forceinline__ void slab_inv_item(const SlabInvArgs<T, TO>& a,
                                              int lb, unsigned char* smem) {
  cplx<T>* lds = reinterpret_cast<cplx<T>*>(smem);
  cplx<T>* tw = lds + CPB * SlabGeom<NN>::PLANE;
  double* red = reinterpret_cast<double*>(tw + NN);
  slab_inv_body<T, TO, NN, CPB, DST>(a, lb, lds, tw, red);
}

template <typename T, bool CG, int CPBS = 3>
__device__ __forceinline__ void slab_fwd_batch_block(const BatchSpec<T>& b,
                                                     int blk,
                                                     unsigned char* smem) {
  const int r = batch_item(b, 0, blk);
  const SpecItem<T>& it = b.items[r];
  if (CG ? it.sc->done : it.sc->inactive) return;
  const int lb = blk - it.blk[0];
  SlabFwdArgs<T> a{};
  a.cs = b.cs;
  a.field = (CG ? b.y : b.field) + it.off;
  a.spec = b.spec + it.soff;
  a.tw = it.tw;
  a.psum = CG ? nullptr : it.psum;
  a.psq = it.psq;
  switch (it.n) {
#define RVE_CASE(NN)                                                         \
  case NN:                                                                   \
    if constexpr ((CPBS & 2) && cpb3_fits<T, NN>())                          \
      if (it.cpb == 3) {                                                     \
        slab_fwd_item<T, NN, 3>(a, lb, smem);                                \
        break;                                                               \
      }                                                                      \
    if constexpr ((CPBS & 1) || !cpb3_fits<T, NN>())                         \
      slab_fwd_item<T, NN, 1>(a, lb, smem);                                  \
    break;
    RVE_BATCH_SIZES(RVE_CASE)
#undef RVE_CASE
  }
}

template <typename T, bool CG, int CPBS>
__global__ __launch_bounds__(kBlock) void slab_fwd_batch_kernel(BatchSpec<T> b) {
  extern __shared__ __align__(16) unsigned char smem[];
  slab_fwd_batch_block<T, CG, CPBS>(b, blockIdx.x, smem);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void kp_batch_kernel(BatchSpec<T> b) {
  __shared__ double red[kBlock / 64];
  kp_batch_block<T>(b, blockIdx.x, red);
}

// G of a field: projection of the pencils (blk[2])
template <typename T>
__global__ __launch_bounds__(kBlock) void pencil_batch_kernel(BatchSpec<T> b) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int r = batch_item(b, 2, blockIdx.x);
  const SpecItem<T>& it = b.items[r];
  if (it.sc->inactive) return;
  const int lb = xcd_remap(blockIdx.x - it.blk[2], 3 * it.npen);
  PencilArgs<T> a{};
  a.spec = b.spec + it.soff;
  a.tw = it.tw;
  a.vt = it.vt;
  cplx<T>* lds = reinterpret_cast<cplx<T>*>(smem);
  switch (it.n) {
#define RVE_PENCIL(NN, TT)                                                   \
  {                                                                          \
    a.invN3 = T(1.0 / (double(NN) * NN * NN));                               \
    pencil_body<T, NN, TT>(a, lb, lds, lds + ProjGeom<T, NN, TT>::LDS);       \
    break;                                                                   \
  }
#define RVE_CASE(NN)                                                         \
  case NN:                                                                   \
    if constexpr (pencil_fits<T, NN, 16>())                                  \
      if (it.tt == 16) RVE_PENCIL(NN, 16)                                    \
    if (it.tt == 4) RVE_PENCIL(NN, 4)                                        \
    RVE_PENCIL(NN, 8)
    RVE_BATCH_SIZES(RVE_CASE)
#undef RVE_CASE
#undef RVE_PENCIL
  }
}

// the residual pass of a CG iteration, or (RES) of the FP64 residual
template <typename T, typename TR, bool RES>
__device__ __forceinline__ void pencil_fwd_batch_block(const BatchSpec<T>& b,
                                                       cplx<TR>* rho, int blk,
                                                       unsigned char* smem) {
  const int r = batch_item(b, 1, blk);
  const SpecItem<T>& it = b.items[r];
  // neighbouring tiles share the 128-byte lines of the spectra, so they go to
  // one XCD (a batch of 664 k voxels, FP32: direction pass 24.3 -> 15.0 us,
  // residual pass 18.7 -> 12.9 us)
  const int lb = xcd_remap(blk - it.blk[1], it.npen);
  PencilFwdArgs<T, TR> a{};
  T alpha = T(0);
  if constexpr (RES) {
    if (it.sc->inactive) return;
    a.pres = it.prr + 2 * it.npen;
  } else if (b.timing) {
    alpha = T(it.sc->alpha);
  } else {
    if (!cg_alpha_consume(it.pkp, it.n * it.n * it.n / kBlock, it.sc, b.parity, lb == 0, alpha))
      return;
  }
  a.spec = b.spec + it.soff;
  a.tw = it.tw;
  a.vt = it.vt;
  a.rho = rho + it.soff / 3;
  a.prec = b.prec;
  a.prr = it.prr;
  a.prz = it.prr + it.npen;
  switch (it.n) {
#define RVE_PENCIL(NN, TT)                                                   \
  {                                                                          \
    a.invN3 = 1.0 / (double(NN) * NN * NN);                                  \
    cplx<T>* lds = reinterpret_cast<cplx<T>*>(smem);                         \
    cplx<T>* tw = lds + PencilGeom<T, NN, TT>::LDS;                          \
    pencil_fwd_body<T, TR, NN, TT, kBlock, RES>(                             \
        a, lb, lds, tw, reinterpret_cast<double*>(tw + NN), alpha, nullptr); \
    break;                                                                   \
  }
#define RVE_CASE(NN)                                                         \
  case NN:                                                                   \
    if constexpr (pencil_fits<T, NN, 16>())                                  \
      if (it.tt == 16) RVE_PENCIL(NN, 16)                                    \
    if (it.tt == 4) RVE_PENCIL(NN, 4)                                        \
    RVE_PENCIL(NN, 8)
    RVE_BATCH_SIZES(RVE_CASE)
#undef RVE_CASE
#undef RVE_PENCIL
  }
}

template <typename T, typename TR, bool RES>
__global__ __launch_bounds__(kBlock) void pencil_fwd_batch_kernel(
    BatchSpec<T> b, cplx<TR>* rho) {
  extern __shared__ __align__(16) unsigned char smem[];
  pencil_fwd_batch_block<T, TR, RES>(b, rho, blockIdx.x, smem);
}

template <typename T, bool FINAL>
__device__ __forceinline__ void pencil_inv_batch_block(const BatchSpec<T>& b,
                                                       int blk,
                                                       unsigned char* smem) {
  const int r = batch_item(b, 1, blk);
  const SpecItem<T>& it = b.items[r];
  // a run that stopped in an earlier iteration stays stopped (halt); done
  // itself is written by block 0 of the RVE in this pass
  if (it.sc->inactive) return;
  const int lb = xcd_remap(blk - it.blk[1], it.npen);
  PencilInvArgs<T> a{};
  a.spec = b.spec + it.soff;
  a.tw = it.tw;
  a.vt = it.vt;
  a.rho = b.rho + it.soff / 3;
  a.pi = b.pi + it.soff / 3;
  a.xi = b.xi + it.soff / 3;
  a.prec = T(b.prec);
  a.prr = b.timing ? nullptr : it.prr;
  a.prz = it.prr + it.npen;
  a.count = it.npen;
  a.scw = it.sc;
  a.parity = b.parity;
  switch (it.n) {
#define RVE_PENCIL(NN, TT)                                                   \
  {                                                                          \
    a.invN3 = T(1.0 / (double(NN) * NN * NN));                               \
    cplx<T>* lds = reinterpret_cast<cplx<T>*>(smem);                         \
    pencil_inv_body<T, NN, TT, kBlock, FINAL>(                               \
        a, lb, lds, lds + PencilGeom<T, NN, TT>::LDS);                       \
    break;                                                                   \
  }
#define RVE_CASE(NN)                                                         \
  case NN:                                                                   \
    if constexpr (pencil_fits<T, NN, 16>())                                  \
      if (it.tt == 16) RVE_PENCIL(NN, 16)                                    \
    if (it.tt == 4) RVE_PENCIL(NN, 4)                                        \
    RVE_PENCIL(NN, 8)
    RVE_BATCH_SIZES(RVE_CASE)
#undef RVE_CASE
#undef RVE_PENCIL
  }
}

template <typename T, bool FINAL>
__global__ __launch_bounds__(kBlock) void pencil_inv_batch_kernel(BatchSpec<T> b) {
  extern __shared__ __align__(16) unsigned char smem[];
  pencil_inv_batch_block<T, FINAL>(b, blockIdx.x, smem);
}

template <typename T, typename TO, int DST, int CPBS = 3>
__device__ __forceinline__ void slab_inv_batch_block(const BatchSpec<T>& b,
                                                     TO* out, int blk,
                                                     unsigned char* smem) {
  const int r = batch_item(b, 0, blk);
  const SpecItem<T>& it = b.items[r];
  if (DST == DST_P ? it.sc->done : it.sc->inactive) return;
  const int lb = blk - it.blk[0];
  SlabInvArgs<T, TO> a{};
  a.cs = b.cs;
  a.spec = b.spec + it.soff;
  a.tw = it.tw;
  a.vt = it.vt;
  a.out = out + it.off;
  switch (it.n) {
#define RVE_CASE(NN)                                                         \
  case NN:                                                                   \
    if constexpr ((CPBS & 2) && cpb3_fits<T, NN>())                          \
      if (it.cpb == 3) {                                                     \
        slab_inv_item<T, TO, NN, 3, DST>(a, lb, smem);                       \
        break;                                                               \
      }                                                                      \
    if constexpr ((CPBS & 1) || !cpb3_fits<T, NN>())                         \
      slab_inv_item<T, TO, NN, 1, DST>(a, lb, smem);                         \
    break;
    RVE_BATCH_SIZES(RVE_CASE)
#undef RVE_CASE
  }
}

template <typename T, typename TO, int DST, int CPBS>
__global__ __launch_bounds__(kBlock) void slab_inv_batch_kernel(BatchSpec<T> b,
                                                                TO* out) {
  extern __shared__ __align__(16) unsigned char smem[];
  slab_inv_batch_block<T, TO, DST, CPBS>(b, out, blockIdx.x, smem);
}

// ------------------------------------------------- persistent batched CG
// The CG iterations of every RVE of a batch in one launch of resident
// blocks: the passes of the one-launch form with a grid-wide barrier between
// them; it stops when every RVE's CG is done (converged, broken down or at
// its cap).  A barrier that waits beyond a bound (blocks not all resident)
// sets an error flag and lets the kernel run out instead of hanging; the
// host turns the flag into an error.
// Barrier state (unsigned words, one 128-byte line each part): [0] the
// generation, [32 (1 + g)] the arrival count of group g = blockIdx.x % 8
// (the hardware deals consecutive blocks round-robin over the eight XCDs),
// [32 * 9] the count of groups arrived.  The last block of a group arrives
// at the group count, the last group releases everyone by advancing the
// generation: eight-way instead of all-block contention on one atomic.
constexpr int kBarGroups = 8;
static_assert(32 * (kBarGroups + 2) == kBatchBarWords, "barrier layout");

__device__ __forceinline__ bool grid_barrier(unsigned* bar, unsigned nblocks,
                                             int* err) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
      const unsigned g = blockIdx.x % kBarGroups;
      const unsigned members =
          nblocks / kBarGroups + (g < nblocks % kBarGroups ? 1u : 0u);
      const unsigned groups = nblocks < kBarGroups ? nblocks : kBarGroups;
      const unsigned gen =
          __hip_atomic_load(&bar[0], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
      unsigned* gcount = bar + 32 * (1 + g);
      unsigned* top = bar + 32 * (1 + kBarGroups);
      const unsigned a = __hip_atomic_fetch_add(gcount, 1u, __ATOMIC_ACQ_REL,
                                                __HIP_MEMORY_SCOPE_AGENT) + 1u;
      bool release = false;
      if (a == members) {
        __hip_atomic_store(gcount, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned t = __hip_atomic_fetch_add(top, 1u, __ATOMIC_ACQ_REL,
                                                  __HIP_MEMORY_SCOPE_AGENT) + 1u;
        if (t == groups) {
          __hip_atomic_store(top, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_fetch_add(&bar[0], 1u, __ATOMIC_RELEASE,
                                 __HIP_MEMORY_SCOPE_AGENT);
          release = true;
        }
      }
      if (!release) {
        // bounded wait (about a second); another block's timeout ends it too
        long spins = 0;
        while (__hip_atomic_load(&bar[0], __ATOMIC_ACQUIRE,
                                 __HIP_MEMORY_SCOPE_AGENT) == gen) {
          if (++spins > 2000000L) {
            __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
          }
          if ((spins & 255) == 0 &&
              __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            break;
          __builtin_amdgcn_s_sleep(8);
        }
      }
    }
    __threadfence();
  }
  __syncthreads();
  return __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
}

// the passes as calls (not inlined into one body, which would hold the
// registers of all of them at once)
template <typename T>
__device__ __noinline__ void pc_dir(const BatchSpec<T>& b, int blk,
                                    unsigned char* smem) {
  pencil_inv_batch_block<T, false>(b, blk, smem);
}
template <typename T>
__device__ __noinline__ void pc_p(const BatchSpec<T>& b, int blk,
                                  unsigned char* smem) {
  slab_inv_batch_block<T, T, DST_P>(b, b.p, blk, smem);
}
template <typename T>
__device__ __noinline__ void pc_kp(const BatchSpec<T>& b, int blk,
                                   unsigned char* smem) {
  kp_batch_block<T>(b, blk, reinterpret_cast<double*>(smem));
}
template <typename T>
__device__ __noinline__ void pc_fwd(const BatchSpec<T>& b, int blk,
                                    unsigned char* smem) {
  slab_fwd_batch_block<T, true>(b, blk, smem);
}
template <typename T>
__device__ __noinline__ void pc_res(const BatchSpec<T>& b, int blk,
                                    unsigned char* smem) {
  pencil_fwd_batch_block<T, T, false>(b, b.rho, blk, smem);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void cg_batch_persistent_kernel(
    BatchCG<T> c) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int active;
  for (int j = 0; j < c.max_iters; ++j) {
    const BatchSpec<T>& b = (j & 1) ? c.odd : c.even;
    for (int vb = blockIdx.x; vb < c.blocksB; vb += gridDim.x) {
      pc_dir<T>(b, vb, smem);
      __syncthreads();
    }
    if (!grid_barrier(c.bar, gridDim.x, c.err)) return;
    // every block takes the same decision: done changes next in the
    // residual pass, two barriers on
    if (threadIdx.x == 0) active = 0;
    __syncthreads();
    for (int r = threadIdx.x; r < c.nitems; r += blockDim.x)
      if (!__hip_atomic_load(&c.scs[r].done, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT))
        active = 1;
    __syncthreads();
    if (!active) break;
    for (int vb = blockIdx.x; vb < c.blocksA; vb += gridDim.x) {
      pc_p<T>(b, vb, smem);
      __syncthreads();
    }
    if (!grid_barrier(c.bar, gridDim.x, c.err)) return;
    for (int vb = blockIdx.x; vb < c.blocksV; vb += gridDim.x) {
      pc_kp<T>(b, vb, smem);
      __syncthreads();
    }
    if (!grid_barrier(c.bar, gridDim.x, c.err)) return;
    for (int vb = blockIdx.x; vb < c.blocksA; vb += gridDim.x) {
      pc_fwd<T>(b, vb, smem);
      __syncthreads();
    }
    if (!grid_barrier(c.bar, gridDim.x, c.err)) return;
    for (int vb = blockIdx.x; vb < c.blocksB; vb += gridDim.x) {
      pc_res<T>(b, vb, smem);
      __syncthreads();
    }
    if (!grid_barrier(c.bar, gridDim.x, c.err)) return;
  }
}

template <typename T>
void launch_cg_batch_persistent(const BatchCG<T>& c, int grid, size_t lds,
                                hipStream_t s) {
  hipLaunchKernelGGL((cg_batch_persistent_kernel<T>), dim3(grid), dim3(kBlock),
                     lds, s, c);
}

template <typename T>
int cg_batch_persistent_grid(size_t lds) {
  int dev = 0, per_cu = 0;
  RVE_HIP(hipGetDevice(&dev));
  hipDeviceProp_t prop;
  RVE_HIP(hipGetDeviceProperties(&prop, dev));
  RVE_HIP(hipFuncSetAttribute(
      reinterpret_cast<const void*>(&cg_batch_persistent_kernel<T>),
      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  RVE_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, reinterpret_cast<const void*>(&cg_batch_persistent_kernel<T>),
      kBlock, lds));
  if (per_cu < 1) throw Error(-3, "persistent CG kernel does not fit a CU");
  return per_cu * prop.multiProcessorCount;
}

template void launch_cg_batch_persistent<float>(const BatchCG<float>&, int,
                                                size_t, hipStream_t);
template void launch_cg_batch_persistent<double>(const BatchCG<double>&, int,
                                                 size_t, hipStream_t);
template int cg_batch_persistent_grid<float>(size_t);
template int cg_batch_persistent_grid<double>(size_t);

// ---------------------------------------------------------------- launchers

template <typename T, int N>
void launch_G_n(const SpectralLaunch<T>& L, hipStream_t s) {
  constexpr int TT = kTile<N>;
  SlabFwdArgs<T> fa{};
  fa.cs = (int64_t)N * N * N;
  fa.field = L.in_field;
  fa.spec = L.spec;
  if constexpr (sizeof(T) == 8 && N <= RVE_NOALLOC_MAX_N) {
    if (L.tables.tw)
      launch((slab_fwd_tables_kernel<N>), dim3(9 * N), dim3(kSlabThreads<T, N>), 0,
             s, fa, L.tables);
  }
  if (!L.tables.tw) {
    fa.tw = L.tw;
    launch((slab_fwd_kernel<T, N, 1, SRC_FIELD>), dim3(9 * N),
           dim3(kSlabThreads<T, N>), 0, s, fa);
  }
  PencilArgs<T> pa{};
  pa.spec = L.spec;
  pa.tw = L.tw;
  pa.vt = L.vt;
  pa.invN3 = T(1.0 / (double(N) * N * N));
  launch((pencil_proj_kernel<T, N, TT>), dim3(N * ProjGeom<T, N, TT>::NTILE * 3),
         dim3(kBlock), 0, s, pa);
  SlabInvArgs<T, double> ia{};
  ia.cs = (int64_t)N * N * N;
  ia.spec = L.spec;
  ia.tw = L.tw;
  ia.vt = L.vt;
  ia.out = L.out_d;
  ia.partial = L.partial_inv;
  launch((slab_inv_kernel<T, double, N, 1, DST_NORM>), dim3(9 * N),
         dim3(kSlabThreads<T, N>), 0, s, ia);
}

// the passes of a CG iteration (mask: kPassDir .. kPassRes) or the end of
// the solve (kPassFinal)
template <typename T, int N, int CPB, int TT>
void launch_cg_sched(const CgLaunch<T>& L, int mask, hipStream_t s) {
  using G = PencilGeom<T, N, TT>;
  const int nslab = N * (9 / CPB), npen = N * G::NTILE;
  const T invN3 = T(1.0 / (double(N) * N * N));
  if (mask & (kPassDir | kPassFinal)) {
    PencilInvArgs<T> a{};
    a.spec = L.spec;
    a.tw = L.tw;
    a.vt = L.vt;
    a.rho = L.rho;
    a.pi = L.pi;
    a.xi = L.xi;
    a.invN3 = invN3;
    a.prec = T(L.prec);
    a.prr = L.prr;
    a.prz = L.prz;
    a.count = npen;
    a.scw = L.sc;
    a.parity = L.parity;
    if (mask & kPassDir)
      launch((pencil_inv_kernel<T, N, TT, false>), dim3(npen),
             dim3(kPencilThreads<N, TT>), 0, s, a);
    else
      launch((pencil_inv_kernel<T, N, TT, true>), dim3(npen),
             dim3(kPencilThreads<N, TT>), 0, s, a);
  }
  if (mask & kPassP) {
    SlabInvArgs<T, T> a{};
    a.cs = (int64_t)N * N * N;
    a.spec = L.spec;
    a.tw = L.tw;
    a.vt = L.vt;
    a.out = L.p;
    a.sc = L.sc;
    launch((slab_inv_kernel<T, T, N, CPB, DST_P>), dim3(nslab),
           dim3(kSlabThreads<T, N>), 0, s, a);
  }
  if (mask & kPassFinal) {
    SlabInvArgs<T, double> a{};
    a.cs = (int64_t)N * N * N;
    a.spec = L.spec;
    a.tw = L.tw;
    a.vt = L.vt;
    a.out = L.F;
    launch((slab_inv_kernel<T, double, N, CPB, DST_ADDF>), dim3(nslab),
           dim3(kSlabThreads<T, N>), 0, s, a);
  }
  if (mask & kPassA) {
    SlabFwdArgs<T> a{};
    a.cs = (int64_t)N * N * N;
    a.spec = L.spec;
    a.tw = L.tw;
    a.sc = L.sc;
    if (L.fused) {
      a.field = L.p;
      a.K = L.K;
      a.kfull = L.kfull;
      a.pkp_out = L.pkp;
      launch((slab_fwd_kernel<T, N, CPB, SRC_KROW>), dim3(nslab),
             dim3(kSlabThreads<T, N>), 0, s, a);
    } else {
      a.field = L.y;
      if (L.prr) {
        a.pkp = L.pkp;
        a.pkp_count = L.pkp_count;
        a.parity = L.parity;
        a.scw = L.sc;
      }
      launch((slab_fwd_kernel<T, N, CPB, SRC_FIELD>), dim3(nslab),
             dim3(kSlabThreads<T, N>), 0, s, a);
    }
  }
  if (mask & kPassRes) {
    PencilFwdArgs<T, T> a{};
    a.spec = L.spec;
    a.tw = L.tw;
    a.vt = L.vt;
    a.rho = L.rho;
    a.invN3 = 1.0 / (double(N) * N * N);
    a.prec = L.prec;
    a.prr = L.prr_out;
    a.prz = L.prz_out;
    a.sc = L.sc;
    a.scw = L.sc;
    a.parity = L.parity;
    if (L.fused && L.prr) {
      a.pkp = L.pkp;
      a.pkp_count = 9 * N;
    }
    launch((pencil_fwd_kernel<T, T, N, TT, false>), dim3(npen),
           dim3(kPencilThreads<N, TT>), 0, s, a);
  }
}

// the FP64 residual of the field P: its norm partials and the start of the
// CG run
template <typename TR, int N>
void launch_residual_n(const ResidualLaunch<TR>& L, hipStream_t s) {
  constexpr int TT = kTile<N>;
  SlabFwdArgs<double> fa{};
  fa.cs = (int64_t)N * N * N;
  fa.field = L.P;
  fa.spec = L.spec;
  fa.tw = L.tw;
  fa.psum = L.psum;
  fa.psq = L.psq;
  launch((slab_fwd_kernel<double, N, 1, SRC_FIELD>), dim3(9 * N),
         dim3(kSlabThreads<double, N>), 0, s, fa);
  PencilFwdArgs<double, TR> a{};
  a.spec = L.spec;
  a.tw = L.tw;
  a.vt = L.vt;
  a.rho = L.rho;
  a.invN3 = 1.0 / (double(N) * N * N);
  a.prec = L.prec;
  a.prr = L.part;
  a.prz = L.part + residual_blocks(N);
  a.pres = L.part + 2 * residual_blocks(N);
  launch((pencil_fwd_kernel<double, TR, N, TT, true>), dim3(residual_blocks(N)),
         dim3(kPencilThreads<N, TT>), 0, s, a);
}

#define RVE_GRID_SIZES(X) X(16) X(24) X(32) X(40) X(48) X(64) X(96) X(128)

template <typename TR>
void launch_residual(int n, const ResidualLaunch<TR>& L, hipStream_t s) {
  switch (n) {
#define RVE_CASE(NN) case NN: return launch_residual_n<TR, NN>(L, s);
    RVE_GRID_SIZES(RVE_CASE)
#undef RVE_CASE
  }
  throw Error(-1, "unsupported grid size for the FFT passes");
}

template <typename T, int N>
void launch_cg_n(const CgLaunch<T>& L, int mask, hipStream_t s) {
  const int cpb = L.cpb, tt = L.tt;
  if (cpb == 3) {
    if constexpr (cpb3_fits<T, N>()) {
      if constexpr (pencil_fits<T, N, 16>())
        if (tt == 16) return launch_cg_sched<T, N, 3, 16>(L, mask, s);
      if (tt == 8) return launch_cg_sched<T, N, 3, 8>(L, mask, s);
      if (tt == 4) return launch_cg_sched<T, N, 3, 4>(L, mask, s);
    }
  } else if (cpb == 1) {
    if constexpr (pencil_fits<T, N, 16>())
      if (tt == 16) return launch_cg_sched<T, N, 1, 16>(L, mask, s);
    if (tt == 8) return launch_cg_sched<T, N, 1, 8>(L, mask, s);
    if (tt == 4) return launch_cg_sched<T, N, 1, 4>(L, mask, s);
  }
  throw Error(-1, "unsupported FFT schedule");
}

template <typename T>
void launch_cg(int n, const CgLaunch<T>& L, int mask, hipStream_t s) {
  switch (n) {
#define RVE_CASE(NN) case NN: return launch_cg_n<T, NN>(L, mask, s);
    RVE_GRID_SIZES(RVE_CASE)
#undef RVE_CASE
  }
  throw Error(-1, "unsupported grid size for the FFT passes");
}

template <typename T>
void launch_G(int n, const SpectralLaunch<T>& L, hipStream_t s) {
  switch (n) {
    case 16: launch_G_n<T, 16>(L, s); break;
    case 24: launch_G_n<T, 24>(L, s); break;
    case 32: launch_G_n<T, 32>(L, s); break;
    case 40: launch_G_n<T, 40>(L, s); break;
    case 48: launch_G_n<T, 48>(L, s); break;
    case 64: launch_G_n<T, 64>(L, s); break;
    case 96: launch_G_n<T, 96>(L, s); break;
    case 128: launch_G_n<T, 128>(L, s); break;
    default: throw Error(-1, "unsupported grid size for the FFT passes");
  }
}

int slab_blocks(int n, int cpb) { return n * (9 / cpb); }

int residual_blocks(int n) { return cg_pencil_blocks(n, cg_tile(n)); }

// kz columns per CG pencil block: four fill the chip better up to 48^3 (48^3
// FP32: direction and residual pass 5.9 + 6.3 us against 6.8 + 6.7 with
// eight), from 64^3 on the 64-byte segments of eight are faster (6.1 + 6.5
// against 6.8 + 7.0 us; 128^3: 31.7 + 29.3 against 36.7 + 31.8); sixteen
// lose everywhere (8.4 + 8.4; 35.8 + 40.1)
int cg_tile(int n) { return n < 64 ? 4 : 8; }

int cg_pencil_blocks(int n, int tt) { return n * ((n / 2 + tt - 1) / tt); }

bool schedule_valid(int n, bool fp64, int cpb, int tt) {
  if (tt != 4 && tt != 8 && tt != 16) return false;
  if (cpb != 1 && cpb != 3) return false;
  auto fits = [&](auto tag) -> bool {
    using T = decltype(tag);
    switch (n) {
#define RVE_FITS(NN)                                                        \
  case NN:                                                                  \
    return (cpb == 1 || cpb3_fits<T, NN>()) &&                              \
           (tt != 16 || pencil_fits<T, NN, 16>());
      RVE_FITS(16) RVE_FITS(24) RVE_FITS(32) RVE_FITS(40) RVE_FITS(48)
      RVE_FITS(64) RVE_FITS(96) RVE_FITS(128)
#undef RVE_FITS
    }
    return false;
  };
  return fp64 ? fits(double{}) : fits(float{});
}

bool batch_supported(int n) {
  switch (n) {
#define RVE_CASE(NN) case NN:
    RVE_BATCH_SIZES(RVE_CASE)
#undef RVE_CASE
    return true;
  }
  return false;
}

template <typename T>
void batch_lds(int n, int cpb, int tt, size_t& slab, size_t& pencil) {
  if (!batch_supported(n)) throw Error(-1, "grid edge not supported in a batch");
  if (!schedule_valid(n, sizeof(T) == 8, cpb, tt))
    throw Error(-1, "no such FFT schedule for this grid edge and precision");
  // the layouts of slab_fwd_item / slab_inv_item and the CG pencils
  const size_t plane = (size_t)(n / 2) * (n + 1);
  slab = (cpb * plane + n) * sizeof(cplx<T>) + kBlock * sizeof(double);
  pencil = (6 * ((size_t)n * (tt + 1) + tt) + n) * sizeof(cplx<T>) +
           kBlock / 64 * sizeof(double);
}

// f(integral_constant of the slab schedules present)
template <typename F>
void with_cpbs(int cpbs, F&& f) {
  if (cpbs == 1) f(std::integral_constant<int, 1>{});
  else if (cpbs == 2) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, 3>{});
}

template <typename T>
void launch_G_batch(const BatchSpec<T>& b, double* out, const BatchGrid& g,
                    hipStream_t s) {
  with_cpbs(b.cpbs, [&](auto cp) {
    constexpr int C = decltype(cp)::value;
    hipLaunchKernelGGL((slab_fwd_batch_kernel<T, false, C>), dim3(g.A),
                       dim3(kBlock), g.ldsA, s, b);
    hipLaunchKernelGGL((pencil_batch_kernel<T>), dim3(3 * g.B), dim3(kBlock),
                       g.ldsB, s, b);
    hipLaunchKernelGGL((slab_inv_batch_kernel<T, double, DST_NORM, C>),
                       dim3(g.A), dim3(kBlock), g.ldsA, s, b, out);
  });
}

template <typename TR>
void launch_residual_batch(const BatchSpec<double>& b, cplx<TR>* rho,
                           const BatchGrid& g, hipStream_t s) {
  with_cpbs(b.cpbs, [&](auto cp) {
    constexpr int C = decltype(cp)::value;
    hipLaunchKernelGGL((slab_fwd_batch_kernel<double, false, C>), dim3(g.A),
                       dim3(kBlock), g.ldsA, s, b);
  });
  hipLaunchKernelGGL((pencil_fwd_batch_kernel<double, TR, true>), dim3(g.B),
                     dim3(kBlock), g.ldsB, s, b, rho);
}

template <typename T>
void launch_cg_batch(const BatchSpec<T>& b, const BatchGrid& g, hipStream_t s) {
  with_cpbs(b.cpbs, [&](auto cp) {
    constexpr int C = decltype(cp)::value;
    hipLaunchKernelGGL((pencil_inv_batch_kernel<T, false>), dim3(g.B),
                       dim3(kBlock), g.ldsB, s, b);
    hipLaunchKernelGGL((slab_inv_batch_kernel<T, T, DST_P, C>), dim3(g.A),
                       dim3(kBlock), g.ldsA, s, b, b.p);
    if (g.V)   // the tuner's timings leave out what no schedule changes
      hipLaunchKernelGGL((kp_batch_kernel<T>), dim3(g.V), dim3(kBlock), 0, s, b);
    hipLaunchKernelGGL((slab_fwd_batch_kernel<T, true, C>), dim3(g.A),
                       dim3(kBlock), g.ldsA, s, b);
    hipLaunchKernelGGL((pencil_fwd_batch_kernel<T, T, false>), dim3(g.B),
                       dim3(kBlock), g.ldsB, s, b, b.rho);
  });
}

template <typename T>
void launch_cg_final_batch(const BatchSpec<T>& b, double* F, const BatchGrid& g,
                           hipStream_t s) {
  with_cpbs(b.cpbs, [&](auto cp) {
    constexpr int C = decltype(cp)::value;
    hipLaunchKernelGGL((pencil_inv_batch_kernel<T, true>), dim3(g.B),
                       dim3(kBlock), g.ldsB, s, b);
    hipLaunchKernelGGL((slab_inv_batch_kernel<T, double, DST_ADDF, C>),
                       dim3(g.A), dim3(kBlock), g.ldsA, s, b, F);
  });
}

// Dynamic LDS above the default 64 KiB must be allowed per kernel before
// the first launch.
template <typename T>
void batch_allow_lds(size_t slab, size_t pencil) {
  auto allow = [](const void* f, size_t bytes) {
    RVE_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)bytes));
  };
  for (int cpbs = 1; cpbs <= 3; ++cpbs)
    with_cpbs(cpbs, [&](auto cp) {
      constexpr int C = decltype(cp)::value;
      allow((const void*)&slab_fwd_batch_kernel<T, false, C>, slab);
      allow((const void*)&slab_fwd_batch_kernel<T, true, C>, slab);
      allow((const void*)&slab_inv_batch_kernel<T, double, DST_NORM, C>, slab);
      allow((const void*)&slab_inv_batch_kernel<T, double, DST_ADDF, C>, slab);
      allow((const void*)&slab_inv_batch_kernel<T, T, DST_P, C>, slab);
    });
  allow((const void*)&pencil_batch_kernel<T>, pencil);
  allow((const void*)&pencil_fwd_batch_kernel<T, T, false>, pencil);
  allow((const void*)&pencil_inv_batch_kernel<T, false>, pencil);
  allow((const void*)&pencil_inv_batch_kernel<T, true>, pencil);
  if constexpr (sizeof(T) == 8) {
    allow((const void*)&pencil_fwd_batch_kernel<double, float, true>, pencil);
    allow((const void*)&pencil_fwd_batch_kernel<double, double, true>, pencil);
  }
}

template void batch_allow_lds<float>(size_t, size_t);
template void batch_allow_lds<double>(size_t, size_t);
template void launch_G_batch<float>(const BatchSpec<float>&, double*,
                                    const BatchGrid&, hipStream_t);
template void launch_G_batch<double>(const BatchSpec<double>&, double*,
                                     const BatchGrid&, hipStream_t);
template void launch_residual_batch<float>(const BatchSpec<double>&,
                                           cplx<float>*, const BatchGrid&,
                                           hipStream_t);
template void launch_residual_batch<double>(const BatchSpec<double>&,
                                            cplx<double>*, const BatchGrid&,
                                            hipStream_t);
template void launch_cg_batch<float>(const BatchSpec<float>&, const BatchGrid&,
                                     hipStream_t);
template void launch_cg_batch<double>(const BatchSpec<double>&,
                                      const BatchGrid&, hipStream_t);
template void launch_cg_final_batch<float>(const BatchSpec<float>&, double*,
                                           const BatchGrid&, hipStream_t);
template void launch_cg_final_batch<double>(const BatchSpec<double>&, double*,
                                            const BatchGrid&, hipStream_t);
template void batch_lds<float>(int, int, int, size_t&, size_t&);
template void batch_lds<double>(int, int, int, size_t&, size_t&);
template void launch_cg<float>(int, const CgLaunch<float>&, int, hipStream_t);
template void launch_cg<double>(int, const CgLaunch<double>&, int, hipStream_t);
template void launch_residual<float>(int, const ResidualLaunch<float>&, hipStream_t);
template void launch_residual<double>(int, const ResidualLaunch<double>&, hipStream_t);
template void launch_G<float>(int, const SpectralLaunch<float>&, hipStream_t);
template void launch_G<double>(int, const SpectralLaunch<double>&, hipStream_t);

}  // namespace rve
