// Warm-start network kernels: 3x3x3 circular convolutions as implicit GEMMs
// on the bf16 matrix cores (v_mfma_f32_16x16x16_bf16), FP32 accumulation.
//
// Layouts (all device memory):
//   activations  bf16 [N][C] channels-last (C a multiple of 16), voxel
//                v = (x*n + y)*n + z, periodic neighbours v + d_t;
//   tap t = (dx+1)*9 + (dy+1)*3 + (dz+1);
//   master weights FP32 per layer: W[27][cin][cout] then b[cout];
//   MFMA B fragments bf16 [27][CIN/16][COUT/16][64 lanes][4]: lane l of
//   fragment (t, kc, nt) holds W[t][16 kc + 4 (l/16) + i][16 nt + l%16].
// The convolutions take the weight fragment as the A operand: one wave
// computes 16 consecutive voxels along z times all output channels, lane l
// feeding voxel l%16 (4 consecutive input channels) and receiving four
// consecutive output channels 4 (l/16) + i of that voxel.
#include "nn.hpp"
#include "kernels.hpp"

namespace rve {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// four floats of a caller's array, aligned as floats are
typedef f32x4 f32x4a __attribute__((aligned(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) {
  return __uint_as_float(((uint32_t)h) << 16);
}

__device__ __forceinline__ int wrap(int i, int n) {
  return i < 0 ? i + n : (i >= n ? i - n : i);
}
// place of W[t][ci][co] in the fragments of a CIN -> COUT convolution
__device__ __forceinline__ int frag_index(int t, int ci, int co, int CIN, int COUT) {
  const int f = (t * (CIN / 16) + ci / 16) * (COUT / 16) + co / 16;
  return f * 256 + ((ci % 16) / 4 * 16 + co % 16) * 4 + ci % 4;
}

// ---------------------------------------------------------------- staging
// The lines yb - 1 .. yb + nl - 2 (periodic, all z) of one x plane go from
// global memory straight to LDS (no registers in between, so all of a
// wave's loads are in flight at once), 16 bytes = 8 channels per lane.  A
// load writes the LDS of a wave contiguously, so instead of padded rows the
// 16-byte pieces of a voxel are permuted by swz<C>(z), on the global side of
// the load: with it neither the 16 voxels x 16 bytes that half a wave reads
// for a convolution nor the 8 voxels x 32 bytes of a transposed read share
// a bank.
template <int C>
__device__ __forceinline__ int swz(int z) {
  return C == 32 ? (((z >> 1) & 2) | ((z >> 3) & 1)) : ((z >> 3) & 1);
}

typedef __attribute__((address_space(1))) const void gvoid;
typedef __attribute__((address_space(3))) void lvoid;

// 16 bytes per active lane from src (per lane) to dst + 16 lane (dst the
// same in all lanes)
__device__ __forceinline__ void load_lds16(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds((gvoid*)src, (lvoid*)dst, 16, 0, 0);
}
// the block's loads into LDS have landed
__device__ __forceinline__ void lds_arrived() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// `count` 16-byte pieces of src, in order (wv: the wave's index, uniform)
template <int THREADS>
__device__ __forceinline__ void stage_flat(const uint16_t* src, uint16_t* dst,
                                           int count, int wv, int lane) {
  for (int i0 = 64 * wv; i0 < count; i0 += THREADS)
    if (i0 + lane < count) load_lds16(src + 8 * (i0 + lane), dst + 8 * i0);
}

// nl lines from yb - 1 of plane xp, permuted; inv_n = ceil(2^22 / n) (exact
// quotients: a staged voxel's index is below 2^12 and n at most 2^9)
template <int C, int THREADS>
__device__ __forceinline__ void stage_lines(const uint16_t* __restrict__ X,
                                            uint16_t* dst, int xp, int yb,
                                            int nl, int n, unsigned inv_n,
                                            int wv, int lane) {
  constexpr int CH = C / 8;
  const int count = nl * n * CH;
  for (int i0 = 64 * wv; i0 < count; i0 += THREADS) {
    const int i = i0 + lane;
    if (i >= count) continue;
    const int vz = i / CH, pos = i % CH;
    const int j = (int)(((unsigned)vz * inv_n) >> 22), z = vz - j * n;
    const int yg = wrap(yb - 1 + j, n);
    load_lds16(X + (((int64_t)xp * n + yg) * n + z) * C + 8 * (pos ^ swz<C>(z)),
               dst + 8 * i0);
  }
}
static unsigned inv_edge(int n) { return ((1u << 22) + n - 1) / n; }

// lines a block of vox consecutive voxels stages: those it touches (it
// starts at a multiple of gcd(vox, n)) and one on either side
static int conv_lines(int n, int vox) {
  int g = vox, r = n;
  while (r) {
    const int t = g % r;
    g = r;
    r = t;
  }
  return (n - g + vox + n - 1) / n + 2;
}

// blocks of neighbouring voxels run on one XCD, whose L2 then holds the
// lines and planes that they share
__device__ __forceinline__ int xcd_block() {
  const int g = (int)gridDim.x, b = (int)blockIdx.x;
  return g % 8 ? b : (b % 8) * (g / 8) + b / 8;
}

// ------------------------------------------------------------- convolution
// EPI: 0 bias + ReLU -> bf16; 1 bias, linear -> f32; 2 no bias, multiply by
// the mask (mask_act > 0) -> bf16 (backward through the previous ReLU)
//
// A block of four waves computes 64 TPW consecutive voxels (TPW 16-voxel
// tiles per wave; with n % 16 == 0 a block never leaves its x plane).  For
// each dx slice of the stencil it stages the fragments of the nine taps and
// the input lines that it reads, and the waves read both operands of every
// MFMA from LDS.  Staging through registers, one dependent load at a time,
// bound the kernel before (32 -> 32 channels at 64^3: 51 us, now 28 us = 515
// TFLOP/s; at 32^3 23, now 8 us); now the MFMAs (11.5 us at the rate of a
// 16x16x16 product), the waits at the slices' ends and a last round of
// blocks that fills a third of the chip do.
template <int CIN, int COUT>
constexpr int conv_slice() { return 9 * (CIN / 16) * (COUT / 16) * 64 * 4; }
template <int CIN, int COUT>
size_t conv_lds_bytes(int n, int vox) {
  return ((size_t)conv_slice<CIN, COUT>() +
          (size_t)conv_lines(n, vox) * n * CIN) * sizeof(uint16_t);
}

template <int CIN, int COUT, int EPI, int TPW>
__global__ __launch_bounds__(256) void conv_mfma_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ Wf,
    const float* __restrict__ bias, uint16_t* __restrict__ Yb,
    float* __restrict__ Yf, const uint16_t* __restrict__ mask_act, int n,
    unsigned inv_n, int nl, int cout_real) {
  constexpr int KC = CIN / 16, NT = COUT / 16;
  constexpr int SLICE = conv_slice<CIN, COUT>();  // bf16 of one dx slice
  extern __shared__ __align__(16) uint16_t smem_conv[];
  uint16_t* wl = smem_conv;
  uint16_t* al = smem_conv + SLICE;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int row = lane & 15, grp = lane >> 4;
  // n^3 is a multiple of the block's voxels and below 2^31
  const int vb = xcd_block() * (64 * TPW);
  const int xb = vb / (n * n), yb = (vb / n) % n;
  // byte offsets into the staged lines: of the tile's line, and per dz of the
  // lane's voxel and of its four channels' piece
  int line[TPW], zo[TPW][3];
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    const int v0 = vb + (wv * TPW + u) * 16;
    line[u] = ((v0 / n) % n - yb + 1) * n * CIN * 2;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int zz = wrap(v0 % n + row + d - 1, n);
      zo[u][d] = zz * CIN * 2 + (((grp >> 1) ^ swz<CIN>(zz)) * 16) + (grp & 1) * 8;
    }
  }
  f32x4 acc[TPW][NT];
#pragma unroll
  for (int u = 0; u < TPW; ++u)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[u][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int sl = 0; sl < 3; ++sl) {
    if (sl) __syncthreads();
    stage_lines<CIN, 256>(X, al, wrap(xb + sl - 1, n), yb, nl, n, inv_n, wv, lane);
    stage_flat<256>(Wf + (size_t)sl * SLICE, wl, SLICE / 8, wv, lane);
    lds_arrived();
#pragma unroll
    for (int tl = 0; tl < 9; ++tl) {
      const int dy = tl / 3 - 1, d = tl % 3;
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        bf16x4 b[NT], a[TPW];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          b[nt] = *reinterpret_cast<const bf16x4*>(
              wl + (((tl * KC + kc) * NT + nt) * 64 + lane) * 4);
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
          // pieces 2 kc, 2 kc + 1: the permutation moves both bits of a
          // 32-channel voxel's index, one of the others'
          const int zk = CIN == 32 ? zo[u][d] ^ (32 * kc) : zo[u][d] + 32 * kc;
          a[u] = *reinterpret_cast<const bf16x4*>(
              reinterpret_cast<const char*>(al) + line[u] + dy * n * CIN * 2 + zk);
        }
#pragma unroll
        for (int u = 0; u < TPW; ++u)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[u][nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                b[nt], a[u], acc[u][nt], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int co = nt * 16 + 4 * grp;
    // the bias has only the real output channels
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (EPI != 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (co + i < cout_real) bv[i] = bias[co + i];
    }
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int64_t o = (int64_t)(vb + (wv * TPW + u) * 16 + row) * COUT + co;
      float val[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) val[i] = acc[u][nt][i] + bv[i];
      if constexpr (EPI == 1) {
        *reinterpret_cast<f32x4a*>(Yf + o) = (f32x4){val[0], val[1], val[2], val[3]};
      } else {
        ushort4 m;
        if constexpr (EPI == 2) m = *reinterpret_cast<const ushort4*>(mask_act + o);
        const uint16_t mk[4] = {m.x, m.y, m.z, m.w};
        uint16_t r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          r[i] = f2bf((EPI == 0 ? val[i] : bf2f(mk[i])) > 0.f ? val[i] : 0.f);
        *reinterpret_cast<ushort4*>(Yb + o) = make_ushort4(r[0], r[1], r[2], r[3]);
      }
    }
  }
}

// --------------------------------------------------------- weight gradient
// dW[t][i][o] = sum_v X[v + d_t][i] dZ[v][o] and db[o] = sum_v dZ[v][o]:
// partials of a chunk of voxels, part[chunk][27][CIN][COUT] and
// bpart[chunk][COUT], summed in fixed order by update_kernel.
//
// An MFMA takes M = i, N = o, K = 32 voxels.  A block handles one dx (its
// blockIdx.y) of `groups` groups of 256 consecutive voxels, wave w the three
// taps of dy = w - 1; the staged lines of X and the group's dZ are
// channels-last, and the transposed LDS read (ds_read_b64_tr_b16: the lanes
// of a group of 16 read 4 voxels x 16 channels and each receives one
// channel of the four voxels) yields both operands, a neighbour being an
// address.  The bias gradient is one more product, with A = 1, of the wave at
// dx = dy = 0.  Before, each operand was gathered from global memory one bf16
// at a time, once per tap (32 -> 32
// channels at 32^3: 88 us; now 12 us, bound by the staging and by writing
// 27 x 32 x 32 partials per chunk).
constexpr int kGroupVox = 256;
constexpr int kWgThreads = 192;
// An MFMA accumulator sums up to kRun groups, 64 products of 32 voxels.  A
// block of more (96^3, 128^3) adds it to a second sum every kFlush groups and
// starts again, at most 16 times (kMaxGroups), so that a term passes 48
// roundings before the FP64 sum over the chunks; in one run it would pass 512
// at 128^3 (a training step there 3.23 ms, with the second sum 3.37).
constexpr int kRun = 8;
constexpr int kFlush = 4;
constexpr int kMaxGroups = 64;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

__device__ __forceinline__ bf16x4 read_tr(const uint16_t* base, int byte) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (lds_bf16x4*)(reinterpret_cast<const char*>(base) + byte));
}
__device__ __forceinline__ bf16x8 join(bf16x4 a, bf16x4 b) {
  typedef short s8 __attribute__((ext_vector_type(8)));
  const s8 r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, r);
}

template <int CIN, int COUT, bool LONG>
__global__ __launch_bounds__(kWgThreads) void conv_wgrad_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ dZ,
    float* __restrict__ part, float* __restrict__ bpart, int n, unsigned inv_n,
    int nl, int groups) {
  constexpr int KC = CIN / 16, NT = COUT / 16;
  extern __shared__ __align__(16) uint16_t smem_conv[];
  uint16_t* zl = smem_conv;                       // dZ [256][COUT]
  uint16_t* al = smem_conv + kGroupVox * COUT;    // X lines
  const int lane = threadIdx.x & 63;
  const int dy = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int row = lane & 15, grp = lane >> 4;
  const int dx = blockIdx.y;
  const int total = (int)((int64_t)n * n * n / kGroupVox);
  const int g0 = (int)blockIdx.x * groups;
  const int g1 = g0 + groups < total ? g0 + groups : total;
  const bool bias = bpart && dx == 1 && dy == 1;
  const int tv = 4 * grp + (row >> 2);            // voxel of the tile read
  const int q = (row & 3) >> 1, half = (row & 1) * 8;
  // dZ offsets: a tile starts at a multiple of 16 voxels
  const int zb = tv * COUT * 2 + (q ^ swz<COUT>(tv)) * 16 + half;
  f32x4 acc[3][KC][NT], accb[NT];
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    accb[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int a = 0; a < KC; ++a) acc[d][a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  // LONG: what the accumulators are added to every kFlush groups
  f32x4 sum[LONG ? 3 : 1][LONG ? KC : 1][LONG ? NT : 1], sumb[LONG ? NT : 1];
  if constexpr (LONG) {
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      sumb[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int a = 0; a < KC; ++a) sum[d][a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
  }
  const bf16x4 one4 = {0x3F80, 0x3F80, 0x3F80, 0x3F80};
  const bf16x8 ones = join(one4, one4);
  for (int g = g0; g < g1; ++g) {
    const int vb = g * kGroupVox;
    const int xb = vb / (n * n), yb = (vb / n) % n;
    if (g > g0) __syncthreads();
    stage_lines<CIN, kWgThreads>(X, al, wrap(xb + dx - 1, n), yb, nl, n, inv_n,
                                 dy, lane);
    {
      constexpr int CH = COUT / 8;
      for (int i0 = 64 * dy; i0 < kGroupVox * CH; i0 += kWgThreads) {
        const int v = (i0 + lane) / CH, pos = (i0 + lane) % CH;
        load_lds16(dZ + ((int64_t)vb + v) * COUT + 8 * (pos ^ swz<COUT>(v)),
                   zl + 8 * i0);
      }
    }
    lds_arrived();
    for (int u = 0; u < kGroupVox / 16; u += 2) {
      int line[2], z0[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int v0 = vb + 16 * (u + h);
        line[h] = ((v0 / n) % n - yb + dy) * n * CIN * 2;
        z0[h] = v0 % n + tv;
      }
      bf16x8 b[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int o = u * 16 * COUT * 2 +
                      (COUT == 32 ? zb ^ (32 * nt) : zb + 32 * nt);
        b[nt] = join(read_tr(zl, o), read_tr(zl, o + 16 * COUT * 2));
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        int o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int zz = wrap(z0[h] + d - 1, n);
          o[h] = zz * CIN * 2 + (q ^ swz<CIN>(zz)) * 16 + half;
        }
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
          const int k0 = CIN == 32 ? o[0] ^ (32 * kc) : o[0] + 32 * kc;
          const int k1 = CIN == 32 ? o[1] ^ (32 * kc) : o[1] + 32 * kc;
          const bf16x8 a = join(read_tr(al, line[0] + k0), read_tr(al, line[1] + k1));
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[d][kc][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                a, b[nt], acc[d][kc][nt], 0, 0, 0);
        }
      }
      if (bias)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          accb[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, b[nt], accb[nt],
                                                             0, 0, 0);
    }
    if constexpr (LONG)
      if ((g - g0) % kFlush == kFlush - 1 || g == g1 - 1) {
        auto flush = [](f32x4& t, f32x4& x) {
          t += x;
          x = (f32x4){0.f, 0.f, 0.f, 0.f};
        };
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if (bias) flush(sumb[nt], accb[nt]);
#pragma unroll
          for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) flush(sum[d][kc][nt], acc[d][kc][nt]);
        }
      }
  }
  // D[4 grp + i][row] = dW[16 kc + 4 grp + i][16 nt + row]
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    float* out = part + ((size_t)blockIdx.x * 27 + dx * 9 + dy * 3 + d) * CIN * COUT;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          out[(16 * kc + 4 * grp + i) * COUT + 16 * nt + row] =
              LONG ? sum[LONG ? d : 0][LONG ? kc : 0][LONG ? nt : 0][i]
                   : acc[d][kc][nt][i];
  }
  if (bias && grp == 0)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      bpart[(size_t)blockIdx.x * COUT + 16 * nt + row] =
          LONG ? sumb[LONG ? nt : 0][0] : accb[nt][0];
}

// loss L = mean over N*CREAL of (Y - T)^2 and dY = 2 (Y - T)/count, written
// as bf16 (input of the backward convolutions); the block's sums of the loss
// and, from the unrounded dY, of the last layer's bias gradient.  A thread
// takes four of a voxel's kOut channels, always the same ones.
__global__ __launch_bounds__(256) void mse_kernel(
    const float* __restrict__ Y, const float* __restrict__ T, int creal,
    int64_t N, uint16_t* __restrict__ dYb, float* __restrict__ bpart,
    double* __restrict__ part) {
  __shared__ double red[256];
  __shared__ double redb[4][kOut];
  static_assert(kOut == 16, "four threads per voxel");
  const double inv = 1.0 / ((double)N * creal);
  const int c0 = 4 * (threadIdx.x & 3);
  double s = 0.0, sb[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < N * (kOut / 4);
       i += (int64_t)gridDim.x * 256) {
    const f32x4 y = reinterpret_cast<const f32x4*>(Y)[i];
    const f32x4 t = reinterpret_cast<const f32x4a*>(T)[i];
    uint16_t r[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float g = 0.f;
      if (c0 + c < creal) {
        const float d = y[c] - t[c];
        s += (double)d * d;
        g = (float)(2.0 * d * inv);
      }
      sb[c] += g;
      r[c] = f2bf(g);
    }
    reinterpret_cast<ushort4*>(dYb)[i] = make_ushort4(r[0], r[1], r[2], r[3]);
  }
  // the 16 lanes of a wave with the same channels
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    for (int m = 4; m < 64; m <<= 1) sb[c] += __shfl_xor(sb[c], m);
    if ((threadIdx.x & 63) < 4) redb[threadIdx.x >> 6][c0 + c] = sb[c];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0] * inv;
  if (threadIdx.x < kOut)
    bpart[blockIdx.x * kOut + threadIdx.x] =
        (float)(redb[0][threadIdx.x] + redb[1][threadIdx.x] +
                redb[2][threadIdx.x] + redb[3][threadIdx.x]);
}

// One launch after the backward pass: per master parameter the sum of its
// partials in fixed order, the gradient, the Adam step (Kingma & Ba) and the
// weight's places in the forward and backward fragments (11 us for the 128
// partials of 32^3; before, eight sums, four copies into place, Adam and four
// repacks, 22 launches and 150 us).  A block takes 64
// parameters, its four waves a quarter of the partials each.
__global__ __launch_bounds__(256) void update_kernel(UpdateArgs a) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  const bool live = e < a.size;
  int k = 0;
  while (k < 3 && e >= a.layer[k + 1].off) ++k;
  const UpdateLayer& L = a.layer[k];
  const int r = (int)(e - L.off), nw = 27 * L.cin * L.cout;
  const int o = r < nw ? r % L.cout : r - nw;
  const int i = r < nw ? (r / L.cout) % L.cin : 0;
  const int t = r < nw ? r / (L.cout * L.cin) : 0;
  double s = 0.0;
  if (live) {
    const float* p = r < nw ? L.part + ((size_t)t * L.CIN + i) * L.COUT + o
                            : L.bpart + o;
    const size_t stride = r < nw ? (size_t)27 * L.CIN * L.COUT : (size_t)L.COUT;
    const int np = r < nw ? L.nparts : L.nbparts;
    const int lo = np * wv / 4, hi = np * (wv + 1) / 4;
#pragma unroll 8
    for (int q = lo; q < hi; ++q) s += p[q * stride];
  }
  red[wv][lane] = s;
  __syncthreads();
  if (wv || !live) return;
  const float g = (float)(red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane]);
  a.g[e] = g;
  const float m = a.b1 * a.m[e] + (1.f - a.b1) * g;
  const float v = a.b2 * a.v[e] + (1.f - a.b2) * g * g;
  a.m[e] = m;
  a.v[e] = v;
  const float w = a.w[e] - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
  a.w[e] = w;
  if (r >= nw) return;
  const uint16_t h = f2bf(w);
  L.wf[frag_index(t, i, o, L.CIN, L.COUT)] = h;
  L.wb[frag_index(26 - t, o, i, L.COUT, L.CIN)] = h;
}

// master W[27][cin][cout] -> MFMA B fragments for the forward pass, and the
// flipped, transposed fragments of the backward-data pass
// (W'[26 - t][o][i] = W[t][i][o]); padded channels are zero
__global__ void pack_kernel(const float* __restrict__ W, int cin, int cout,
                            int CIN, int COUT, uint16_t* __restrict__ Wf,
                            uint16_t* __restrict__ Wb) {
  const int KC = CIN / 16, NT = COUT / 16;
  const int64_t total = (int64_t)27 * KC * NT * 64 * 4;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e % 4);
    const int lane = (int)((e / 4) % 64);
    const int64_t f = e / 256;
    const int nt = (int)(f % NT), kc = (int)((f / NT) % KC), t = (int)(f / (NT * KC));
    const int ci = 16 * kc + 4 * (lane / 16) + i, co = 16 * nt + lane % 16;
    const float val = (ci < cin && co < cout) ? W[((size_t)t * cin + ci) * cout + co] : 0.f;
    Wf[e] = f2bf(val);
  }
  // backward data: input channels = COUT, output channels = CIN
  const int KCb = COUT / 16, NTb = CIN / 16;
  const int64_t totb = (int64_t)27 * KCb * NTb * 64 * 4;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < totb;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e % 4);
    const int lane = (int)((e / 4) % 64);
    const int64_t f = e / 256;
    const int nt = (int)(f % NTb), kc = (int)((f / NTb) % KCb), t = (int)(f / (NTb * KCb));
    const int o = 16 * kc + 4 * (lane / 16) + i, ci = 16 * nt + lane % 16;
    const int ts = 26 - t;
    const float val = (ci < cin && o < cout) ? W[((size_t)ts * cin + ci) * cout + o] : 0.f;
    Wb[e] = f2bf(val);
  }
}

// ----------------------------------------------------------------- launchers
namespace {
// Up to this edge a wave computes one tile instead of four: the blocks of
// four tiles leave most of the chip idle (a forward pass of four layers, one
// tile / four tiles: 37 / 57 us at 16^3, 43 / 60 us at 32^3), while from 48^3
// on there are enough of them and a staged weight serves four tiles (86 / 73
// us at 48^3, 154 / 119 us at 64^3, 1500 / 820 us at 128^3).
constexpr int kConvSmall = 32;
// largest grid edge that is taken: the fragments and staged lines of 48
// channels take 144 KB of a CU's 160 there
constexpr int kConvMaxEdge = 304;

// dynamic LDS above 64 KiB is allowed per kernel before its launch
void allow_lds(const void* f, size_t lds) {
  if (lds > 64 * 1024)
    RVE_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds));
}

template <int CIN, int COUT, int EPI, int TPW>
void conv_t(const uint16_t* X, const uint16_t* Wf, const float* b, uint16_t* Yb,
            float* Yf, const uint16_t* mask, int n, int creal, hipStream_t s) {
  constexpr int vox = 64 * TPW;
  const size_t lds = conv_lds_bytes<CIN, COUT>(n, vox);
  allow_lds(reinterpret_cast<const void*>(&conv_mfma_kernel<CIN, COUT, EPI, TPW>), lds);
  const int64_t N = (int64_t)n * n * n;
  hipLaunchKernelGGL((conv_mfma_kernel<CIN, COUT, EPI, TPW>),
                     dim3((unsigned)(N / vox)), dim3(256), lds, s,
                     X, Wf, b, Yb, Yf, mask, n, inv_edge(n), conv_lines(n, vox),
                     creal);
}
}  // namespace

void nn_conv(int cin, int cout, int epi, const uint16_t* X, const uint16_t* Wf,
             const float* b, uint16_t* Yb, float* Yf, const uint16_t* mask,
             int n, int64_t N, int cout_real, hipStream_t s) {
  if (n % 16 || N != (int64_t)n * n * n)
    throw Error(-1, "convolution grid must be n^3 with n % 16 == 0");
  if (n > kConvMaxEdge) throw Error(-1, "convolution grid edge too large");
  const bool small = n <= kConvSmall;
#define RVE_CONV(CI, CO, E)                                              \
  if (cin == CI && cout == CO && epi == E) {                             \
    if (small) conv_t<CI, CO, E, 1>(X, Wf, b, Yb, Yf, mask, n, cout_real, s); \
    else conv_t<CI, CO, E, 4>(X, Wf, b, Yb, Yf, mask, n, cout_real, s);    \
    return;                                                              \
  }
  RVE_CONV(48, 32, 0)
  RVE_CONV(32, 32, 0)
  RVE_CONV(32, 16, 1)
  RVE_CONV(16, 32, 2)
  RVE_CONV(32, 32, 2)
#undef RVE_CONV
  throw Error(-1, "unsupported convolution shape");
}

// groups of 256 voxels per weight-gradient block (as few as leave
// kChunks chunks, at most kMaxGroups), and the chunks that makes
static int wgrad_groups(int64_t N) {
  const int64_t g = (N / kGroupVox + kChunks - 1) / kChunks;
  return (int)(g < kMaxGroups ? g : kMaxGroups);
}
int64_t nn_wgrad_max_chunks(int64_t N) {
  const int64_t all = N / kGroupVox, few = all < kChunks ? all : kChunks;
  const int64_t most = (all + kMaxGroups - 1) / kMaxGroups;
  return few > most ? few : most;
}
int nn_wgrad_chunks(int64_t N) {
  const int g = wgrad_groups(N);
  return (int)((N / kGroupVox + g - 1) / g);
}

void nn_wgrad(int cin, int cout, const uint16_t* X, const uint16_t* dZ,
              float* part, float* bpart, int n, int64_t N, hipStream_t s) {
  if (n % 16 || N != (int64_t)n * n * n)
    throw Error(-1, "convolution grid must be n^3 with n % 16 == 0");
  const int nl = conv_lines(n, kGroupVox);
  dim3 grid((unsigned)nn_wgrad_chunks(N), 3);
  auto run = [&](auto kernel) {
    const size_t lds = ((size_t)kGroupVox * cout + (size_t)nl * n * cin) * sizeof(uint16_t);
    allow_lds(reinterpret_cast<const void*>(kernel), lds);
    hipLaunchKernelGGL(kernel, grid, dim3(kWgThreads), lds, s, X, dZ, part, bpart,
                       n, inv_edge(n), nl, wgrad_groups(N));
  };
  const bool lng = wgrad_groups(N) > kRun;
  if (cin == 48 && cout == 32)
    lng ? run(&conv_wgrad_kernel<48, 32, true>) : run(&conv_wgrad_kernel<48, 32, false>);
  else if (cin == 32 && cout == 32)
    lng ? run(&conv_wgrad_kernel<32, 32, true>) : run(&conv_wgrad_kernel<32, 32, false>);
  else if (cin == 32 && cout == 16)
    lng ? run(&conv_wgrad_kernel<32, 16, true>) : run(&conv_wgrad_kernel<32, 16, false>);
  else throw Error(-1, "unsupported weight-gradient shape");
}

void nn_mse(const float* Y, const float* T, int creal, int64_t N, uint16_t* dYb,
            float* bpart, double* part, int nblk, hipStream_t s) {
  hipLaunchKernelGGL(mse_kernel, dim3(nblk), dim3(256), 0, s, Y, T, creal, N, dYb,
                     bpart, part);
}

void nn_update(const UpdateArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(update_kernel, dim3((unsigned)((a.size + 63) / 64)), dim3(256),
                     0, s, a);
}

void nn_pack(const float* W, int cin, int cout, int CIN, int COUT, uint16_t* Wf,
             uint16_t* Wb, hipStream_t s) {
  hipLaunchKernelGGL(pack_kernel, dim3(128), dim3(256), 0, s, W, cin, cout, CIN,
                     COUT, Wf, Wb);
}

// network input of one increment (channels, kFeat padded):
//   0-8   (Fbar_k - Fbar_{k-1}) / s_k                 (broadcast)
//   9-17  fluctuation increment of increment k-1 / s_{k-1}
//   18-26 100 (F_{k-1} - Fbar_{k-1})                   (current fluctuation)
//   27-35 orientation matrix of the voxel's grain (zero in particles)
//   36    particle flag
//   37    reversal indicator dFbar_k : dFbar_{k-1} / (s_k s_{k-1})
//   38    sum_a |dgamma_a| of increment k-1 / s_{k-1}
//   39    1
__global__ void features_kernel(FeatArgs a) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= a.N) return;
  const int64_t N = a.N;
  const double* tb = a.table + (int64_t)a.phase[v] * kTableStride;
  const bool part = tb[0] != 0.0;
  float f[kFeat];
#pragma unroll
  for (int c = 0; c < kFeat; ++c) f[c] = 0.f;
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    f[c] = (float)a.dfbar_n[c];
    f[9 + c] = (float)(a.dFt_prev[c * N + v] * a.inv_s_prev);
    f[18 + c] = (float)(100.0 * (a.Fprev[c * N + v] - a.fbar_prev[c]));
    f[27 + c] = part ? 0.f : (float)tb[kTabR + c];
  }
  f[36] = part ? 1.f : 0.f;
  f[37] = (float)a.reversal;
  double sg = 0.0;
#pragma unroll
  for (int al = 0; al < 12; ++al) sg += fabs(a.dg_prev[al * N + v]);
  f[38] = (float)(sg * a.inv_s_prev);
  f[39] = 1.f;
  uint16_t* out = a.X + v * kFeat;
#pragma unroll
  for (int c = 0; c < kFeat; ++c) out[c] = f2bf(f[c]);
}

void nn_features(const FeatArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(features_kernel, dim3((unsigned)((a.N + 255) / 256)),
                     dim3(256), 0, s, a);
}

// T[v][c] = dFt[c][v] / s for c < 9, zero padding up to kOut
__global__ void target_kernel(const double* __restrict__ dFt, double inv_s,
                              const double* __restrict__ dFt2, double coef,
                              float* __restrict__ T, int64_t N) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
#pragma unroll
  for (int c = 0; c < kOut; ++c)
    T[v * kOut + c] = (c < kOutReal) ? (float)(dFt[c * N + v] * inv_s -
                                               coef * dFt2[c * N + v])
                                     : 0.f;
}

void nn_target(const double* dFt, double inv_s, const double* dFt2,
               double coef, float* T, int64_t N, hipStream_t s) {
  hipLaunchKernelGGL(target_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256),
                     0, s, dFt, inv_s, dFt2, coef, T, N);
}

// out[c][v] = scale * Y[v][c], c < 9
__global__ void out_field_kernel(const float* __restrict__ Y, double scale,
                                 double* __restrict__ out, int64_t N) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
#pragma unroll
  for (int c = 0; c < kOutReal; ++c) out[c * N + v] = scale * (double)Y[v * kOut + c];
}

void nn_output_to_field(const float* Y, double scale, double* out, int64_t N,
                        hipStream_t s) {
  hipLaunchKernelGGL(out_field_kernel, dim3((unsigned)((N + 255) / 256)),
                     dim3(256), 0, s, Y, scale, out, N);
}

// fluctuation increment of a converged increment: F_k - F_{k-1} - dFbar
__global__ void fluct_kernel(const double* __restrict__ Fn,
                             const double* __restrict__ Fo, double d0,
                             double d1, double d2, double d3, double d4,
                             double d5, double d6, double d7, double d8,
                             double* __restrict__ out, int64_t N) {
  const double d[9] = {d0, d1, d2, d3, d4, d5, d6, d7, d8};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 9 * N;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = Fn[i] - Fo[i] - d[i / N];
}

void nn_fluct_increment(const double* Fnew, const double* Fold,
                        const double dFbar[9], double* out, int64_t N,
                        hipStream_t s) {
  hipLaunchKernelGGL(fluct_kernel, dim3(2048), dim3(256), 0, s, Fnew, Fold,
                     dFbar[0], dFbar[1], dFbar[2], dFbar[3], dFbar[4], dFbar[5],
                     dFbar[6], dFbar[7], dFbar[8], out, N);
}

__global__ void axpy_kernel(double* __restrict__ F, const double* __restrict__ d,
                            double a, int64_t n9) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n9;
       i += (int64_t)gridDim.x * blockDim.x)
    F[i] += a * d[i];
}

void nn_axpy_field(double* F, const double* d, double a, int64_t n9,
                   hipStream_t s) {
  hipLaunchKernelGGL(axpy_kernel, dim3(2048), dim3(256), 0, s, F, d, a, n9);
}

}  // namespace rve
