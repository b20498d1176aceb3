// Point constitutive update (Sec. 2.1, Eq. 2) and material tangent
// K = dP/dF (Eq. 13) in FP64: the return mapping runs four lanes per voxel
// (three slip systems per lane), the tangent one lane per voxel.
//
// Grains: FCC crystal plasticity with the power-law flow rule of Sec. 3.2,
// Eq. 22 (constant critical stress g, rate exponent n) and an
// Armstrong-Frederick back stress, integrated by backward Euler over dt at
// the committed state (Fp^-1_0, chi_0):
//   Fp^-1 = Fp^-1_0 (I - sum_a dg_a s_a (x) m_a),  Fe = F Fp^-1,
//   S = C : (Fe^T Fe - I)/2,  tau_a = s_a . S m_a,
//   chi_a = (chi_0a + c dg_a)/(1 + d |dg_a|),  x_a = (tau_a - chi_a)/g,
//   P = Fe S Fp^-T.
// The 12 slips solve R_a = asinh(dg_a/a) - asinh(|x_a|^n sign x_a) = 0
// (a = dt gdot0), which has the roots of dg_a = a |x_a|^n sign x_a but stays
// well scaled under large overstress.  Damped Newton with backtracking on
// |R|^2/2; a failed warm-started solve is retried from zero slips.  R is
// formed in FP64 with one logarithm per slip (flow_residual); the Jacobian,
// which only steers the iteration towards the root of R, in FP32.
//
// The 12x12 Jacobian is diag(D) + U W^T with low-rank factors (the resolved
// stresses depend on the slips only through the symmetric elastic strain,
// and not on its trace), so each Newton step costs one 5x5 solve and the
// tangent one 5x5 factorisation (Sherman-Morrison-Woodbury) instead of 12x12
// ones.
//
// Work order: crystal voxels first, then the particle voxels (an index list
// built with the microstructure), so that wavefronts iterating the local
// solve carry no particle lanes.
//
// Particles: isotropic St-Venant-Kirchhoff, P = F S, S = lam tr(E) I + 2 mu E.
#include "kernels.hpp"
#include "kp_apply.hpp"

namespace rve {

namespace {

constexpr int LOCAL_MAXIT = 60;
constexpr double LOCAL_RTOL = 1e-10;
constexpr double LOCAL_ATOL = 1e-18;
constexpr double LOCAL_RFLOOR = 1e-10;

// Hides an offset of zero from the optimizer so that table entries are
// re-read (from cache) at each use instead of being hoisted out of the local
// Newton loop into registers, which would exhaust the register file.  The
// pointer itself stays visible, so the loads remain global-memory loads
// (not flat ones).  The asm is empty: no instruction is emitted and no
// memory is accessed.
__device__ __forceinline__ const double* opaque(const double* p) {
  int64_t z = 0;
  asm volatile("" : "+v"(z));
  return p + z;
}

__device__ __forceinline__ double sgn(double x) {
  return (x > 0.0) ? 1.0 : ((x < 0.0) ? -1.0 : 0.0);
}

// b^ni by repeated squaring
__device__ __forceinline__ double ipow_n(double b, int ni) {
  if (ni == 20) {   // the workloads' exponent: five products
    const double b2 = b * b, b4 = b2 * b2, b8 = b4 * b4, b16 = b8 * b8;
    return b16 * b4;
  }
  double y = 1.0;
  for (int e = ni; e; e >>= 1) {   // uniform over the wavefront
    if (e & 1) y *= b;
    b *= b;
  }
  return y;
}

// asinh(|x|^n sign x) and its derivative d/dx = n y / (|x| sqrt(1 + y^2)),
// y = |x|^n, through s = min(y, 1/y) = exp(-|n ln|x||), for any exponent and
// any |x|:
//   y >= 1: asinh(y) = n ln|x| + log1p(q),                q = sqrt(1 + s^2)
//   y <  1: asinh(y) = log1p(s + s^2 / (1 + q)).
__device__ __forceinline__ void asinh_pow(double x, double n, double& val,
                                          double& der) {
  const double ax = fabs(x);
  const double e = n * log(ax);          // ln y (-inf at x = 0)
  const bool big = e > 0.0;
  const double s = exp(-fabs(e));        // 0 at x = 0
  const double q = sqrt(1.0 + s * s);
  const double L = log1p(big ? q : s + s * s / (1.0 + q));
  val = sgn(x) * ((big ? e : 0.0) + L);
  der = (ax > 0.0) ? n * (big ? 1.0 : s) / (ax * q) : 0.0;
}

__device__ __forceinline__ void mm3(const double* A, const double* B,
                                    double* C) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      C[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] +
                     A[3 * i + 2] * B[6 + j];
}

// d/dx asinh(|x|^n sign x) = n y / (|x| sqrt(1 + y^2)), y = |x|^n (FP64; y by
// products for an integer exponent while y^2 stays in range)
__device__ __forceinline__ double flow_slope(double x, const LawParams& lp) {
  const double ax = fabs(x);
  if (lp.nint > 0 && ax < lp.xmax) {
    const double y = ipow_n(ax, lp.nint);
    return (ax > 0.0) ? lp.nexp * (y / (ax * sqrt(fma(y, y, 1.0)))) : 0.0;
  }
  double val, der;
  asinh_pow(x, lp.nexp, val, der);
  return der;
}

__device__ __forceinline__ void load9(const double* __restrict__ p, int64_t v,
                                      int64_t N, double* o) {
#pragma unroll
  for (int c = 0; c < 9; ++c) o[c] = p[c * N + v];
}

// E = R^T (Fe^T Fe - 1) R / 2
__device__ __forceinline__ void lattice_strain(const double* Fe, const double* R,
                                               double* E) {
  double C[9], B[9];
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int q = 0; q < 3; ++q)
      C[3 * p + q] = 0.5 * (Fe[p] * Fe[q] + Fe[3 + p] * Fe[3 + q] +
                            Fe[6 + p] * Fe[6 + q] - (p == q ? 1.0 : 0.0));
  mm3(C, R, B);
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int q = 0; q < 3; ++q)
      E[3 * p + q] = R[p] * B[q] + R[3 + p] * B[3 + q] + R[6 + p] * B[6 + q];
}

// ---- return mapping, four lanes per voxel -----------------------------------
// The local problem is solved in the lattice frame, G = Fe R with R the
// grain's orientation, where the slip systems and the cubic stiffness are the
// same constants for every grain: no table is read inside the iteration but
// R once.  Lane h of a quad owns the three slips of plane h.  The planes are
// (1 1 1) with the signs sg_h applied to the lattice axes, (+++), (-++),
// (+-+), (++-), and with them its directions are (1 -1 0), (1 0 -1),
// (0 1 -1) up to the sign of the whole system (plane_slip), so every lane
// runs the same constants.  With m = (1 1 1)/sqrt 3 for a plane's three
// slips, its sum over slips is one vector times m:
//   G = Gs - sum_h v_h (x) sg_h / sqrt 3,  v_h = Gs (sg_h d_h),
// d_h = sum_j dg_j s_j, completed over the quad by three butterflies (the
// same value on every lane, since floating-point addition commutes) and the
// columns' single sign changes by broadcasts.  All lanes of a voxel take
// every decision on identical numbers and run the same iterations.

// the value of another lane of the quad (quad_perm control)
template <int CTRL>
__device__ __forceinline__ double quad_perm(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)(u & 0xffffffffull),
                                          CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), CTRL, 0xF,
                                          0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) |
                                          (unsigned long long)(unsigned)lo));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;  // quad_perm 1,0,3,2 and 2,3,0,1
__device__ __forceinline__ double quad_sum(double x) {
  x = x + quad_perm<kXor1>(x);
  return x + quad_perm<kXor2>(x);
}
__device__ __forceinline__ double quad_max(double x) {
  x = fmax(x, quad_perm<kXor1>(x));
  return fmax(x, quad_perm<kXor2>(x));
}
__device__ __forceinline__ float quad_sumf(float x) {
  x = x + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(
              __builtin_bit_cast(int, x), kXor1, 0xF, 0xF, false));
  return x + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(
                 __builtin_bit_cast(int, x), kXor2, 0xF, 0xF, false));
}
// 1.0 on any lane of the quad -> true on all
__device__ __forceinline__ bool quad_any(bool b) {
  int v = b ? 1 : 0;
  v |= __builtin_amdgcn_mov_dpp(v, kXor1, 0xF, 0xF, false);
  v |= __builtin_amdgcn_mov_dpp(v, kXor2, 0xF, 0xF, false);
  return v != 0;
}

// index of plane h's slip j in the order of the state arrays, and the sign of
// that system relative to the plane's signs applied to (1 -1 0), (1 0 -1) and
// (0 1 -1): slips and back stresses change sign with it
__device__ __forceinline__ int plane_slip(int h, int j) {
  const unsigned t = j == 0 ? 0x9740u : (j == 1 ? 0xA651u : 0xB832u);
  return (int)((t >> (4 * h)) & 15u);
}
__device__ __forceinline__ double plane_sign(int h, int j) {
  return (j < 2 ? h == 1 : h == 2) ? -1.0 : 1.0;
}

// x with its sign changed where bit 31 of mask is set
__device__ __forceinline__ double flip(double x, unsigned mask) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  return __longlong_as_double((long long)(u ^ ((unsigned long long)mask << 32)));
}
__device__ __forceinline__ float flip(float x, unsigned mask) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, x) ^ mask);
}
// the signs of plane h on the lattice axes, as masks
struct PlaneSigns {
  unsigned m[3];
  __device__ __forceinline__ explicit PlaneSigns(int h) {
#pragma unroll
    for (int i = 0; i < 3; ++i) m[i] = h == i + 1 ? 0x80000000u : 0u;
  }
  __device__ __forceinline__ unsigned both(int i, int j) const { return m[i] ^ m[j]; }
};

// x > 0 of normal range: Goldschmidt's iteration for the square root and
// Newton's for the quotient from the hardware's reciprocal estimates, a last
// correction with the fused residual (results within one unit in the last
// place; the special cases of the library functions do not occur here)
__device__ __forceinline__ double sqrt_pos(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  double g = x * r, h = 0.5 * r;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  return fma(fma(-g, g, x), h, g);
}
__device__ __forceinline__ double div_pos(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  r = fma(fma(-b, r, 1.0), r, r);
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// 2 atanh(q), |q| <= 0.2005: the first term left out is below 2e-17 of the sum
__device__ __forceinline__ double atanh2(double q) {
  const double q2 = q * q;
  double p = 1.0 / 21.0;
#pragma unroll
  for (int m = 9; m >= 0; --m) p = fma(q2, p, 1.0 / (2 * m + 1));
  return 2.0 * q * p;
}
constexpr double kLn2 = 0.69314718055994530942;

// k = log2(p / d) rounded (p and d positive): the exponent and the leading
// bits of the mantissa are log2 to within 0.086, so |log2(p / d) - k| < 0.587,
// and k = 0 where p and d are close
__device__ __forceinline__ int octaves(double p, double d) {
  return (__double2hiint(p) - __double2hiint(d) + (1 << 19)) >> 20;
}

// The local residual R = asinh(u) - asinh(|x|^n sign x), u = dg / a, through
// A = |u| + sqrt(1 + u^2) and B = y + sqrt(1 + y^2), y = |x|^n:
// R = s ln(A / B) when the signs agree (or one is zero; s the nonzero one)
// and R = su ln(A B) when they differ -- exact identities.  The logarithm of
// p / d is k ln 2 + 2 atanh(q), q = (p 2^-k - d)/(p 2^-k + d), with the k
// that keeps q small: near the root k = 0, and R there carries an absolute
// error of a few units of 1e-16, which is what the converged slips depend on.
// FP64 throughout and free of branches.  The derivative of
// asinh(|x|^n sign x) (Jacobian only) is in single precision.  Past
// LawParams::xmax, where y^2 would leave the FP64 range (|x| of 1e7 up to
// n = 21, 1e3 for n = 50, 220 for n = 64), y is the power of |x| 2^-j, still
// so large that B = 2 y, and n j octaves are added to the logarithm.
// Non-integer n (INTN false): the two functions are evaluated apart.
__device__ __forceinline__ double asinh_bf(double u);
template <bool INTN>
__device__ __forceinline__ void flow_residual(double t, double x,
                                              const LawParams& lp, double& R,
                                              float& der) {
  const double ax = fabs(x), n = lp.nexp, inv_a = lp.inv_a;
  if constexpr (INTN) {
    const int j = ax >= lp.xmax ? __builtin_amdgcn_frexp_exp(ax) - lp.xexp : 0;
    const double y = ipow_n(__builtin_amdgcn_ldexp(ax, -j), lp.nint);
    const double B = y + sqrt_pos(fma(y, y, 1.0));
    const double au = fabs(t * inv_a);
    const double A = au + sqrt_pos(fma(au, au, 1.0));
    const bool differ = (t > 0.0 && x < 0.0) || (t < 0.0 && x > 0.0);
    const double m = differ ? B : 1.0, d = differ ? 1.0 : B;
    const int k = octaves(A * m, d);
    const double As = __builtin_amdgcn_ldexp(A, -k);
    const double q = div_pos(fma(As, m, -d), fma(As, m, d));
    const int oct = k + (differ ? lp.nint * j : -lp.nint * j);
    const double r = fma((double)oct, kLn2, atanh2(q));
    const double s = (t != 0.0) ? t : x;
    R = s < 0.0 ? -r : r;
    const float yf = (float)y;
    const float rs = (y >= 1e18) ? 1.0f : yf * rsqrtf(fmaf(yf, yf, 1.0f));
    der = (ax > 1e-30) ? (float)n * rs * __builtin_amdgcn_rcpf((float)ax) : 0.0f;
  } else {
    double val, d;
    asinh_pow(x, n, val, d);
    R = asinh_bf(t * inv_a) - val;
    der = (float)d;
  }
}

// asinh(u) in one branch-free form, exact for every u:
// asinh(|u|) = log1p(|u| + u^2 / (1 + sqrt(1 + u^2))), with the quotient
// written as |u| (|u| / (1 + q)) so that it cannot overflow.
__device__ __forceinline__ double asinh_bf(double u) {
  const double au = fabs(u);
  const double q = sqrt(1.0 + au * au);
  return copysign(log1p(au + au * (au / (1.0 + q))), u);
}

constexpr double kInvSqrt6 = 0.40824829046386301637;
constexpr float kInvSqrt6f = 0.40824829046386302f;

// dG = sum over the slips of dg_a (B s_a) (x) m_a for the lane's slips t and
// a matrix B in the lattice frame, completed over the quad
__device__ __forceinline__ void slip_sum(const double* B, const double* t,
                                         const PlaneSigns& sg, double* dG) {
  const double d0 = flip(kInvSqrt6 * (t[0] + t[1]), sg.m[0]);
  const double d1 = flip(kInvSqrt6 * (t[2] - t[0]), sg.m[1]);
  const double d2 = flip(-kInvSqrt6 * (t[1] + t[2]), sg.m[2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double v = B[3 * i] * d0 + B[3 * i + 1] * d1 + B[3 * i + 2] * d2;
    const double T = quad_sum(v);
    dG[3 * i] = fma(-2.0, quad_perm<0x55>(v), T);
    dG[3 * i + 1] = fma(-2.0, quad_perm<0xAA>(v), T);
    dG[3 * i + 2] = fma(-2.0, quad_perm<0xFF>(v), T);
  }
}

// The elastic strain in the lattice frame at G = Gs - dG: with that of Gs,
//   E = Es - sym((Gs - dG/2)^T dG),
// which subtracts no unit matrix (Es = R^T (Fes^T Fes - 1) R / 2 is exactly
// zero in an undeformed voxel, and so are then its stress and P).
__device__ __forceinline__ double strain_term(const double* Gs, const double* dG,
                                              int p, int q) {
  double e = 0.0;
#pragma unroll
  for (int i = 0; i < 9; i += 3) {
    e += fma(-0.5, dG[i + p], Gs[i + p]) * dG[i + q];
    if (p != q) e += fma(-0.5, dG[i + q], Gs[i + q]) * dG[i + p];
  }
  return p == q ? e : 0.5 * e;
}

// R and slopes of the lane's slips at t = dg + lam * step, and Q = G^T Gs
// there, with the plane's signs on both indices, for the Jacobian; es: the
// strain Es as e11 - e22, e11 - e33, e12, e13, e23 (m and s of a slip are
// orthogonal: only these enter its resolved shear)
template <bool INTN>
__device__ __forceinline__ void pr_eval(const double* Gs, const double* es,
                                        const double* chi0,
                                        const double* dg, const double* step,
                                        double lam, const PlaneSigns& sg,
                                        const LawParams& lp, double* R,
                                        float* hd, float* Q) {
  double t[3], G[9];
#pragma unroll
  for (int j = 0; j < 3; ++j) t[j] = dg[j] + lam * step[j];
  slip_sum(Gs, t, sg, G);   // dG
  const double x0 = strain_term(Gs, G, 0, 0);
  const double kd = kInvSqrt6 * lp.c11m12, k44 = 2.0 * kInvSqrt6 * lp.c44;
  const double d01 = kd * (es[0] - (x0 - strain_term(Gs, G, 1, 1)));
  const double d02 = kd * (es[1] - (x0 - strain_term(Gs, G, 2, 2)));
  const double c01 = flip(k44 * (es[2] - strain_term(Gs, G, 0, 1)), sg.both(0, 1));
  const double c02 = flip(k44 * (es[3] - strain_term(Gs, G, 0, 2)), sg.both(0, 2));
  const double c12 = flip(k44 * (es[4] - strain_term(Gs, G, 1, 2)), sg.both(1, 2));
#pragma unroll
  for (int i = 0; i < 9; ++i) G[i] = Gs[i] - G[i];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const float q = (float)(G[i] * Gs[j] + G[3 + i] * Gs[3 + j] + G[6 + i] * Gs[6 + j]);
      Q[3 * i + j] = flip(q, sg.both(i, j));
    }
  const double tau[3] = {d01 + (c02 - c12), d02 + (c01 - c12),
                         (d02 - d01) + (c01 - c02)};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double chi = div_pos(chi0[j] + lp.c_af * t[j], 1.0 + lp.d_af * fabs(t[j]));
    flow_residual<INTN>(t[j], (tau[j] - chi) * lp.inv_g, lp, R[j], hd[j]);
  }
}

// The slips' symmetric Schmid tensors have no trace: in the orthonormal basis
// (e11 - e22)/sqrt 2, (e11 + e22 - 2 e33)/sqrt 6, sqrt 2 e23, sqrt 2 e13,
// sqrt 2 e12 of the trace-free tensors they are five-vectors.  Those of the
// plane (1 1 1), in units of 1/sqrt 12:
__device__ constexpr float kSchmid5[3][5] = {{2.0f, 0.0f, -1.0f, 1.0f, 0.0f},
                                             {1.0f, 1.7320508075688773f, -1.0f, 0.0f, 1.0f},
                                             {-1.0f, 1.7320508075688773f, 0.0f, -1.0f, 1.0f}};

__device__ constexpr double kSchmid5d[3][5] = {
    {2.0, 0.0, -1.0, 1.0, 0.0},
    {1.0, 1.73205080756887729353, -1.0, 0.0, 1.0},
    {-1.0, 1.73205080756887729353, 0.0, -1.0, 1.0}};

// z <- M^-1 z by elimination, with row interchanges or without
template <bool PIVOT>
__device__ __forceinline__ void solve5(float* M, float* z) {
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    if constexpr (PIVOT) {
#pragma unroll
      for (int r = k + 1; r < 5; ++r) {
        const bool s = fabsf(M[5 * r + k]) > fabsf(M[6 * k]);
#pragma unroll
        for (int J = k; J < 5; ++J) {
          const float a = M[5 * k + J], b = M[5 * r + J];
          M[5 * k + J] = s ? b : a;
          M[5 * r + J] = s ? a : b;
        }
        const float a = z[k], b = z[r];
        z[k] = s ? b : a;
        z[r] = s ? a : b;
      }
    }
    const float ip = __builtin_amdgcn_rcpf(M[6 * k]);
    M[6 * k] = ip;
#pragma unroll
    for (int r = k + 1; r < 5; ++r) {
      const float m = M[5 * r + k] * ip;
#pragma unroll
      for (int J = k + 1; J < 5; ++J) M[5 * r + J] -= m * M[5 * k + J];
      z[r] -= m * z[k];
    }
  }
#pragma unroll
  for (int k = 4; k >= 0; --k) {
#pragma unroll
    for (int J = k + 1; J < 5; ++J) z[k] -= M[5 * k + J] * z[J];
    z[k] *= M[6 * k];
  }
}

// Newton step of the lane's slips: step = -J^-1 R.  J = diag(1/D) + h N V^T
// with V_a = sym((Q s_a) (x) m_a), Q = G^T Gs, and N_a = C : sym(S0_a); in
// the basis above Woodbury's capacitance matrix is the 5x5
// 1 + sum_a D_a h_a v_a (x) C n_a.  v_a differs from n_a by the elastic strain
// only, so with D_a h_a >= 0 and moduli that are not negative the matrix is,
// up to a diagonal similarity, which changes no pivot, close to symmetric
// positive definite, and it is eliminated without pivoting.  Softening
// back stresses (D_a h_a < 0) and other constants take row interchanges.
// The Jacobian only steers the iteration (the root is that of the FP64
// residual R): single precision.
__device__ __forceinline__ void pr_step(const double* dg, const double* R,
                                        const float* hd, const float* Q,
                                        const double* chi0, const PlaneSigns& sg,
                                        const LawParams& lp, float a2, double* step) {
  // basis components' moduli, with their signs in the plane's frame
  const float kd = (float)lp.c11m12, ks = 2.0f * (float)lp.c44;
  const float k5[5] = {kd, kd, flip(ks, sg.both(1, 2)), flip(ks, sg.both(0, 2)),
                       flip(ks, sg.both(0, 1))};
  bool indefinite = !lp.definite;
  const float inv_g = (float)lp.inv_g, c_af = (float)lp.c_af, d_af = (float)lp.d_af;
  float M[25], V[3][5], D[3], z[5];
#pragma unroll
  for (int i = 0; i < 25; ++i) M[i] = 0.0f;
#pragma unroll
  for (int i = 0; i < 5; ++i) z[i] = 0.0f;
  float f[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const float dgf = (float)dg[j];
    const float den = __builtin_amdgcn_rcpf(1.0f + d_af * fabsf(dgf));
    const float chi = ((float)chi0[j] + c_af * dgf) * den;
    const float s = (dgf > 0.0f) ? 1.0f : ((dgf < 0.0f) ? -1.0f : 0.0f);
    const float dchi = (c_af - d_af * s * chi) * den;
    D[j] = __builtin_amdgcn_rcpf(rsqrtf(a2 + dgf * dgf) + hd[j] * inv_g * dchi);
    f[j] = hd[j] * inv_g * D[j];
    indefinite = indefinite || f[j] < 0.0f;
    // Q s_j of (1 -1 0), (1 0 -1), (0 1 -1), in units of 1/sqrt 2
    constexpr int ps[3] = {0, 0, 1}, ms[3] = {1, 2, 2};
    const float q0 = Q[ps[j]] - Q[ms[j]], q1 = Q[3 + ps[j]] - Q[3 + ms[j]],
                q2 = Q[6 + ps[j]] - Q[6 + ms[j]];
    // sym(q (x) (1 1 1)) in the basis, in units of 1/sqrt 6
    constexpr float r2 = 0.70710678118654752f, r6 = 0.40824829046386302f;
    V[j][0] = kInvSqrt6f * r2 * (q0 - q1);
    V[j][1] = kInvSqrt6f * r6 * (q0 + q1 - 2.0f * q2);
    V[j][2] = flip(kInvSqrt6f * r2 * (q1 + q2), sg.both(1, 2));
    V[j][3] = flip(kInvSqrt6f * r2 * (q0 + q2), sg.both(0, 2));
    V[j][4] = flip(kInvSqrt6f * r2 * (q0 + q1), sg.both(0, 1));
    const float sj = -(float)R[j] * D[j];
    step[j] = -R[j] * (double)D[j];
#pragma unroll
    for (int I = 0; I < 5; ++I) {
      z[I] += V[j][I] * sj;
      const float fv = f[j] * V[j][I];
#pragma unroll
      for (int J = 0; J < 5; ++J)
        if (kSchmid5[j][J] != 0.0f) M[5 * I + J] += fv * kSchmid5[j][J];
    }
  }
  constexpr float r12 = 0.28867513459481288f;   // 1/sqrt 12
#pragma unroll
  for (int I = 0; I < 5; ++I) {
    z[I] = quad_sumf(z[I]);
#pragma unroll
    for (int J = 0; J < 5; ++J)
      M[5 * I + J] = (I == J ? 1.0f : 0.0f) + quad_sumf(M[5 * I + J] * (r12 * k5[J]));
  }
  if (quad_any(indefinite))
    solve5<true>(M, z);
  else
    solve5<false>(M, z);
#pragma unroll
  for (int I = 0; I < 5; ++I) z[I] *= r12 * k5[I];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    float u = 0.0f;
#pragma unroll
    for (int J = 0; J < 5; ++J)
      if (kSchmid5[j][J] != 0.0f) u += kSchmid5[j][J] * z[J];
    step[j] -= (double)(f[j] * u);
  }
}

__device__ __forceinline__ double half_sq(const double* R) {
  return 0.5 * (R[0] * R[0] + R[1] * R[1] + R[2] * R[2]);
}

// damped Newton with Armijo backtracking on |R|^2/2 over the quad; dg holds
// the lane's slips
template <bool INTN>
__device__ __forceinline__ bool pr_local_solve(const double* Gs,
                                               const double* es,
                                               const double* chi0, double* dg,
                                               const PlaneSigns& sg,
                                               const LawParams& lp, double a,
                                               int& iters, int& evals) {
  double R[3], step[3] = {0.0, 0.0, 0.0};
  float hd[3], Q[9];
  const float a2 = (float)(a * a);
  pr_eval<INTN>(Gs, es, chi0, dg, step, 0.0, sg, lp, R, hd, Q);
  ++evals;
  for (int it = 0; it < LOCAL_MAXIT; ++it) {
    ++iters;
    pr_step(dg, R, hd, Q, chi0, sg, lp, a2, step);
    double smax = 0.0, dmax = 0.0, rmax = 0.0;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      smax = fmax(smax, fabs(step[j]));
      dmax = fmax(dmax, fabs(dg[j] + step[j]));
      rmax = fmax(rmax, fabs(R[j]));
      bad = bad || !isfinite(step[j]);
    }
    smax = quad_max(smax);
    dmax = quad_max(dmax);
    if (!quad_any(bad) && smax <= LOCAL_ATOL + LOCAL_RTOL * dmax) {
#pragma unroll
      for (int j = 0; j < 3; ++j) dg[j] += step[j];
      return true;
    }
    const double merit0 = quad_sum(half_sq(R));
    double lam = 1.0, lam_used = 1.0;
    bool accepted = false;
    for (int ls = 0; ls < 40; ++ls) {
      pr_eval<INTN>(Gs, es, chi0, dg, step, lam, sg, lp, R, hd, Q);
      ++evals;
      lam_used = lam;
      const double mt = quad_sum(half_sq(R));
      if (isfinite(mt) && mt <= (1.0 - 1e-4 * lam) * merit0) {
        accepted = true;
        break;
      }
      lam *= 0.5;
    }
    bool nf = false;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      dg[j] = dg[j] + lam_used * step[j];
      nf = nf || !isfinite(dg[j]);
    }
    if (quad_any(nf)) return false;
    if (!accepted && quad_max(rmax) <= LOCAL_RFLOOR) return true;
  }
  return false;
}

}  // namespace

// Bound by the issue of the local iteration (about 1000 vector instructions
// per Newton step and residual, a third of them FP64, for the sixteen voxels
// of a wavefront): after three tensile increments of 3e-4, in the sample frame
// with tables / now: 128^3 5350 / 1745 us, 64^3 719 / 250, 32^3 115 / 50, 16^3
// 86 / 34.  The 178 MB of a 64^3 launch would take 35 us.
template <bool INTN, int BLK, int WAVES>
__global__ __launch_bounds__(BLK, WAVES) void return_map_kernel(ConstArgs A) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t g = t / 4;
  const int h = (int)(t % 4);
  if (g >= A.N) return;  // all lanes of a voxel leave together
  const int64_t v = A.order ? (int64_t)A.order[g] : g;
  if (A.vrve && A.scs[A.vrve[v]].inactive) return;
  const int64_t N = A.N;
  const double* __restrict__ tb = A.table + (int64_t)A.phase[v] * kTableStride;
  double F[9];
  load9(A.F, v, N, F);
  if (tb[0] != 0.0) {  // isotropic SVK particle
    const double lam = tb[kTabLam], mu = tb[kTabMu];
    double C[9];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        C[3 * p + q] = F[p] * F[q] + F[3 + p] * F[3 + q] + F[6 + p] * F[6 + q];
    const double tr = 0.5 * (C[0] + C[4] + C[8] - 3.0);
    double S[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) S[i] = mu * (C[i] - ((i % 4 == 0) ? 1.0 : 0.0));
    S[0] += lam * tr;
    S[4] += lam * tr;
    S[8] += lam * tr;
    double P[9];
    mm3(F, S, P);
#pragma unroll
    for (int c = 0; c < 9; ++c)
      if (c % 4 == h) {
        A.P[c * N + v] = P[c];
        A.Fpi[c * N + v] = A.Fpi0[c * N + v];
      }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int al = 3 * h + j;
      A.chi[al * N + v] = A.chi0[al * N + v];
      A.dg[al * N + v] = 0.0;
    }
    if (A.iters && h == 0) {
      A.iters[v] = -1;  // particle voxel
      A.evals[v] = 0;
    }
    return;
  }
  const PlaneSigns sg(h);
  double dg[3], chi0[3];
  bool warm = false;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int64_t at = plane_slip(h, j) * N + v;
    chi0[j] = plane_sign(h, j) * A.chi0[at];
    dg[j] = A.dg0 ? plane_sign(h, j) * A.dg0[at] : 0.0;
    warm = warm || dg[j] != 0.0;
  }
  warm = quad_any(warm);
  // Gs = F Fp^-1_0 R and its strain in the lattice frame
  double Gs[9], es[5], e0;
  {
    double Fp0[9], Rm[9], Fes[9];
    load9(A.Fpi0, v, N, Fp0);
#pragma unroll
    for (int i = 0; i < 9; ++i) Rm[i] = tb[kTabR + i];
    mm3(F, Fp0, Fes);
    mm3(Fes, Rm, Gs);
    double E[9];
    lattice_strain(Fes, Rm, E);
    e0 = E[0];
    es[0] = E[0] - E[4];
    es[1] = E[0] - E[8];
    es[2] = E[1];
    es[3] = E[2];
    es[4] = E[5];
  }
  const double a = A.lp.dt * A.lp.gdot0;
  int iters = 0, evals = 0;
  bool ok = false;
  for (int attempt = 0; attempt < 2 && !ok; ++attempt) {
    if (attempt == 1) {
      if (!warm) break;
#pragma unroll
      for (int j = 0; j < 3; ++j) dg[j] = 0.0;  // retry from zero slips
    }
    ok = pr_local_solve<INTN>(Gs, es, chi0, dg, sg, A.lp, a, iters, evals);
  }
  if (!ok && h == 0) atomicAdd(A.vrve ? &A.scs[A.vrve[v]].fails : A.fails, 1);
  // final state: Fp^-1 = Fp^-1_0 - dFp R^T, G = Fe R, S = C : Ee, and
  // P = Fe S Fp^-T = G S (Fp^-1 R)^T, S in the lattice frame
  double G[9], GS[9];
  slip_sum(Gs, dg, sg, G);
  {
    const double x0 = e0 - strain_term(Gs, G, 0, 0);
    const double x1 = (e0 - es[0]) - strain_term(Gs, G, 1, 1);
    const double x2 = (e0 - es[1]) - strain_term(Gs, G, 2, 2);
    const double tr = A.lp.c12 * (x0 + x1 + x2), k44 = 2.0 * A.lp.c44;
    const double s01 = k44 * (es[2] - strain_term(Gs, G, 0, 1));
    const double s02 = k44 * (es[3] - strain_term(Gs, G, 0, 2));
    const double s12 = k44 * (es[4] - strain_term(Gs, G, 1, 2));
    const double S[9] = {A.lp.c11m12 * x0 + tr, s01, s02, s01,
                         A.lp.c11m12 * x1 + tr, s12, s02, s12,
                         A.lp.c11m12 * x2 + tr};
#pragma unroll
    for (int i = 0; i < 9; ++i) G[i] = Gs[i] - G[i];
    mm3(G, S, GS);
  }
  double Fp0[9], Rm[9], B[9], dFp[9];
  load9(opaque(A.Fpi0), v, N, Fp0);
#pragma unroll
  for (int i = 0; i < 9; ++i) Rm[i] = opaque(tb)[kTabR + i];
  mm3(Fp0, Rm, B);
  slip_sum(B, dg, sg, dFp);
#pragma unroll
  for (int i = 0; i < 9; ++i) B[i] -= dFp[i];
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    if (c % 4 != h) continue;
    const int i = c / 3, j = c - 3 * (c / 3);
    A.P[c * N + v] = GS[3 * i] * B[3 * j] + GS[3 * i + 1] * B[3 * j + 1] +
                     GS[3 * i + 2] * B[3 * j + 2];
    A.Fpi[c * N + v] = Fp0[c] - (dFp[3 * i] * Rm[3 * j] + dFp[3 * i + 1] * Rm[3 * j + 1] +
                                 dFp[3 * i + 2] * Rm[3 * j + 2]);
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int64_t at = plane_slip(h, j) * N + v;
    const double sj = plane_sign(h, j);
    A.chi[at] = sj * (chi0[j] + A.lp.c_af * dg[j]) / (1.0 + A.lp.d_af * fabs(dg[j]));
    A.dg[at] = sj * dg[j];
  }
  if (A.iters && h == 0) {
    A.iters[v] = iters;
    A.evals[v] = evals;
  }
}

// Work counts of the last return mapping: stats[0] += local Newton steps,
// [1] += residual evaluations, [2] += crystal voxels, [3] += particle voxels
__global__ __launch_bounds__(256) void rm_count_kernel(
    const int32_t* __restrict__ iters, const int32_t* __restrict__ evals,
    int64_t N, unsigned long long* __restrict__ stats) {
  __shared__ unsigned long long red[4][256];
  unsigned long long c[4] = {0, 0, 0, 0};
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < N;
       v += (int64_t)gridDim.x * blockDim.x) {
    const int it = iters[v];
    if (it < 0) {
      c[3] += 1;
    } else {
      c[0] += (unsigned long long)it;
      c[1] += (unsigned long long)evals[v];
      c[2] += 1;
    }
  }
  for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = c[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) atomicAdd(&stats[threadIdx.x], red[threadIdx.x][0]);
}

// ---- consistent tangent ----------------------------------------------------
// P = F S2(C), C = F^T F, with the second Piola stress S2 = Fp^-1 S Fp^-T, so
//   K_ijkl = d_ik (S2)_lj + F_im D_mj,nl F_kn,   D = 2 dS2/dC,
// and K is stored as D, S2 and F - 1 (kKComp entries per voxel): six strain
// directions instead of nine gradients here, and 51 instead of 81 numbers
// for every K:p (kp_apply).  In the lattice frame, A = Fp^-1 R:
//   dS = C Y^-1 (A^T dE A),   Y = 1 + sum_a f_a V_a (x) (C S0_a),
//   dg_a = f_a S0_a : dS,   dS2 = A dS A^T - sum_a dg_a 2 sym(y_a (x) u_a),
// y_a = Fp^-1_0 R s_a, u_a = A S m_a, f_a = (h_a/g) / (1/sqrt(a^2 + dg^2) +
// (h_a/g) dchi/ddg), V_a = sym((G^T Gs s_a) (x) m_a).  In the orthonormal
// basis of kSchmid5 completed by the trace, C is diagonal and S0_a has no
// trace: Y is a 5x5 block, close to symmetric positive definite up to a
// diagonal similarity (eliminated without pivoting unless a constant or some
// f_a is negative), and one row for the trace, solved by substitution.
// Frames, stresses, the basis pushed forward and f_a in FP64, the rest in the
// precision of K.
//
// Bound by its instructions (about 2500 per voxel) and 540 B per voxel in
// FP32.  64^3: 307 us with nine Woodbury solves per voxel on table entries
// (448 B of scratch per lane) -> 44 us, 128^3 2350 -> 431 us, 64^3 in FP64 401
// -> 71 us; three wavefronts per SIMD need 464 B of scratch per lane and took
// 115 us where two took 52.
constexpr int kPlaneSign[4][3] = {{1, 1, 1}, {-1, 1, 1}, {1, -1, 1}, {1, 1, -1}};
constexpr int kPlaneSlip[4][3] = {{0, 1, 2}, {4, 5, 3}, {7, 6, 8}, {9, 10, 11}};
constexpr int kPlaneFlip[4][3] = {{1, 1, 1}, {-1, -1, 1}, {1, 1, -1}, {1, 1, 1}};

template <typename TK>
__device__ __forceinline__ void tangent_voxel(const TangentArgs<TK>& A, int64_t v) {
  const int64_t N = A.N;
  const double* __restrict__ tb = A.table + (int64_t)A.phase[v] * kTableStride;
  double F[9];
  load9(A.F, v, N, F);
#pragma unroll
  for (int c = 0; c < 9; ++c)
    A.K[(42 + c) * N + v] = TK(F[c] - (c % 4 == 0 ? 1.0 : 0.0));
  if (tb[0] != 0.0) {   // isotropic SVK: S2 = lam tr E + 2 mu E
    const double lam = tb[kTabLam], mu = tb[kTabMu];
    double C[9];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        C[3 * p + q] = F[p] * F[q] + F[3 + p] * F[3 + q] + F[6 + p] * F[6 + q];
    const double tr = 0.5 * (C[0] + C[4] + C[8] - 3.0);
    A.K[36 * N + v] = TK(mu * (C[0] - 1.0) + lam * tr);
    A.K[37 * N + v] = TK(mu * (C[4] - 1.0) + lam * tr);
    A.K[38 * N + v] = TK(mu * (C[8] - 1.0) + lam * tr);
    A.K[39 * N + v] = TK(mu * C[5]);
    A.K[40 * N + v] = TK(mu * C[2]);
    A.K[41 * N + v] = TK(mu * C[1]);
#pragma unroll
    for (int I = 0; I < 6; ++I)
#pragma unroll
      for (int J = 0; J < 6; ++J) {
        double d = (I < 3 && J < 3) ? lam : 0.0;
        if (I == J) d += I < 3 ? 2.0 * mu : mu;
        A.K[(6 * I + J) * N + v] = TK(d);
      }
    return;
  }
  const LawParams& lp = A.lp;
  const double a = lp.dt * lp.gdot0;
  // slips in the planes' frames, and the plastic increment 1 - sum dg s (x) m
  double dg[4][3], Ap[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) Ap[i] = (i % 4 == 0) ? 1.0 : 0.0;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
      dg[h][j] = kPlaneFlip[h][j] * A.dg[kPlaneSlip[h][j] * N + v];
    const double d[3] = {kInvSqrt6 * (dg[h][0] + dg[h][1]),
                         kInvSqrt6 * (dg[h][2] - dg[h][0]),
                         -kInvSqrt6 * (dg[h][1] + dg[h][2])};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        Ap[3 * i + j] -= (kPlaneSign[h][i] * kPlaneSign[h][j]) * d[i];
  }
  TK Y0[9], Q[9], Fs[9];   // Fp^-1_0 R, G^T Gs, Fp^-1 R S
  double Ac[9], S64[6];    // Fp^-1 R, S
  {
    double Fp0[9], Rm[9], B[9], Gs[9], G[9];
    load9(A.Fpi0, v, N, Fp0);
#pragma unroll
    for (int i = 0; i < 9; ++i) Rm[i] = tb[kTabR + i];
    mm3(Fp0, Rm, B);
    mm3(F, B, Gs);
    mm3(B, Ap, Ac);
    mm3(Gs, Ap, G);
    double E[6];
    constexpr int vi[6] = {0, 1, 2, 1, 0, 0}, vj[6] = {0, 1, 2, 2, 2, 1};
#pragma unroll
    for (int I = 0; I < 6; ++I)
      E[I] = 0.5 * (G[vi[I]] * G[vj[I]] + G[3 + vi[I]] * G[3 + vj[I]] +
                    G[6 + vi[I]] * G[6 + vj[I]] - (I < 3 ? 1.0 : 0.0));
    const double tr = lp.c12 * (E[0] + E[1] + E[2]);
#pragma unroll
    for (int I = 0; I < 6; ++I)
      S64[I] = I < 3 ? lp.c11m12 * E[I] + tr : 2.0 * lp.c44 * E[I];
#pragma unroll
    for (int i = 0; i < 9; ++i) Y0[i] = TK(B[i]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        Q[3 * i + j] = TK(G[i] * Gs[j] + G[3 + i] * Gs[3 + j] + G[6 + i] * Gs[6 + j]);
  }
  {
    double fs[9];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      fs[3 * i] = Ac[3 * i] * S64[0] + Ac[3 * i + 1] * S64[5] + Ac[3 * i + 2] * S64[4];
      fs[3 * i + 1] = Ac[3 * i] * S64[5] + Ac[3 * i + 1] * S64[1] + Ac[3 * i + 2] * S64[3];
      fs[3 * i + 2] = Ac[3 * i] * S64[4] + Ac[3 * i + 1] * S64[3] + Ac[3 * i + 2] * S64[2];
    }
    auto s2 = [&](int i, int j) {
      return TK(fs[3 * i] * Ac[3 * j] + fs[3 * i + 1] * Ac[3 * j + 1] +
                fs[3 * i + 2] * Ac[3 * j + 2]);
    };
    A.K[36 * N + v] = s2(0, 0);
    A.K[37 * N + v] = s2(1, 1);
    A.K[38 * N + v] = s2(2, 2);
    A.K[39 * N + v] = s2(1, 2);
    A.K[40 * N + v] = s2(0, 2);
    A.K[41 * N + v] = s2(0, 1);
#pragma unroll
    for (int i = 0; i < 9; ++i) Fs[i] = TK(fs[i]);
  }
  // Phi: the basis tensors pushed forward by A (columns), in the order 11,
  // 22, 33, 23, 13, 12; L starts as Phi C and takes the plastic part
  TK Phi[6][6], L[6][5], Y[25], yt[5];
  const TK cd = TK(lp.c11m12), cs = TK(2.0 * lp.c44);
  bool pivot = !lp.definite;
  {
    constexpr int vi[6] = {0, 1, 2, 1, 0, 0}, vj[6] = {0, 1, 2, 2, 2, 1};
    constexpr double r2 = 0.70710678118654752440, r3 = 0.57735026918962576451,
                     r6 = 0.40824829046386301637;
#pragma unroll
    for (int I = 0; I < 6; ++I) {
      const double* p = Ac + 3 * vi[I];
      const double* q = Ac + 3 * vj[I];
      const double w0 = p[0] * q[0], w1 = p[1] * q[1], w2 = p[2] * q[2];
      Phi[I][0] = TK(r2 * (w0 - w1));
      Phi[I][1] = TK(r6 * (w0 + w1 - 2.0 * w2));
      Phi[I][2] = TK(r2 * (p[1] * q[2] + p[2] * q[1]));
      Phi[I][3] = TK(r2 * (p[0] * q[2] + p[2] * q[0]));
      Phi[I][4] = TK(r2 * (p[0] * q[1] + p[1] * q[0]));
      Phi[I][5] = TK(r3 * (w0 + w1 + w2));
#pragma unroll
      for (int k = 0; k < 5; ++k) L[I][k] = Phi[I][k] * (k < 2 ? cd : cs);
    }
  }
#pragma unroll
  for (int i = 0; i < 25; ++i) Y[i] = TK(0);
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    Y[6 * i] = TK(1);
    yt[i] = TK(0);
  }
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    constexpr double k6 = kInvSqrt6;
    const int g0 = kPlaneSign[h][0], g1 = kPlaneSign[h][1], g2 = kPlaneSign[h][2];
    const double t0 = S64[0] + (g0 * g1) * S64[5] + (g0 * g2) * S64[4];
    const double t1 = (g0 * g1) * S64[5] + S64[1] + (g1 * g2) * S64[3];
    const double t2 = (g0 * g2) * S64[4] + (g1 * g2) * S64[3] + S64[2];
    const double tau[3] = {k6 * (t0 - t1), k6 * (t0 - t2), k6 * (t1 - t2)};
    const TK u0 = g0 * Fs[0] + g1 * Fs[1] + g2 * Fs[2];
    const TK u1 = g0 * Fs[3] + g1 * Fs[4] + g2 * Fs[5];
    const TK u2 = g0 * Fs[6] + g1 * Fs[7] + g2 * Fs[8];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double d = dg[h][j], ad = fabs(d);
      const double chi0 = kPlaneFlip[h][j] * A.chi0[kPlaneSlip[h][j] * N + v];
      const double iden = 1.0 / (1.0 + lp.d_af * ad);
      const double chi = (chi0 + lp.c_af * d) * iden;
      // f = hg / (1/w + hg dchi), w^2 = a^2 + dg^2, in FP64 like its terms
      const double hg = flow_slope((tau[j] - chi) * lp.inv_g, lp) * lp.inv_g;
      const double w = sqrt(a * a + d * d);
      const double dchi = (lp.c_af - lp.d_af * sgn(d) * chi) * iden;
      const TK f = TK(hg * w / fma(hg * w, dchi, 1.0));
      // the system s = (sg_p e_p - sg_m e_m)/sqrt 2
      constexpr int ps[3] = {0, 0, 1}, ms[3] = {1, 2, 2};
      const int gp = kPlaneSign[h][ps[j]], gm = kPlaneSign[h][ms[j]];
      const TK q0 = gp * Q[ps[j]] - gm * Q[ms[j]];
      const TK q1 = gp * Q[3 + ps[j]] - gm * Q[3 + ms[j]];
      const TK q2 = gp * Q[6 + ps[j]] - gm * Q[6 + ms[j]];
      const TK y0 = gp * Y0[ps[j]] - gm * Y0[ms[j]];
      const TK y1 = gp * Y0[3 + ps[j]] - gm * Y0[3 + ms[j]];
      const TK y2 = gp * Y0[6 + ps[j]] - gm * Y0[6 + ms[j]];
      pivot = pivot || f < TK(0);
      const TK f12 = f * TK(k6 * 0.28867513459481288225);
      const TK fd = f12 * cd, fs = f12 * cs;
      const TK w0 = g0 * q0, w1 = g1 * q1, w2 = g2 * q2;
      const TK V[5] = {TK(0.70710678118654752440) * (w0 - w1),
                       TK(k6) * (w0 + w1 - TK(2) * w2),
                       TK(0.70710678118654752440) * (g2 * q1 + g1 * q2),
                       TK(0.70710678118654752440) * (g2 * q0 + g0 * q2),
                       TK(0.70710678118654752440) * (g1 * q0 + g0 * q1)};
      const TK Vt = TK(0.57735026918962576451) * (w0 + w1 + w2);
      const TK Z[6] = {TK(2) * y0 * u0, TK(2) * y1 * u1, TK(2) * y2 * u2,
                       y1 * u2 + y2 * u1, y0 * u2 + y2 * u0, y0 * u1 + y1 * u0};
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const double c5 = kSchmid5d[j][k] *
                          (k == 2 ? g1 * g2 : (k == 3 ? g0 * g2 : (k == 4 ? g0 * g1 : 1)));
        if (c5 == 0.0) continue;
        const TK fc = (k < 2 ? fd : fs) * TK(c5);
#pragma unroll
        for (int I = 0; I < 5; ++I) Y[5 * I + k] += V[I] * fc;
        yt[k] += Vt * fc;
#pragma unroll
        for (int I = 0; I < 6; ++I) L[I][k] -= Z[I] * fc;
      }
    }
  }
  // eliminate Y (pivots' reciprocals on the diagonal)
  unsigned swaps = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    if (pivot) {
#pragma unroll
      for (int r = k + 1; r < 5; ++r) {
        const bool s = fabs(Y[5 * r + k]) > fabs(Y[6 * k]);
        swaps |= (s ? 1u : 0u) << (5 * k + r);
#pragma unroll
        for (int J = 0; J < 5; ++J) {
          const TK a = Y[5 * k + J], b = Y[5 * r + J];
          Y[5 * k + J] = s ? b : a;
          Y[5 * r + J] = s ? a : b;
        }
      }
    }
    const TK ip = TK(1) / Y[6 * k];
    Y[6 * k] = ip;
#pragma unroll
    for (int r = k + 1; r < 5; ++r) {
      const TK m = Y[5 * r + k] * ip;
      Y[5 * r + k] = m;
#pragma unroll
      for (int J = k + 1; J < 5; ++J) Y[5 * r + J] -= m * Y[5 * k + J];
    }
  }
  const TK k3 = TK(lp.c11m12 + 3.0 * lp.c12);   // C11 + 2 C12
#pragma unroll
  for (int J = 0; J < 6; ++J) {   // strain direction J (engineering shears)
    TK z[5], zt = Phi[J][5];
#pragma unroll
    for (int k = 0; k < 5; ++k) z[k] = Phi[J][k];
    if (swaps) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = k + 1; r < 5; ++r) {
          const bool s = (swaps >> (5 * k + r)) & 1u;
          const TK a = z[k], b = z[r];
          z[k] = s ? b : a;
          z[r] = s ? a : b;
        }
    }
#pragma unroll
    for (int k = 1; k < 5; ++k)
#pragma unroll
      for (int r = 0; r < k; ++r) z[k] -= Y[5 * k + r] * z[r];
#pragma unroll
    for (int k = 4; k >= 0; --k) {
#pragma unroll
      for (int r = k + 1; r < 5; ++r) z[k] -= Y[5 * k + r] * z[r];
      z[k] *= Y[6 * k];
      zt -= yt[k] * z[k];
    }
    zt *= k3;
#pragma unroll
    for (int I = 0; I < 6; ++I) {
      TK d = Phi[I][5] * zt;
#pragma unroll
      for (int k = 0; k < 5; ++k) d += L[I][k] * z[k];
      A.K[(6 * I + J) * N + v] = d;
    }
  }
}

template <typename TK>
__global__ __launch_bounds__(128, sizeof(TK) == 4 ? 2 : 1) void
tangent_kernel(TangentArgs<TK> A) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.N) return;
  const int64_t v = A.order ? (int64_t)A.order[i] : i;
  if (A.vrve && A.scs[A.vrve[v]].inactive) return;
  tangent_voxel(A, v);
}

// K of the test hook: all 81 components from the stored form
template <typename TK>
__global__ __launch_bounds__(256) void expand_tangent_kernel(
    const TK* __restrict__ K, TK* __restrict__ out, int64_t N) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
  TK Kv[kKComp];
#pragma unroll
  for (int i = 0; i < kKComp; ++i) Kv[i] = K[i * N + v];
  for (int kl = 0; kl < 9; ++kl) {
    TK p[9], y[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) p[i] = (i == kl) ? TK(1) : TK(0);
    kp_apply(Kv, p, y);
#pragma unroll
    for (int i = 0; i < 9; ++i) out[(9 * i + kl) * N + v] = y[i];
  }
}

// Three wavefronts per SIMD (166 registers) beat two once the grid fills them
// (64^3 253 against 279 us, 40^3 89 against 96 us); up to 32^3, whose
// wavefronts are two per SIMD in all, they bring nothing (32^3 49.3 against
// 50.6 us, 24^3 44.6 against 43.4, 16^3 35.8 against 34.9), and blocks of one
// wavefront let the smallest grids reach every CU.  For an exponent that is no
// integer two are faster by a fifth up to 32^3 (32^3 89 against 105 us), three,
// with 168 bytes of scratch, slower by a tenth above (64^3 488 against 450 us).
template <bool INTN>
static void return_map_sized(const ConstArgs& a, hipStream_t s) {
  if (a.N <= 32768)
    launch(return_map_kernel<INTN, 64, 2>, dim3((unsigned)((4 * a.N + 63) / 64)),
           dim3(64), 0, s, a);
  else
    launch(return_map_kernel<INTN, 256, 3>,
           dim3((unsigned)((4 * a.N + 255) / 256)), dim3(256), 0, s, a);
}

void launch_return_map(const ConstArgs& a, hipStream_t s) {
  if (a.lp.nint > 0)
    return_map_sized<true>(a, s);
  else
    return_map_sized<false>(a, s);
}

void launch_rm_count(const int32_t* iters, const int32_t* evals, int64_t N,
                     unsigned long long* stats, hipStream_t s) {
  hipLaunchKernelGGL(rm_count_kernel, dim3(512), dim3(256), 0, s, iters, evals,
                     N, stats);
}

template <typename TK>
void launch_tangent(const TangentArgs<TK>& a, hipStream_t s) {
  const int blk = 128;
  const int64_t grid = (a.N + blk - 1) / blk;
  launch((tangent_kernel<TK>), dim3((unsigned)grid), dim3(blk), 0,
                     s, a);
}

template <typename TK>
void launch_expand_tangent(const TK* K, TK* out, int64_t N, hipStream_t s) {
  hipLaunchKernelGGL((expand_tangent_kernel<TK>), dim3((unsigned)((N + 255) / 256)),
                     dim3(256), 0, s, K, out, N);
}

template void launch_expand_tangent<float>(const float*, float*, int64_t, hipStream_t);
template void launch_expand_tangent<double>(const double*, double*, int64_t, hipStream_t);
template void launch_tangent<float>(const TangentArgs<float>&, hipStream_t);
template void launch_tangent<double>(const TangentArgs<double>&, hipStream_t);

}  // namespace rve
