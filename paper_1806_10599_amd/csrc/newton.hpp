// Control of the Newton iteration shared by single and batched solves.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace rve {

// Share of the residual used by the superlinear term of forcing mode 2.
constexpr double kForcingTheta = 0.05;

// Relative tolerance of the linear solve of a Newton iteration that starts
// at the FP64 relative residual rel (inexact Newton; the equilibrium test
// itself never changes):
//   0: cg_tol;
//   1: min(0.1, max(cg_tol, newton_tol / (4 rel))): only as tight as
//      reaching the equilibrium tolerance needs (the linear part of the
//      next residual at most a quarter of the tolerance);
//   2: min(0.1, max(cg_tol, newton_tol / (2 rel), kForcingTheta * rel)):
//      half of the tolerance for the linear part (the quadratic remainder
//      of the last correction is orders of magnitude below it), and never
//      tighter than kForcingTheta * rel: far from equilibrium the next
//      residual is dominated by the quadratic term of Newton's method,
//      which a tighter solve cannot reduce.
// (host and device: the batch takes the decision on the device)
__host__ __device__ inline double forcing_eta(int32_t mode, double cg_tol,
                                              double newton_tol, double rel) {
  if (mode == 0 || !(rel > 0.0)) return cg_tol;
  double eta = fmax(cg_tol, (mode == 2 ? 0.5 : 0.25) * newton_tol / rel);
  if (mode == 2) eta = fmax(eta, kForcingTheta * rel);
  return fmin(0.1, eta);
}

// (lambda + mu)/(lambda + 2 mu) of the isotropic medium whose Green operator
// preconditions the CG runs, from the grains' cubic constants (params: C11,
// C12, C44 first): their Voigt average, with 0.7 of its shear modulus, since
// the flowing grains are softer in shear but not in bulk.  Only this ratio
// matters to CG, and the optimum is flat: on 16^3 and 24^3 polycrystals
// without and with 8 % particles, 0.75 to 0.87 take the same iterations to
// within one in twenty, 0.5 a quarter more, 0 (plain CG) 1.7 times as many.
// Constants without a positive medium: plain CG; one close to incompressible:
// that of an unknown material.
//
// An unknown material (a user's): 0.5, that of lambda = 0.  A medium of any
// stable lambda and mu wants 1/4 to 1, so against plain CG this halves the
// condition number wherever lambda >= 0 and raises it by an eighth at worst
// (Poisson's ratio -1).  Plain CG in the five passes of an iteration was
// slower than the four of a CG on real fields had been (neo-Hookean 16^3
// FP64 1.06 -> 1.20, mixed 1.01 -> 1.21 ms per increment).
constexpr double kPrecUnknown = 0.5;
inline double cg_preconditioner(const double* params) {
  const double mu_el = (params[0] - params[1] + 3.0 * params[2]) / 5.0;
  const double bulk = (params[0] + 2.0 * params[1]) / 3.0;
  const double mu = 0.7 * mu_el, lam = bulk - 2.0 / 3.0 * mu;
  const double c = (lam + mu) / (lam + 2.0 * mu);
  if (!(mu > 0.0 && bulk > 0.0 && c > 0.0)) return 0.0;
  return c < 0.99 ? c : kPrecUnknown;
}

}  // namespace rve
