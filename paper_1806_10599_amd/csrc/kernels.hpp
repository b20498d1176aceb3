// Launch interfaces of the HIP kernels (host side sees only these).
#pragma once

#include <cmath>

#include "common.hpp"

namespace rve {

// pass A inputs: a field, or this block's rows of K:p from the direction's
// field
enum { SRC_FIELD = 0, SRC_KROW = 1 };
// pass C outputs: the field (||out||^2 partials), the direction's field,
// F += the iterate
enum { DST_NORM = 0, DST_P = 1, DST_ADDF = 2 };

template <typename T>
struct SlabFwdArgs {
  const T* field;      // [9][N^3] (SRC_KROW: the direction)
  const T* K;          // SRC_KROW: the tangent, 81 components with kfull,
  bool kfull;          // else its stored form
  cplx<T>* spec;       // [9][N][N][N/2]
  const cplx<T>* tw;   // exp(-2 pi i m / N)
  double* psum;        // optional [9][N] per-slab sums
  double* psq;         // optional [9][N] per-slab sums of squares
  const Scalars* sc;
  int64_t cs;          // component stride of the real fields (N^3, or the
                       // voxel count of a batch arena)
  // optional (CG run): block 0 reduces these p.(K:p) partials and publishes
  // alpha in slot `parity` of scw (cg_alpha_publish)
  const double* pkp = nullptr;
  int pkp_count = 0;
  int parity = 0;
  Scalars* scw = nullptr;
  double* pkp_out = nullptr;  // SRC_KROW: [9][N] partials of p.(K:p)
};

template <typename T>
struct PencilArgs {
  cplx<T>* spec;
  const cplx<T>* tw;
  const T* vt;         // [3][N] wave-vector components per axis
  T invN3;
};

// Tables that pass A of a projection computes and writes (tw null: none)
struct ProjTables {
  cplx<double>* tw = nullptr;
  double* vt = nullptr;
  double L0 = 1.0, L1 = 1.0, L2 = 1.0;
  bool continuous = false;
};

// CG vectors per frequency: see pencil_fwd_body and pencil_inv_body
template <typename T, typename TR>
struct PencilFwdArgs {
  const cplx<T>* spec;
  const cplx<T>* tw;
  const T* vt;
  cplx<TR>* rho;       // [3][N][N][N/2]
  double invN3, prec;
  double *prr, *prz;   // per-block r.r and r.z
  double* pres;        // per-block ||G(P)||^2 (residual)
  const Scalars* sc;
  int parity;
  // K:p folded into pass A: its p.(K:p) partials (alpha is formed here)
  const double* pkp;
  int pkp_count;
  Scalars* scw;
};
template <typename T>
struct PencilInvArgs {
  cplx<T>* spec;
  const cplx<T>* tw;
  const T* vt;
  const cplx<T>* rho;
  cplx<T>* pi;
  cplx<T>* xi;
  T invN3, prec;
  const double *prr, *prz;  // partials of the last pass (null: timing)
  int count;
  Scalars* scw;
  int parity;
};

template <typename T, typename TO>
struct SlabInvArgs {
  const cplx<T>* spec;
  const cplx<T>* tw;
  TO* out;             // [9][N^3]
  double* partial;     // per block
  const Scalars* sc;   // optional early exit
  int64_t cs;          // component stride of out
  const T* vt = nullptr;    // wave vectors of the expansion
};

// G of a field
template <typename T>
struct SpectralLaunch {
  const T* in_field = nullptr;
  cplx<T>* spec = nullptr;
  const cplx<T>* tw = nullptr;
  const T* vt = nullptr;
  double* out_d = nullptr;
  double* partial_inv = nullptr;
  ProjTables tables;
};

// Passes of a single-RVE CG iteration in launch order: the direction (inverse
// x FFT), p in real space, [K:p,] pass A, the residual (forward x FFT); and
// the end of the solve, F += x.
enum { kPassDir = 1, kPassP = 2, kPassA = 4, kPassRes = 8, kPassFinal = 16 };
template <typename T>
struct CgLaunch {
  const T* K = nullptr;
  bool kfull = false;          // K is dP/dF, 81 components (user materials)
  T* p = nullptr;              // direction [9][N^3]
  const T* y = nullptr;        // K : p [9][N^3]
  double* F = nullptr;         // kPassFinal
  cplx<T>* spec = nullptr;
  const cplx<T>* tw = nullptr;
  const T* vt = nullptr;
  cplx<T>* rho = nullptr;      // CG vectors [3][N][N][N/2]
  cplx<T>* pi = nullptr;
  cplx<T>* xi = nullptr;
  double prec = 0.0;           // (lambda + mu)/(lambda + 2 mu) of M
  double* pkp = nullptr;       // p.(K:p) partials
  int pkp_count = 0;
  const double *prr = nullptr, *prz = nullptr;  // last pass's (null: timing)
  double *prr_out = nullptr, *prz_out = nullptr;
  Scalars* sc = nullptr;
  int parity = 0;
  int cpb = 0, tt = 0;         // components per slab block, kz columns per
  int fused = 0;               // pencil block; K:p folded into pass A
};
template <typename T>
void launch_cg(int n, const CgLaunch<T>& L, int mask, hipStream_t s);

// FP64 residual of P: rho = -(P v) in the CG precision TR, psum/psq of P,
// and 3 * residual_blocks(n) partials (r.r, r.z, ||G(P)||^2)
template <typename TR>
struct ResidualLaunch {
  const double* P = nullptr;
  cplx<double>* spec = nullptr;
  const cplx<double>* tw = nullptr;
  const double* vt = nullptr;
  cplx<TR>* rho = nullptr;
  double prec = 0.0;
  double *psum = nullptr, *psq = nullptr;
  double* part = nullptr;
};
template <typename TR>
void launch_residual(int n, const ResidualLaunch<TR>& L, hipStream_t s);
int residual_blocks(int n);
int cg_pencil_blocks(int n, int tt);
int cg_tile(int n);   // the kz columns of a pencil block a handle picks

template <typename T>
void launch_G(int n, const SpectralLaunch<T>& L, hipStream_t s);
// G in FP64 with the static scratch array of noalloc.hip (no allocation)
void noalloc_apply_G(int n, const double L[3], int projection, const double* in,
                     double* out, hipStream_t s);
// blocks of the slab grids
int slab_blocks(int n, int cpb);
// whether a (cpb, tt) schedule exists for the grid edge and precision
bool schedule_valid(int n, bool fp64, int cpb, int tt);

// One RVE of a batch: where its voxels, spectrum and scalars live and where
// its blocks start in the grids of the slab passes (blk[0]), the CG pencil
// passes (blk[1]) and the pencil pass of G (blk[2]).
template <typename T>
struct SpecItem {
  int n;
  int blk[3];
  int cpb;              // components per slab block (1 or 3)
  int tt;               // kz columns per pencil block (4, 8 or 16)
  int npen;             // CG pencil blocks of this RVE
  int64_t off;          // voxel offset in the arena
  int64_t soff;         // complex offset of the spectrum (CG vectors: / 3)
  const cplx<T>* tw;
  const T* vt;
  Scalars* sc;          // this RVE's scalars
  double* pkp;          // p.(K:p) partials (kp_blocks)
  double* prr;          // pencil partials: r.r, r.z, ||G(P)||^2 (3 npen)
  double* psum;         // residual pass sums [9][n]
  double* psq;
};

template <typename T>
struct BatchSpec {
  const SpecItem<T>* items;
  int nitems;
  int cpbs = 3;         // slab schedules among the items (bit 0: cpb 1,
                        // bit 1: cpb 3)
  int64_t cs;           // voxels in the arena (component stride)
  const T* field;       // input of the forward slab pass (CG: K:p)
  const T* K;           // stored tangent
  T* p;                 // CG direction and K:p
  T* y;
  const uint8_t* vrve;  // RVE of each voxel
  cplx<T>* spec;
  cplx<T>* rho;         // CG vectors
  cplx<T>* pi;
  cplx<T>* xi;
  double prec;
  int parity;
  int timing;           // alpha and beta from the scalars (schedule tuner)
};
// blocks of the slab and CG pencil grids and their dynamic LDS
struct BatchGrid {
  int A = 0, B = 0;
  int V = 0;            // voxels / kBlock
  size_t ldsA = 0, ldsB = 0;
};

// out = G(field)
template <typename T>
void launch_G_batch(const BatchSpec<T>& b, double* out, const BatchGrid& g,
                    hipStream_t s);
// FP64 residual of the field: rho, norm partials, psum and psq
template <typename TR>
void launch_residual_batch(const BatchSpec<double>& b, cplx<TR>* rho,
                           const BatchGrid& g, hipStream_t s);
// one CG iteration; the end of the solve, F += x
template <typename T>
void launch_cg_batch(const BatchSpec<T>& b, const BatchGrid& g, hipStream_t s);
template <typename T>
void launch_cg_final_batch(const BatchSpec<T>& b, double* F, const BatchGrid& g,
                           hipStream_t s);
// dynamic LDS of the batched slab and pencil passes of one grid edge
// under a schedule (throws for an invalid one)
template <typename T>
void batch_lds(int n, int cpb, int tt, size_t& slab, size_t& pencil);


bool batch_supported(int n);
template <typename T>
void batch_allow_lds(size_t slab, size_t pencil);

// ---------------------------------------------------------- constitutive
// Per-label table, kTableStride doubles per label:
//   [0] law (0 crystal, 1 isotropic SVK)
//   crystal: s[12][3] at kTabS, m[12][3] at kTabM, Cv[6][6] at kTabC (C_IJ in
//            Voigt order 11,22,33,23,13,12), orientation R[3][3] at kTabR
//   SVK: lambda at kTabLam, mu at kTabMu
constexpr int kTableStride = 128;
constexpr int kTabS = 8, kTabM = 44, kTabC = 80, kTabR = 116;
constexpr int kTabLam = 8, kTabMu = 9;

struct LawParams {
  double gdot0, g, nexp, c_af, d_af, dt;
  double inv_g, inv_a;   // 1/g and 1/(dt gdot0), formed once on the host
  int32_t nint;          // nexp when it is an integer in [1, 64], else 0
  double xmax;           // |x|^(2 nexp) stays below 1e300 up to this |x|
  int32_t xexp;          // 2^xexp is the largest power of two up to xmax
  double c11m12, c12, c44;   // cubic constants of the grains: C11 - C12, ...
  int32_t definite;      // C11 - C12 and C44 are not negative
};

// from the constants of a microstructure (rve.h) and the time step
inline LawParams law_params(const double* p, double dt) {
  LawParams lp{};
  lp.gdot0 = p[3];
  lp.g = p[4];
  lp.nexp = p[5];
  lp.c_af = p[6];
  lp.d_af = p[7];
  lp.dt = dt;
  lp.inv_g = 1.0 / lp.g;
  lp.inv_a = 1.0 / (dt * lp.gdot0);
  // the exponent as an integer when it is one (powers by products)
  const int32_t ni = lp.nexp <= 64.0 ? (int32_t)lp.nexp : 0;
  lp.nint = (double)ni == lp.nexp && ni >= 1 ? ni : 0;
  lp.xmax = std::pow(10.0, std::fmin(7.0, 150.0 / lp.nexp));
  lp.xexp = std::ilogb(lp.xmax);
  lp.c11m12 = p[0] - p[1];
  lp.c12 = p[1];
  lp.c44 = p[2];
  lp.definite = lp.c11m12 >= 0.0 && lp.c44 >= 0.0;
  return lp;
}

struct ConstArgs {
  const double* F;       // [9][N]
  const double* Fpi0;    // committed [9][N]
  const double* chi0;    // committed [12][N]
  const double* dg0;     // starting slips [12][N] or null (zeros)
  const int32_t* phase;  // [N]
  const double* table;   // [labels][kTableStride]
  double* P;             // [9][N]
  double* Fpi;           // trial [9][N]
  double* chi;           // trial [12][N]
  double* dg;            // trial [12][N]
  int32_t* fails;        // counter
  int32_t* iters;        // optional per-voxel local Newton steps (-1: particle)
  int32_t* evals;        // with iters: per-voxel residual evaluations
  LawParams lp;
  int64_t N;
  const uint8_t* vrve;   // batch: RVE of each voxel (null for one RVE)
  Scalars* scs;          // batch: per-RVE flags (skip when inactive) and
                         // per-RVE failure counts (fails unused)
  const int32_t* order;  // optional voxel of each work item: crystal voxels
                         // first, then the particle voxels (null: identity)
};

template <typename TK>
struct TangentArgs {
  const double* F;
  const double* Fpi0;
  const double* chi0;
  const double* dg;      // converged trial slips
  const int32_t* phase;
  const double* table;
  TK* K;                 // [51][N]: D, S2, F - 1 (kp_apply.hpp)
  LawParams lp;
  int64_t N;
  const uint8_t* vrve;
  const Scalars* scs;
  const int32_t* order;  // optional work order (as ConstArgs::order)
};

void launch_return_map(const ConstArgs& a, hipStream_t s);
// Appendix A bridge: F [9][N], sigma [6][N], ddsdde [36][N] -> P [9][N]
// (Eq. A.1), K [81][N] (Eq. A.16); fused, P only, K only (in T)
void launch_umat_bridge(const double* F, const double* sigma,
                        const double* ddsdde, int64_t N, double* P, double* K,
                        hipStream_t s);
void launch_umat_piola(const double* F, const double* sigma, int64_t N,
                       double* P, hipStream_t s);
template <typename T>
void launch_umat_tangent(const double* F, const double* sigma,
                         const double* ddsdde, int64_t N, T* K, hipStream_t s);
// example user material (compressible neo-Hookean) in the same form
void launch_neo_hooke_umat(const double* F1, const double* F0,
                           const double* sv0, double* sv1, int nsv,
                           double* sigma, double* ddsdde, int32_t* fails,
                           int64_t N, hipStream_t s);
void launch_rm_count(const int32_t* iters, const int32_t* evals, int64_t N,
                     unsigned long long* stats, hipStream_t s);
template <typename TK>
void launch_tangent(const TangentArgs<TK>& a, hipStream_t s);
// dP/dF, 81 components, from the stored tangent
template <typename TK>
void launch_expand_tangent(const TK* K, TK* out, int64_t N, hipStream_t s);

// ------------------------------------------------------------- solver ops
struct CommitArgs {
  const double* F;
  const double* Fpi_t;
  const double* dg_t;
  const int32_t* phase;
  const double* table;
  double* pcyc;
  double* pcyc_lit;
  double* wcyc;
  double dt;
  int64_t N;
};

void launch_predict(double* F, const double* Fprev, const double dFbar[9],
                    int64_t N, hipStream_t s);
// y = K : p and the per-block p . y (kp_blocks entries); returns at once on
// a stopped run.  full: K is dP/dF, 81 components, else the stored tangent
template <typename T>
void launch_kp(const T* K, bool full, const T* p, T* y, const Scalars* sc,
               int64_t N, double* pkp, hipStream_t s);
int kp_blocks(int64_t N);  // one voxel per thread
// the CG decision after the last update of a chunk from the partials of the
// last pencil pass; parity: that of the iteration that would follow; pub
// (coherent pinned host memory, or null): where the kernel also copies the
// scalars for the host
void launch_cg_close(const double* prr, const double* prz, int count,
                     Scalars* sc, int parity, hipStream_t s,
                     Scalars* pub = nullptr);
template <typename T>
void launch_convert(const double* in, T* out, int64_t n, hipStream_t s);

// the scalars of a residual: ||G(P)||^2 and the r.r, r.z of the CG start
// from 3 x count partials, ||P||^2 and <P>; pub: as for launch_cg_close
void launch_reduce_residual(const double* part, int count, const double* psum,
                            const double* psq, int nslab_sums, double invN3,
                            Scalars* sc, hipStream_t s, Scalars* pub = nullptr);
void launch_commit(const CommitArgs& a, hipStream_t s);
void launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
void launch_fill_f64(double* p, double v, int64_t n, hipStream_t s);
void launch_cauchy(const double* F, const double* P, double* sig, int64_t N,
                   hipStream_t s);
// the start of a CG run: its cap and tolerance, r.r and r.z of its start
void launch_init_scalars(Scalars* sc, int max_iters, double eta, double rr0,
                         double rz0, hipStream_t s);
void launch_bench_scalars(Scalars* sc, hipStream_t s);

// ---------------------------------------------------------- batch helpers
struct RedItem {
  const double* partial;   // 3 x count
  int count;
  const double* psum;
  const double* psq;
  int nss;
  double invN3;
};
// CG of a whole batch in one launch of resident blocks (grid barriers between
// passes); even / odd: the pass arguments of even and odd iterations
template <typename T>
struct BatchCG {
  BatchSpec<T> even, odd;
  Scalars* scs;
  int nitems;
  int blocksA, blocksB, blocksV;
  int max_iters;            // iterations of this launch at most
  unsigned* bar;            // barrier state (kBatchBarWords words, zero at
                            // start but for the generation)
  int* err;                 // set when a barrier waited past its bound
};
constexpr int kBatchBarWords = 32 * 10;
template <typename T>
void launch_cg_batch_persistent(const BatchCG<T>& c, int grid, size_t lds,
                                hipStream_t s);
// blocks of the persistent CG kernel that are resident at once
template <typename T>
int cg_batch_persistent_grid(size_t lds);
// the scalars of every active RVE's residual (launch_reduce_residual)
void launch_reduce_batch(const RedItem* items, int nitems, Scalars* scs,
                         hipStream_t s);
void launch_predict_batch(double* F, const double* Fprev, const uint8_t* vrve,
                          const double* dF /*[B][9]*/, int64_t N,
                          hipStream_t s);
struct CommitBatchArgs {
  const uint8_t* vrve;
  const Scalars* scs;
  const double* dF;   // [B][9] macro increments
  const double* F;    // Newton iterate (converged)
  const double* P;
  const double* Fpi_t;
  const double* chi_t;
  const double* dg_t;
  double* Fprev;
  double* Pc;
  double* Fpi_c;
  double* chi_c;
  double* dg_c;
  double* dFt;
  const int32_t* phase;
  const double* table;
  double* pcyc;
  double* pcyc_lit;
  double* wcyc;
  double dt;
  int64_t N;
};
void launch_commit_batch(const CommitBatchArgs& a, hipStream_t s);

// Device-side Newton control of a batch (Sec. 2.1): per RVE the record of
// its increment, written by the control kernel after each FP64 residual
constexpr int kBatchLog = 64;
struct BatchLog {
  int32_t status;        // 1 running, else RVE_OK / RVE_ENOTCONV / RVE_ELOCAL
  int32_t newton_iters;
  int32_t cg_total;
  int32_t breakdowns;
  int32_t fails;
  int32_t pad;
  double rel;            // last relative residual ||G(P)|| / ||P||
  double predictor_rel;
  double pbar[9];
  double res_hist[kBatchLog];
  int32_t cg_hist[kBatchLog];
};
struct NewtonCtl {
  double newton_tol, cg_tol;
  int32_t newton_max, cg_max, forcing;
};
// after the residual of Newton iteration it: book the previous solve's CG
// count, take the decision (commit, local failure, out of budget) and give
// running RVEs their linear-solve tolerance
void launch_newton_control_batch(Scalars* scs, BatchLog* log, int nitems,
                                 int it, const NewtonCtl& ctl, hipStream_t s);

}  // namespace rve
