// Plain data types shared by the host runtime and the HIP kernels of libodwf.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace odwf {

constexpr int MAXRHS = 16;  // right-hand sides per multi-RHS launch
// reliable-update trigger of the FP32 inner CG: recompute the true residual in
// FP64 once the iterated |r| falls below delta * max |r| since the last update;
// delta = 0.01 (measured at 64^3 x 64 x 16: the same iteration count as 0.1
// with half the updates; 0.001 starts to add iterations)
constexpr double RELIABLE_DELTA2 = 1e-4;
// right-hand sides per launch for a given Ns (Ns * nrhs lanes per site <= 256)
inline int max_rhs_per_launch(int Ns) { return 256 / Ns < MAXRHS ? 256 / Ns : MAXRHS; }

enum Prec { PREC64 = 0, PREC32 = 1, PREC16 = 2, PRECB16 = 3 };

// ---- fifth-dimension programs ---------------------------------------------
// Each operator acting on the fifth dimension is a product of diagonal scalings
// and cyclic bidiagonal matrices (or their inverses) with corner factor kappa =
// -mu, applied per chirality in the chirality-local index order.
enum M5Type : int8_t {
  M5_NOP = 0,
  M5_SCALE = 1,     // y_s *= d_s
  M5_MUL_LO = 2,    // y_s = d_s y_s + e_s y_{s-1},  y_0 = d_0 y_0 + kappa e_0 y_{N-1}
  M5_SOLVE_LO = 3,  // inverse of MUL_LO; d holds the reciprocal diagonal
  M5_MUL_UP = 4,    // y_s = d_s y_s + e_s y_{s+1},  y_{N-1} = d y + kappa e_{N-1} y_0
  M5_SOLVE_UP = 5   // inverse of MUL_UP; d holds the reciprocal diagonal
};

// coefficient arrays, each of length Ns, per chirality (chirality - mirrored)
enum CoefId : int8_t {
  CF_ONE = 0,       // 1
  CF_MONE = 1,      // -1
  CF_OMEGA = 2,     // omega_s
  CF_OMEGA_INV = 3, // 1 / omega_s
  CF_A = 4,         // a_s = (4 - m0) omega_s + 1
  CF_A_INV = 5,     // 1 / a_s
  CF_C = 6,         // c_s = (4 - m0) omega_s - 1
  CF_CSHIFT = 7,    // c_{s+1} (s < N-1), c_0 at s = N-1
  CF_OMEGA2 = 8,    // omega_s^2
  NCOEF = 9
};

struct M5Op {
  int8_t type, d, e, pad;
};
struct M5Prog {
  int n;
  int dense;  // DenseId of the same operator as a dense matrix, or -1 (a scaling, or no program)
  M5Op op[4];
};

// ---- the same programs as dense matrices -------------------------------------
// For N_s <= 16 every program with bidiagonal factors is also held as
//     M(kappa) = M0 + rho u w^T,   rho = kappa / (1 + kappa q),
// with M0, u, w and q independent of the mass: kappa enters each factor only
// through its corner entry (a rank-1 term), and the rank-1 terms of a product
// of a factor and the inverse of another share their row vector
// (Sherman-Morrison).  Tables of 16 x 16 (N_s < 16: block-diagonal copies), in
// slice order for both chiralities, FP64.
enum DenseId : int {
  DN_AINV = 0,    // A^{-1}
  DN_AINV_T = 1,  // A^{-T}
  DN_A = 2,       // A
  DN_A_T = 3,     // A^T
  DN_1PL = 4,     // 1 + L
  DN_1PL_T = 5,   // (1 + L)^T
  DN_1PL_INV = 6, // (1 + L)^{-1}
  DN_AINV_WINV = 7, // A^{-1} omega^{-1}
  NDENSE = 8
};
constexpr int DENSE_N = 16;
constexpr int DENSE_CHI = DENSE_N * DENSE_N + 2 * DENSE_N;  // M0, u, w of one chirality
constexpr int DENSE_LEN = 2 * DENSE_CHI;                    // both chiralities
inline bool dense_ns(int Ns) { return Ns <= DENSE_N; }

// ---- CG scalars, one record per right-hand side ----------------------------
struct CGScal {
  double rr;      // |r|^2 of the iterated residual
  double pAp;     // <p, N p> = |S p|^2
  double alpha;   // step length of the current iteration (0 when inactive)
  double beta;    // search-direction factor (0 when inactive)
  double f2;      // |f|^2 of the right-hand side of the iterated system
  double tol2;    // tol^2
  double rmax2;   // max |r|^2 since the last reliable update (mixed solves)
  double delta2;  // reliable-update threshold factor squared (0: never)
  int active;     // 1 while iterating
  int converged;  // iterated residual reached tol
  int nan;        // NaN/Inf met
  int update;     // reliable update requested
  int iters;      // iterations done
  int maxiter;    // iteration cap
  int confirm;    // 1: iterated convergence or maxiter requests a true-residual update
  int nupd;       // true-residual (reliable) updates this right-hand side iterated into
  int upd_iters;  // iteration count at its last true-residual update
};

// Scalar arrays hold 2 * MAXRHS records: the current ones, and from MAXRHS on
// the copies that get this iteration's alpha.  The current records do not change
// until beta: the launch that forms alpha still reads their gates, and the step
// forms beta from the copies alone, so any block of it may do so at any time
// while one of them writes the current record.
constexpr int SCAL_COPY = MAXRHS;

// which right-hand sides a gated kernel works on
enum GateMode { GATE_NONE = 0, GATE_ACTIVE = 1, GATE_UPDATE = 2 };

struct KappaArr {
  double v[MAXRHS];  // per right-hand side: -mu_r
};

// a dense program of a launch: table (null: none) and rho per chirality and
// right-hand side
struct DenseArg {
  const double* tab;
  double rho[2 * MAXRHS];
  // inputs whose reals stay below this (FP64, FP32 arithmetic) keep rho w^T x finite;
  // NaN where a rho is not finite itself (a singular mass)
  double lim64;
  float lim32;
};

// division of 0 <= n < 2^31 by a fixed 1 <= d < 2^31 as a multiplication:
// with l = ceil(log2 d) and m = floor(2^(31 + l) / d) + 1, n / d = n m >> (31 + l)
struct FastDiv {
  uint32_t m, sh, d;
  FastDiv() = default;
  explicit FastDiv(uint32_t dd) {
    uint32_t l = 0;
    while ((uint64_t(1) << l) < dd) l++;
    d = dd;
    sh = 31 + l;
    m = (uint32_t)((uint64_t(1) << sh) / dd + 1);
  }
#ifdef __HIPCC__
  __host__ __device__
#endif
  uint32_t div(uint32_t n) const { return (uint32_t)(((uint64_t)n * m) >> sh); }
};

// ---- arguments of the fused hopping kernel ----------------------------------
// fields of one output parity
struct HopIo {
  const void* in;
  const float* in_sc;
  const void* links;
  const void* xin;
  const float* xin_sc;
  void* out;
  float* out_sc;
  int out_par;
};
struct HopArgs {
  const void* in;       // opposite-parity input half
  const float* in_sc;
  const void* links;    // links of the output parity
  void* out;            // output half
  float* out_sc;
  const void* xin;      // same-parity input for the x term
  const float* xin_sc;
  // fused CG residual update (CG mode 2): r -= alpha out, |r|^2; cg_p is the
  // right-hand side f of a residual f - out (CG mode 3)
  void* cg_r;
  float* cg_r_sc;
  const void* cg_p;
  const float* cg_p_sc;
  const CGScal* scal;
  double* partial;      // per block, per right-hand side
  // a finished launch's partial sums that block 0 of this one (an extra block)
  // turns into the step lengths alpha while the others work (null: no such block)
  const double* fin_partial;
  int fin_nblocks;
  CGScal* fin_scal;
  const void* coef;     // [2][NCOEF][Ns], compute precision
  double kappa[MAXRHS]; // per right-hand side: -mu_r
  // fifth-dimension programs on the hopping result (h), the x term (x) and the
  // combination (o): N_s <= 16 takes the dense forms (o may be a scaling,
  // diag_o), N_s = 32 the factored ones
  DenseArg dn_h, dn_x, dn_o;
  const double* diag_o;
  M5Prog prog_h, prog_x, prog_o;
  double c_h, c_x;      // combination c_h * prog_h(W in) + c_x * prog_x(x)
  int h, nrhs, spb, out_par, bc_t, dag;
  int plain;  // the hop alone: no program, x term, factor or partial sums
  int rows;   // every block is a segment of one x-row
  int small;  // four waves to 64 lanes of sites
  int pair;   // (small) blockIdx.y = 1 works on `other`, the other output parity of the same operator
  HopIo other;
  int L[4];
  int nblocks;
  // block traversal: xcd != 0 gives each of the 8 XCDs a contiguous range of
  // logical blocks, xcd = 2 walks groups of 8 adjacent (y, z) tiles with one
  // tile per XCD in lockstep; tile_y, tile_z > 0 walk (x-row segments,
  // y, z) tiles with t innermost so that t-neighbours are re-read while still
  // in L2; tile_x > 0 is the number of x-row segments of a tile (all of the
  // row when 0); tile_t > 0 cuts t into chunks of that length, each chunk
  // walking all tiles before the next chunk starts
  int xcd, tile_y, tile_z, tile_t, tile_x;
  int xcd_gy;  // xcd = 2: tiles of a lockstep group along y (1, 2, 4 or 8)
  // divisors of the index arithmetic, set with the launch geometry: L_x / 2, L_y,
  // L_z; of the tiled walk: segments and rows of a tile, t slices, blocks of a
  // tile, and tiles (xcd = 2: groups of tiles) along y, z and x
  FastDiv d_hx, d_y, d_z, d_tx, d_ty, d_tz, d_tl, d_per, d_ny, d_nz, d_nx;
  // gating: lanes of right-hand sides not selected by gate_mode do no work
  const CGScal* gate;
  int gate_mode;
};

}  // namespace odwf
