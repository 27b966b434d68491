// Host runtime of libodwf: lattice and solver objects, workspaces, operator
// sequences built from the kernels, and the solvers.
#pragma once
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/odwf.h"
#include "kernels.h"
#include "odwf_types.h"

#define HIPRET(expr)                 \
  do {                               \
    hipError_t e_ = (expr);          \
    if (e_ != hipSuccess) return e_; \
  } while (0)

namespace odwf {

void set_error(const std::string& msg);

// a device buffer that the library owns
struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
};

// one half field (even or odd sites) in a storage precision
struct HV {
  void* d = nullptr;
  float* sc = nullptr;  // per-5D-site scales (FP16S / BF16S)
  int prec = PREC64;
};

size_t bytes_per_complex(int prec);
size_t half_bytes(long h, int nrhs, int Ns, int prec);   // data
size_t scale_bytes(long h, int nrhs, int Ns, int prec);  // scales (0 if unscaled)

// per-stream cache of named device buffers
struct Workspace {
  std::map<std::string, DevBuf> bufs;
  ~Workspace();
  void* get(const std::string& name, size_t bytes);
  HV half(const std::string& name, long h, int nrhs, int Ns, int prec);
  size_t total() const;
};

}  // namespace odwf

struct odwf_lattice_s {
  int dims[4];
  int bc_t;
  int device;
  odwf::Geom g;
  void* U64[2] = {nullptr, nullptr};  // per output parity, [h][8][18] double
  void* U32[2] = {nullptr, nullptr};  // per output parity, [h][8][12] float
  bool loaded = false;
};

struct odwf_solver_s {
  odwf_lattice lat;
  int Ns;
  double m0;
  std::vector<double> omega;
  void* coef64 = nullptr;  // [2][NCOEF][Ns] double; the block that holds the next two as well
  void* coef32 = nullptr;  // [2][NCOEF][Ns] float
  double* dense = nullptr; // [NDENSE][DENSE_LEN] dense programs (Ns <= 16)
  double dense_q[odwf::NDENSE][2] = {};  // their q per chirality
  double dense_w[odwf::NDENSE] = {};     // their sum of |w|, the larger of the chiralities
  std::mutex mtx;
  std::map<hipStream_t, odwf::Workspace*> ws;
  odwf::Workspace& workspace(hipStream_t st);
};

namespace odwf {

// programs of the fifth-dimension operators
M5Prog prog_none();
M5Prog prog_ainv();      // A^{-1}
M5Prog prog_ainv_t();    // A^{-dag} (A is real per chirality)
M5Prog prog_a();         // A
M5Prog prog_a_t();       // A^dag
M5Prog prog_omega();
M5Prog prog_omega_inv();
M5Prog prog_1pl();       // 1 + L
M5Prog prog_1pl_inv();   // (1 + L)^{-1}
M5Prog prog_1pl_t();     // (1 + L)^dag
M5Prog prog_ainv_winv(); // A^{-1} omega^{-1}
M5Prog prog_omega2();    // omega^2

// tables of the dense programs of a solver (host; Ns <= 16): tab [NDENSE][DENSE_LEN], q [NDENSE][2]
void dense_tables(int Ns, double m0, const double* omega, double* tab, double q[][2]);

// per-call operator context (one chunk of <= MAXRHS right-hand sides)
struct OpCtx {
  odwf_solver S;
  hipStream_t st;
  int prec;  // storage precision of the half fields passed to the helpers
  int nrhs;
  double kappa[MAXRHS];
  bool noprof = false;  // never record profiling events (the allocation-free path)
  const void* coef() const { return prec == PREC64 ? S->coef64 : S->coef32; }
  const void* links(int par) const { return prec == PREC64 ? S->lat->U64[par] : S->lat->U32[par]; }
  long h() const { return S->lat->g.h; }
  int Ns() const { return S->Ns; }
};

struct HopOpt {
  const HV* x = nullptr;
  M5Prog ph, px, po;
  double ch = 1.0, cx = 1.0;
  // CG fusion
  double* partial = nullptr;
  HV* cg_r = nullptr;
  const HV* cg_p = nullptr;  // f of the residual f - N p (mode 3)
  const CGScal* scal = nullptr;
  // alpha of the iteration from an earlier launch's partial sums, formed by an
  // extra block of this one (fin_scal: the records, copies behind them)
  const double* fin_partial = nullptr;
  CGScal* fin_scal = nullptr;
  // gating (GateMode): only right-hand sides selected by gate do any work
  const CGScal* gate = nullptr;
  int gate_mode = GATE_NONE;
  HopOpt() : ph(prog_none()), px(prog_none()), po(prog_none()) {}
};

hipError_t hop(const OpCtx& c, int out_par, int dag, const HV& in, const HV* out, const HopOpt& o);
// both output parities of an operator, each with the own parity's field as its x term (o.x is set here)
hipError_t hop_pair(const OpCtx& c, int dag, const HV& in_e, const HV& in_o, const HV& out_e, const HV& out_o,
                    HopOpt o);
// a program as the kernels take it: its dense form (table null: none) and its
// coefficients when it is a pure scaling (null: not one)
DenseArg dense_arg(const OpCtx& c, const M5Prog& p);
const double* diag_of(const OpCtx& c, const M5Prog& p);

// canonical <-> halves (null halves skipped / zeroed), each parity through its program
hipError_t pack(const OpCtx& c, const void* canon, int r0, const HV* e, const HV* o, const M5Prog& pe, const M5Prog& po);
hipError_t unpack(const OpCtx& c, const HV* e, const HV* o, void* canon, int r0, const M5Prog& p);
inline hipError_t pack(const OpCtx& c, const void* canon, int r0, const HV* e, const HV* o) {
  return pack(c, canon, r0, e, o, prog_none(), prog_none());
}

hipError_t m5(const OpCtx& c, const HV& in, const HV& out, const M5Prog& p);

// profiler hooks
void prof_begin(hipStream_t st, int key);
void prof_end(hipStream_t st, double bytes);
bool prof_on();

}  // namespace odwf
