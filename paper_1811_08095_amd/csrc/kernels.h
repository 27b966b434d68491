// Host-side launchers of the libodwf HIP kernels.  All launches are
// asynchronous on the given stream; they return the launch status.
#pragma once
#include <hip/hip_runtime.h>

#include "odwf_types.h"

namespace odwf {

struct Geom {
  int L[4];  // Lx, Ly, Lz, Lt
  long V, h;
};

inline Geom geom_of(const int dims[4]) {
  Geom g;
  for (int d = 0; d < 4; d++) g.L[d] = dims[d];
  g.V = (long)dims[0] * dims[1] * dims[2] * dims[3];
  g.h = g.V / 2;
  return g;
}

// hopping kernel (hop.hip)
hipError_t launch_hop(const HopArgs& a, int prec, int Ns, hipStream_t st);
// blocks of a fused launch (one partial sum per block and right-hand side), and
// sites per block of a launch
int hop_nblocks(const Geom& g, int nrhs, int Ns, int prec);
int hop_launch_spb(const Geom& g, int nrhs, int Ns, int prec, bool plain);
// the launch takes the four-wave kernel (plain reduced-precision hops never do)
bool hop_small(const Geom& g, int nrhs, int Ns, int prec);

// layouts (pack.hip)
// canonical complex128 [rhs][s][t][z][y][x][4][3] (rhs offset r0, nrhs of them)
// <-> internal halves, both parities in one launch, with a fifth-dimension
// operator per parity applied on the way (one dense program, N_s <= 16, or
// diagonal).  Packing skips a parity whose half is null; unpacking writes zeros
// on its sites.
struct HalfIO {
  void* d = nullptr;
  float* sc = nullptr;
  DenseArg dn = {nullptr, {}};
  const double* diag = nullptr;  // [2 chiralities, NCOEF * Ns apart][Ns], chirality - mirrored
};
hipError_t launch_pack(int prec, const void* canon, int r0, const HalfIO& e, const HalfIO& o, int nrhs, int Ns,
                       const Geom& g, hipStream_t st);
hipError_t launch_unpack(int prec, const HalfIO& e, const HalfIO& o, void* canon, int r0, int nrhs, int Ns,
                         const Geom& g, hipStream_t st);
// boundary maps of the effective 4D operator on canonical complex128 fields:
// embed 4D q [r][site][12] into 5D f [r][s][site][12] (chirality minus into
// slice 0, plus into slice Ns - 1, zeros elsewhere); project back
hipError_t launch_boundary_embed(const void* q, void* f, int nrhs, int Ns, const Geom& g, hipStream_t st);
hipError_t launch_boundary_project(const void* f, void* q, int nrhs, int Ns, const Geom& g, hipStream_t st);
// gauge: canonical complex128 [t][z][y][x][mu][3][3] -> link arrays of both
// parities, [h][8][18 doubles] and [h][8][12 floats]
hipError_t launch_pack_gauge(const void* canon, void* const out64[2], void* const out32[2], const Geom& g,
                             hipStream_t st);

// fifth-dimension programs on a half field (m5.hip):
// out = prog(in), from its dense form dn for N_s <= 16
hipError_t launch_m5(int prec, const void* in, const float* in_sc, void* out, float* out_sc, const M5Prog& prog,
                     const DenseArg& dn, const void* coef, const KappaArr& kappa, long h, int nrhs, int Ns,
                     hipStream_t st);

// BLAS-1 on half fields (blas.hip); n5 = h * nrhs * Ns five-dimensional sites
// gate / gate_mode (GateMode) restrict the work to selected right-hand sides
hipError_t launch_vec_zero(int prec, void* v, float* sc, long h, int nrhs, int Ns, hipStream_t st);
// dst = src, converting storage precision: FP64 to FP32 or a copy, which may be
// gated, or between FP64 and a scaled format (accumulate: dst += src)
hipError_t launch_vec_convert(int prec_src, const void* src, const float* src_sc, int prec_dst,
                              void* dst, float* dst_sc, int accumulate, long h, int nrhs, int Ns,
                              hipStream_t st, const CGScal* gate = nullptr, int gate_mode = GATE_NONE);
// y (FP64) += x (FP32), and x = 0 behind it
hipError_t launch_vec_flush(void* x, void* y, long h, int nrhs, int Ns, hipStream_t st);
// one right-hand side of a field into one right-hand side of another (zeros if src null)
hipError_t launch_vec_copy_rhs(int prec_src, const void* src, const float* src_sc, int nrhs_src,
                               int r_src, int prec_dst, void* dst, float* dst_sc, int nrhs_dst,
                               int r_dst, long h, int Ns, hipStream_t st);
// End of a CG iteration: beta_r and the convergence decisions from the partial
// |r|^2 (nblocks blocks) and the records' copies (SCAL_COPY), into the records
// and, when host is given, their pinned mirror; then x += alpha_r p for
// right-hand sides that iterated, p = r + beta_r p for the active ones and, with
// y (FP32: the FP64 solution), y += x, x = 0 for those that asked for an update.
hipError_t launch_cg_step(int prec, const void* r, const float* r_sc, void* p, float* p_sc, void* x, float* x_sc,
                          void* y, const double* partial, int nblocks, CGScal* scal, CGScal* host, long h, int nrhs,
                          int Ns, hipStream_t st);
// per-block partial sums of |v|^2 per right-hand side
hipError_t launch_vec_norm2(int prec, const void* v, const float* sc, double* partial, long h,
                            int nrhs, int Ns, int* nblocks_out, hipStream_t st);
int vec_nblocks(long h, int nrhs, int Ns);

// fermion force of Re <chi, W psi> on all links (force.hip): chi, psi canonical
// [s][t][z][y][x][4][3] complex128, links the FP64 links by parity, F canonical
// [t][z][y][x][mu][3][3]
hipError_t launch_force(const void* chi, const void* psi, const void* const links[2], void* F, int Ns, int bc_t,
                        int accumulate, const Geom& g, hipStream_t st);

// scalar finalisation (blas.hip), one block
enum FinKind { FIN_SUM = 0, FIN_BETA = 2, FIN_INIT = 3, FIN_F2 = 4 };
// bytes a partial-sum buffer for nblocks blocks needs (includes the second
// reduction stage used for long partial arrays)
size_t partial_bytes(int nblocks, int nrhs);
// gated != 0: only right-hand sides whose update flag is set are finalised
hipError_t launch_fin(int kind, const double* partial, int nblocks, int nrhs, CGScal* scal,
                      double* out, hipStream_t st, int gated = 0, CGScal* host = nullptr);

}  // namespace odwf
