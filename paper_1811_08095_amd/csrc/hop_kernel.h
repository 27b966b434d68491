// Even-odd hopping kernel ("Dslash") of the optimal domain-wall operator with
// fused fifth-dimension epilogues and fused CG updates.
//
// Computes, for every site x of the output parity, right-hand side r and slice s,
//     (W psi)(x, s) = -1/2 sum_mu [ (1 - gamma_mu) U_mu(x) psi(x + mu, s)
//                                 + (1 + gamma_mu) U_mu(x - mu)^dag psi(x - mu, s) ]
// (the hopping part of the 4D Wilson operator D_w of §2 with H = H_w; the
// adjoint W^dag swaps the two projectors), hops across the t boundary
// multiplied by bc_t, then
//     y = c_h * P_h(W psi) + c_x * P_x(x_site),   out = P_o(y)
// where P_h, P_x, P_o are fifth-dimension programs (A^{-1}, A^{-dag}, A^dag, ...
// as products of cyclic bidiagonal factors), and optionally the fused CG
// residual step r -= alpha y with its |r|^2 partial sums.
//
// Thread layout: a block holds spb sites of the output parity; each site has
// nrhs * Ns lanes (s fastest) that read consecutive 16-byte chunks of every
// neighbour.  The 8 links of the block's sites are staged once in LDS and
// shared by all nrhs * Ns lanes of a site (links are stored per output parity
// as [site][8][...] with directions 0-3 forward U_mu(x) and 4-7 backward
// U_mu(x - mu)^dag).  Fifth-dimension programs are dense N_s x N_s matrices per
// chirality on the matrix cores for N_s <= 16 (dense_apply), and run on LDS
// columns (site, r, colour-spin component) for N_s = 32.  The stencil itself is a
// string of 3x3 complex mat-vecs on the vector units.  Its time is set by the L2
// misses (FP64, FP32: 5.3 - 6.6 TB/s), with L1 passes and vector instructions
// close behind, or by vector instructions (FP16, BF16 storage).
#pragma once
#include <algorithm>
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"

namespace odwf {

// --- link formats ---------------------------------------------------------

template <class P>
struct LinkFmt;
// FP64: 18 reals = 9 complex doubles per matrix
template <>
struct LinkFmt<SP64> {
  static constexpr int REALS = 18;
  using R = double;
};
// reduced precisions: 12 reals (rows 0, 1) as floats, row 2 rebuilt as
// conj(row0 x row1), valid for SU(3)
struct LinkF12 {
  static constexpr int REALS = 12;
  using R = float;
};
template <>
struct LinkFmt<SP32> : LinkF12 {};
template <>
struct LinkFmt<SP16> : LinkF12 {};
template <>
struct LinkFmt<SPB16> : LinkF12 {};

// stage the links of `nsb` sites starting at j0 into LDS as 9 complex per
// matrix, times -1/2 (the factor of the hopping term: a power of two, so the
// hop sums round exactly as with the factor applied at the end)
template <class P>
__device__ __forceinline__ void stage_links(const void* links, long j0, int nsb,
                                            cpx<typename P::real>* lnk, int tid) {
  using R = typename P::real;
  const int nmat = nsb * 8;
  if constexpr (LinkFmt<P>::REALS == 18) {
    // flat copy of 16-byte chunks (one complex double each)
    const uint4* src = reinterpret_cast<const uint4*>(links) + j0 * 8 * 9;
    // five chunks of a thread in flight (all of them at Ns = 16: a round trip,
    // not one per chunk)
    constexpr int K = 5;
    for (int q0 = tid; q0 < nmat * 9; q0 += K * blockDim.x) {
      uint4 v[K];
#pragma unroll
      for (int k = 0; k < K; k++) v[k] = src[min(q0 + k * (int)blockDim.x, nmat * 9 - 1)];
#pragma unroll
      for (int k = 0; k < K; k++) {
        const int q = q0 + k * blockDim.x;
        cpx<double> z;
        unpack_chunk<SP64>(v[k], &z);
        if (q < nmat * 9) lnk[q] = cscale(-0.5, z);
      }
    }
  } else {
    const float4* src = reinterpret_cast<const float4*>(links) + j0 * 8 * 3;
    for (int m = tid; m < nmat; m += blockDim.x) {
#if ODWF_NT_LINKS
      // links are read once per launch: keep them from displacing spinor rows in L2
      typedef float f32x4 __attribute__((ext_vector_type(4)));
      const f32x4* sv = reinterpret_cast<const f32x4*>(src + m * 3);
      const f32x4 av = __builtin_nontemporal_load(sv), bv = __builtin_nontemporal_load(sv + 1),
                  cv = __builtin_nontemporal_load(sv + 2);
      float4 a = make_float4(av.x, av.y, av.z, av.w), b = make_float4(bv.x, bv.y, bv.z, bv.w),
             c = make_float4(cv.x, cv.y, cv.z, cv.w);
#else
      float4 a = src[m * 3 + 0], b = src[m * 3 + 1], c = src[m * 3 + 2];
#endif
      cpx<float> u[6] = {{a.x, a.y}, {a.z, a.w}, {b.x, b.y}, {b.z, b.w}, {c.x, c.y}, {c.z, c.w}};
      cpx<R>* d = lnk + m * 9;
#pragma unroll
      for (int k = 0; k < 6; k++) d[k] = cscale(-0.5f, u[k]);
      // row2[a] = conj(row0[b] row1[c] - row0[c] row1[b]), (a, b, c) cyclic
#pragma unroll
      for (int a0 = 0; a0 < 3; a0++) {
        const int b0 = (a0 + 1) % 3, c0 = (a0 + 2) % 3;
        cpx<float> t = csub(cmul(u[b0], u[3 + c0]), cmul(u[c0], u[3 + b0]));
        d[6 + a0] = {-0.5f * t.re, 0.5f * t.im};
      }
    }
  }
}

// neighbour scales of the FP16S/BF16S formats folded into the accumulating
// fma (1, default) or multiplied into the link product first (0)
#ifndef ODWF_SCALE_IN_FMA
#define ODWF_SCALE_IN_FMA 1
#endif

// acc += [g; -SIG B^dag g]; (B^dag g)_b = conj(f_{p_b}) g_{p_b}
template <int MU, int SIG, class R>
__device__ __forceinline__ void reconstruct(const cpx<R> (&g)[6], cpx<R> (&acc)[12]) {
  using B = GammaB<MU>;
  // p is an involution here: p_b = p0 for b = 0, p1 for b = 1
  constexpr int q0 = B::p0, q1 = B::p1;
  constexpr int fq0 = (q0 == 0) ? B::f0 : B::f1;
  constexpr int fq1 = (q1 == 0) ? B::f0 : B::f1;
#pragma unroll
  for (int c = 0; c < 3; c++) {
    acc[c] = cadd(acc[c], g[c]);
    acc[3 + c] = cadd(acc[3 + c], g[3 + c]);
    cpx<R> l0 = mulf<ConjCode<fq0>::v>(g[q0 * 3 + c]);
    cpx<R> l1 = mulf<ConjCode<fq1>::v>(g[q1 * 3 + c]);
    if constexpr (SIG > 0) {
      acc[6 + c] = csub(acc[6 + c], l0);
      acc[9 + c] = csub(acc[9 + c], l1);
    } else {
      acc[6 + c] = cadd(acc[6 + c], l0);
      acc[9 + c] = cadd(acc[9 + c], l1);
    }
  }
}

// the same with every term scaled by sc, the per-site scale of a neighbour
// stored with one: acc += sc [g; -SIG B^dag g], each real one fma
template <int MU, int SIG>
__device__ __forceinline__ void reconstruct_scaled(const cpx<float> (&g)[6], float sc, cpx<float> (&acc)[12]) {
  using B = GammaB<MU>;
  constexpr int q0 = B::p0, q1 = B::p1;
  constexpr int fq0 = (q0 == 0) ? B::f0 : B::f1;
  constexpr int fq1 = (q1 == 0) ? B::f0 : B::f1;
  const float sl = SIG > 0 ? -sc : sc;  // the lower components enter with -SIG
#pragma unroll
  for (int c = 0; c < 3; c++) {
    acc[c] = {fmaf(sc, g[c].re, acc[c].re), fmaf(sc, g[c].im, acc[c].im)};
    acc[3 + c] = {fmaf(sc, g[3 + c].re, acc[3 + c].re), fmaf(sc, g[3 + c].im, acc[3 + c].im)};
    const cpx<float> l0 = mulf<ConjCode<fq0>::v>(g[q0 * 3 + c]);
    const cpx<float> l1 = mulf<ConjCode<fq1>::v>(g[q1 * 3 + c]);
    acc[6 + c] = {fmaf(sl, l0.re, acc[6 + c].re), fmaf(sl, l0.im, acc[6 + c].im)};
    acc[9 + c] = {fmaf(sl, l1.re, acc[9 + c].re), fmaf(sl, l1.im, acc[9 + c].im)};
  }
}

// g = U h for both spins of the half spinor
template <class R>
__device__ __forceinline__ void su3_mul(const cpx<R>* __restrict__ U, const cpx<R> (&h)[6],
                                        cpx<R> (&g)[6]) {
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const cpx<R> u0 = U[a * 3 + 0], u1 = U[a * 3 + 1], u2 = U[a * 3 + 2];
#pragma unroll
    for (int sp = 0; sp < 2; sp++) {
      cpx<R> v = cmul(u0, h[sp * 3 + 0]);
      v = cfma(u1, h[sp * 3 + 1], v);
      v = cfma(u2, h[sp * 3 + 2], v);
      g[sp * 3 + a] = v;
    }
  }
}

// one hop: acc += [g; -SIG B^dag g] with g = U (psi_up - SIG B psi_dn)
template <int MU, int SIG, class R>
__device__ __forceinline__ void hop_one(const cpx<R> (&psi)[12], const cpx<R>* U, cpx<R> (&acc)[12]) {
  cpx<R> h[6], g[6];
  project<MU, SIG>(psi, h);
  su3_mul(U, h, g);
  reconstruct<MU, SIG>(g, acc);
}

// the same hop for a neighbour stored with a per-site scale: the projection and
// the link product are linear, so the scale enters only where the terms are
// accumulated (one fma per real instead of a product and a sum)
template <int MU, int SIG, class R>
__device__ __forceinline__ void hop_one_scaled(const cpx<R> (&psi)[12], R sc, const cpx<R>* U,
                                               cpx<R> (&acc)[12]) {
  cpx<R> h[6], g[6];
  project<MU, SIG>(psi, h);
  su3_mul(U, h, g);
  if constexpr (ODWF_SCALE_IN_FMA && sizeof(R) == 4) {
    reconstruct_scaled<MU, SIG>(g, sc, acc);
  } else {
#pragma unroll
    for (int k = 0; k < 6; k++) g[k] = cscale(sc, g[k]);
    reconstruct<MU, SIG>(g, acc);
  }
}

// first site of this block under the configured traversal
//
// Tiled walk (tile_y, tile_z > 0): a tile is tile_x x-row segments (of spb
// half-row sites) by tile_y by tile_z rows, walked segment-fastest, then y, z,
// with t innermost over tile_t slices (all of t when 0), so that the t
// neighbours a slice reads were fetched by the slices just before it.
// xcd = 1: hardware dispatches block b to XCD b % 8; XCD x is given the
// contiguous logical range [start(x), start(x) + count(x)), one run of tiles
// per XCD.  xcd = 2 (lockstep): the eight XCDs walk the eight tiles of a
// group of xgy (y) x 8 / xgy (z) adjacent tiles at the same time, block for
// block, so the halo rows two XCDs share are fetched by both at about the same
// time and the second read is served by the memory-side cache.
__device__ __forceinline__ uint32_t block_first_site(const HopArgs& a, uint32_t lb) {
  auto split = [](uint32_t& n, const FastDiv& d) {  // n mod d, n <- n / d
    const uint32_t q = d.div(n), r = n - q * d.d;
    n = q;
    return r;
  };
  const uint32_t hx = a.d_hx.d;
  if (a.xcd == 1) {
    const uint32_t q = a.nblocks >> 3, rem = a.nblocks & 7;
    const uint32_t x = lb & 7, k = lb >> 3;
    lb = x * q + min(x, rem) + k;
  }
  if (a.tile_y == 0) return lb * a.spb;
  uint32_t seg, y, z, t;
  if (a.xcd == 2) {
    const uint32_t x = lb & 7;
    uint32_t grp = lb >> 3;
    uint32_t r2 = split(grp, a.d_per);
    const uint32_t gy = x & (a.xcd_gy - 1), gz = x / a.xcd_gy;  // this XCD's tile in the group
    seg = split(r2, a.d_tx);
    y = split(r2, a.d_ty);
    z = split(r2, a.d_tz);
    t = r2;
    // groups: xgy x xgz tiles in (y, z), then x tiles, then t chunks
    y += (split(grp, a.d_ny) * a.xcd_gy + gy) * a.tile_y;
    z += (split(grp, a.d_nz) * (8 / a.xcd_gy) + gz) * a.tile_z;
    seg += split(grp, a.d_nx) * a.d_tx.d;
    t += grp * a.d_tl.d;
  } else {
    uint32_t rest = lb;
    seg = split(rest, a.d_tx);
    y = split(rest, a.d_ty);
    z = split(rest, a.d_tz);
    t = split(rest, a.d_tl);
    y += split(rest, a.d_ny) * a.tile_y;
    z += split(rest, a.d_nz) * a.tile_z;
    seg += split(rest, a.d_nx) * a.d_tx.d;
    t += rest * a.d_tl.d;
  }
  return ((t * a.d_z.d + z) * a.d_y.d + y) * hx + seg * a.spb;
}

#ifndef ODWF_HOP_GROUP64
#define ODWF_HOP_GROUP64 2
#endif
#ifndef ODWF_HOP_GROUP32
#define ODWF_HOP_GROUP32 2
#endif

// neighbour loads issued together before any of them is used: enough bytes
// in flight per wave to cover HBM latency at the occupancy the kernel reaches
template <class P>
struct HopGroup {
  static constexpr int G = sizeof(typename P::real) == 8 ? ODWF_HOP_GROUP64 : ODWF_HOP_GROUP32;
};

// the fused epilogue's own-site streams (x term, CG residual, output) are read
// or written once per launch: nontemporal (1, default), so that they do not
// displace the neighbour rows the hop re-reads from L2; 0: plain accesses
#ifndef ODWF_NT_FUSED
#define ODWF_NT_FUSED 1
#endif

// LDS of the fused epilogue's programs: dense images (N_s <= 16), one per
// program, or the column buffer (N_s = 32)
template <class R>
struct ProgLds {
  R* h;
  R* x;
  R* o;
  R* scr;  // the wave's scratch (dense programs)
};
// the fused epilogue's x term: transformed in LDS before the hop (N_s = 32), or
// loaded (and transformed) here
enum XMode { X_LDS = 1, X_LOAD = 2 };

__device__ __forceinline__ HopIo first_io(const HopArgs& a) {
  return {a.in, a.in_sc, a.links, a.xin, a.xin_sc, a.out, a.out_sc, a.out_par};
}

// what the epilogue reads, loaded ahead of the hop where registers allow
// (small launches): x term, CG residual or f, rho per program and chirality
template <class P, int NS>
__device__ __forceinline__ void tail_preload(const HopArgs& a, const HopIo& io, bool valid, long j, int r, int s,
                                             cpx<typename P::real> (&xv)[12], cpx<typename P::real> (&rv)[12],
                                             typename P::real (&rho)[6], typename P::real& alpha, bool& cg_update) {
  using R = typename P::real;
#pragma unroll
  for (int chi = 0; chi < 2; chi++) {  // zeros where there is no program
    rho[chi] = (R)a.dn_h.rho[chi * MAXRHS + r];
    rho[2 + chi] = (R)a.dn_x.rho[chi * MAXRHS + r];
    rho[4 + chi] = (R)a.dn_o.rho[chi * MAXRHS + r];
  }
  cg_update = a.partial && a.cg_r && valid && a.scal[r].active;
  alpha = cg_update ? (R)a.scal[r].alpha : R(0);
  if (io.xin && valid) load_site<P, ODWF_NT_FUSED, false>(io.xin, io.xin_sc, j, r, s, a.nrhs, NS, xv);
  if (cg_update || (a.partial && !a.cg_r && a.cg_p && valid)) {
    const bool upd = a.cg_r != nullptr;
    load_site<P, ODWF_NT_FUSED, false>(upd ? a.cg_r : a.cg_p, upd ? a.cg_r_sc : a.cg_p_sc, j, r, s, a.nrhs, NS, rv);
  }
}

// Fused epilogue of one output site after the hop: the fifth-dimension
// programs, the x term, the norm for the partial sums, and the residual, the CG
// update or the store.  Every thread of the block calls it (whole waves enter
// the matrix instructions; the column passes of N_s = 32 synchronise the
// block); returns this lane's share of the partial sum.
template <class P, int NS, bool PRE>
__device__ __forceinline__ double fused_tail(const HopArgs& a, const HopIo& io, cpx<typename P::real> (&acc)[12], bool valid,
                                             long j, int sl, int r, int s, int nsb,
                                             const ProgLds<typename P::real>& pl, const typename P::real* kap,
                                             int xmode, cpx<typename P::real> (&xv)[12],
                                             cpx<typename P::real> (&rv)[12], const typename P::real (&rho)[6],
                                             typename P::real alpha, bool cg_pre, int tid) {
  using R = typename P::real;
  constexpr int NSP = NS + 1;
  const int nrhs = a.nrhs;
  auto column = [&](cpx<R>* b, int c) -> cpx<R>& { return b[((size_t)(sl * nrhs + r) * 12 + c) * NSP + s]; };
  auto program = [&](int p, const DenseArg& dn, const M5Prog& prog, R* lds, cpx<R>(&v)[12]) {
    if constexpr (NS <= DENSE_N) {
      if (!dn.tab) return;
      if constexpr (PRE) dense_apply<NS, true>(v, lds, pl.scr, rho[2 * p], rho[2 * p + 1], dense_lim<R>(dn), tid);
      else dense_apply<NS>(v, lds, pl.scr, (R)dn.rho[r], (R)dn.rho[MAXRHS + r], dense_lim<R>(dn), tid);
    } else {
      if (prog.n == 0) return;
      cpx<R>* buf = reinterpret_cast<cpx<R>*>(lds);
      __syncthreads();
      if (valid) {
#pragma unroll
        for (int c = 0; c < 12; c++) column(buf, c) = v[c];
      }
      __syncthreads();
      column_pass_lds<R, NS>(buf, nsb, nrhs, prog, reinterpret_cast<const R*>(a.coef), kap, tid);
      __syncthreads();
      if (valid) {
#pragma unroll
        for (int c = 0; c < 12; c++) v[c] = column(buf, c);
      }
    }
  };

  program(0, a.dn_h, a.prog_h, pl.h, acc);  // N_s = 32: never together with X_LDS
  const int cgmode = a.partial ? (a.cg_r ? 2 : (a.cg_p ? 3 : 1)) : 0;
  const bool cg_update = PRE ? cg_pre : cgmode == 2 && valid && a.scal[r].active;
  bool r_loaded = PRE;
  const bool has_x = io.xin != nullptr;
  if (has_x) {
    if (xmode == X_LDS) {  // transformed before the hop, still in the column buffer
      if (valid) {
#pragma unroll
        for (int c = 0; c < 12; c++) xv[c] = column(reinterpret_cast<cpx<R>*>(pl.h), c);
      }
    } else {
      if constexpr (NS <= DENSE_N && !PRE) {
#pragma unroll
        for (int c = 0; c < 12; c++) xv[c] = {R(0), R(0)};
      }
      if (!PRE && valid) load_site<P, ODWF_NT_FUSED>(io.xin, io.xin_sc, j, r, s, nrhs, NS, xv);
      if constexpr (!PRE && sizeof(R) == 4 && NS <= DENSE_N && !P::SCALED) {
        // the CG residual travels with the x term: one memory round trip fewer
        if (cg_update) {
          load_site<P, ODWF_NT_FUSED>(a.cg_r, a.cg_r_sc, j, r, s, nrhs, NS, rv);
          r_loaded = true;
        }
      }
      program(1, a.dn_x, a.prog_x, pl.x, xv);
    }
  }
  if (has_x) {
    const R ch = (R)a.c_h, cx = (R)a.c_x;
#pragma unroll
    for (int c = 0; c < 12; c++) acc[c] = cadd(cscale(ch, acc[c]), cscale(cx, xv[c]));
  } else if (a.c_h != 1.0) {
    const R ch = (R)a.c_h;
#pragma unroll
    for (int c = 0; c < 12; c++) acc[c] = cscale(ch, acc[c]);
  }

  double nval = 0.0;
  if (cgmode == 1 && valid) {
#pragma unroll
    for (int c = 0; c < 12; c++) nval += (double)cnorm2(acc[c]);
  }
  program(2, a.dn_o, a.prog_o, pl.o, acc);
  if constexpr (NS <= DENSE_N) {
    if (a.diag_o) {
      const R p = (R)a.diag_o[s], m = (R)a.diag_o[NCOEF * NS + NS - 1 - s];
#pragma unroll
      for (int c = 0; c < 12; c++) acc[c] = cscale(c < 6 ? p : m, acc[c]);
    }
  }

  if (cgmode == 3 && valid) {  // residual: out = f - y
    cpx<R> f[12];
    if constexpr (PRE) {
#pragma unroll
      for (int c = 0; c < 12; c++) f[c] = rv[c];
    } else {
      load_site<P>(a.cg_p, a.cg_p_sc, j, r, s, nrhs, NS, f);
    }
#pragma unroll
    for (int c = 0; c < 12; c++) {
      acc[c] = csub(f[c], acc[c]);
      nval += (double)cnorm2(acc[c]);
    }
  }
  void* dst = io.out;
  float* dst_sc = io.out_sc;
  bool store = valid && io.out;
  if (cgmode == 2) {
    // x += alpha p runs in the vector step after beta (launch_cg_step),
    // which reads p there anyway
    dst = a.cg_r;
    dst_sc = a.cg_r_sc;
    store = cg_update;
    if (cg_update) {  // r -= alpha N p, |r|^2
      const R al = PRE ? alpha : (R)a.scal[r].alpha;
      if (!r_loaded) load_site<P, ODWF_NT_FUSED>(a.cg_r, a.cg_r_sc, j, r, s, nrhs, NS, rv);
#pragma unroll
      for (int c = 0; c < 12; c++) {
        acc[c] = csub(rv[c], cscale(al, acc[c]));
        nval += (double)cnorm2(acc[c]);
      }
    }
  }
  if (store) store_site<P, ODWF_NT_FUSED>(dst, dst_sc, j, r, s, nrhs, NS, acc);

  return nval;
}

// FP16 storage: the spin projection reads the stored halves directly.  Each
// real of h = psi_up -/+ f psi_dn (f in {+-1, +-i}) is one fma(+-1, dn, up) of
// the two halves (v_fma_mix_f32 converts and adds in one instruction); it
// rounds exactly as the sum of the converted values.  `one` is 1.0 held where
// the compiler cannot fold it (a product by the literal 1.0 would turn back
// into a conversion and an add).
template <int CODE, int SIG>
__device__ __forceinline__ cpx<float> proj_h16(uint32_t up, uint32_t dn, float one) {
  const __half2 u = *reinterpret_cast<const __half2*>(&up), d = *reinterpret_cast<const __half2*>(&dn);
  const float ur = __low2float(u), ui = __high2float(u), dr = __low2float(d), di = __high2float(d);
  const float m = SIG > 0 ? -one : one;  // h = up + m (f dn)
  if constexpr (CODE == 0) return {fmaf(m, dr, ur), fmaf(m, di, ui)};
  if constexpr (CODE == 1) return {fmaf(-m, dr, ur), fmaf(-m, di, ui)};
  if constexpr (CODE == 2) return {fmaf(-m, di, ur), fmaf(m, dr, ui)};
  return {fmaf(m, di, ur), fmaf(-m, dr, ui)};
}
template <int MU, int SIG>
__device__ __forceinline__ void hop_one_h16(const uint32_t (&w)[12], float sc, float one, const cpx<float>* U,
                                            cpx<float> (&acc)[12]) {
  using B = GammaB<MU>;
  cpx<float> h[6], g[6];
#pragma unroll
  for (int c = 0; c < 3; c++) {
    h[c] = proj_h16<B::f0, SIG>(w[c], w[(2 + B::p0) * 3 + c], one);
    h[3 + c] = proj_h16<B::f1, SIG>(w[3 + c], w[(2 + B::p1) * 3 + c], one);
  }
  su3_mul(U, h, g);
  if constexpr (ODWF_SCALE_IN_FMA) {
    reconstruct_scaled<MU, SIG>(g, sc, acc);
  } else {
#pragma unroll
    for (int k = 0; k < 6; k++) g[k] = cscale(sc, g[k]);
    reconstruct<MU, SIG>(g, acc);
  }
}
template <bool DAG>
__device__ __forceinline__ void hop_dir_h16(int dir, const uint32_t (&w)[12], float sc, float one,
                                            const cpx<float>* U, cpx<float> (&acc)[12]) {
  const bool minus = (dir < 4) != DAG;
  const cpx<float>* Ud = U + dir * 9;
  switch (dir & 3) {
    case 0: if (minus) hop_one_h16<0, +1>(w, sc, one, Ud, acc); else hop_one_h16<0, -1>(w, sc, one, Ud, acc); break;
    case 1: if (minus) hop_one_h16<1, +1>(w, sc, one, Ud, acc); else hop_one_h16<1, -1>(w, sc, one, Ud, acc); break;
    case 2: if (minus) hop_one_h16<2, +1>(w, sc, one, Ud, acc); else hop_one_h16<2, -1>(w, sc, one, Ud, acc); break;
    default: if (minus) hop_one_h16<3, +1>(w, sc, one, Ud, acc); else hop_one_h16<3, -1>(w, sc, one, Ud, acc); break;
  }
}

// one neighbour's hopping term: acc += (1 -/+ gamma_mu) U psi for the
// direction dir (0-3 forward, 4-7 backward); the scaled formats carry the
// neighbour's per-site scale sc separately
template <class P, bool DAG>
__device__ __forceinline__ void hop_dir(int dir, const cpx<typename P::real> (&psi)[12], typename P::real sc,
                                        const cpx<typename P::real>* U, cpx<typename P::real> (&acc)[12]) {
  // forward hop: (1 - gamma) for W, (1 + gamma) for W^dag; backward swapped
  const bool minus = (dir < 4) != DAG;
  const cpx<typename P::real>* Ud = U + dir * 9;
  if constexpr (P::SCALED) {
    switch (dir & 3) {
      case 0: if (minus) hop_one_scaled<0, +1>(psi, sc, Ud, acc); else hop_one_scaled<0, -1>(psi, sc, Ud, acc); break;
      case 1: if (minus) hop_one_scaled<1, +1>(psi, sc, Ud, acc); else hop_one_scaled<1, -1>(psi, sc, Ud, acc); break;
      case 2: if (minus) hop_one_scaled<2, +1>(psi, sc, Ud, acc); else hop_one_scaled<2, -1>(psi, sc, Ud, acc); break;
      default: if (minus) hop_one_scaled<3, +1>(psi, sc, Ud, acc); else hop_one_scaled<3, -1>(psi, sc, Ud, acc); break;
    }
  } else {
    switch (dir & 3) {
      case 0: if (minus) hop_one<0, +1>(psi, Ud, acc); else hop_one<0, -1>(psi, Ud, acc); break;
      case 1: if (minus) hop_one<1, +1>(psi, Ud, acc); else hop_one<1, -1>(psi, Ud, acc); break;
      case 2: if (minus) hop_one<2, +1>(psi, Ud, acc); else hop_one<2, -1>(psi, Ud, acc); break;
      default: if (minus) hop_one<3, +1>(psi, Ud, acc); else hop_one<3, -1>(psi, Ud, acc); break;
    }
  }
}

// a neighbour in registers.  FP16 stays packed until the projection (see
// proj_h16), in the row and the general path alike, so that a site's sum is the
// same bits in both; the plain hop of the general path unpacks first (PACKED =
// false): the compiler contracts the link products of the two forms differently,
// and a plain hop's bits in 16-bit storage do not change from one version to the next.
template <class P, bool PACKED = true>
struct Neighbour {
  static constexpr bool RAW16 = PACKED && std::is_same<P, SP16>::value;
  static constexpr bool RAW64 = std::is_same<P, SP64>::value;
  using Site = cpx<typename P::real>[12];
  using V = typename std::conditional<RAW16, uint32_t[12], typename std::conditional<RAW64, u32x4[12], Site>::type>::type;
  // keep the chunks of the site (FP64, FP16), or unpack them
  __device__ static __forceinline__ void set(V& v, const u32x4 (&q)[12 / P::CPB]) {
#pragma unroll
    for (int cg = 0; cg < 12 / P::CPB; cg++) {
      if constexpr (RAW64) {
        v[cg] = q[cg];
      } else if constexpr (RAW16) {
        v[cg * 4 + 0] = q[cg].x;
        v[cg * 4 + 1] = q[cg].y;
        v[cg * 4 + 2] = q[cg].z;
        v[cg * 4 + 3] = q[cg].w;
      } else {
        unpack_chunk<P>(make_uint4(q[cg].x, q[cg].y, q[cg].z, q[cg].w), &v[cg * P::CPB]);
      }
    }
  }
  __device__ static __forceinline__ void get(const V& v, Site& z) {  // FP64
#pragma unroll
    for (int c = 0; c < 12; c++) unpack_chunk<SP64>(whole_chunk(v[c]), &z[c]);
  }
  __device__ static __forceinline__ void negate(Site& z) {
#pragma unroll
    for (int c = 0; c < 12; c++) z[c] = {-z[c].re, -z[c].im};
  }
  // its hopping term, with the boundary sign of a wrapping t hop
  template <bool DAG>
  __device__ static __forceinline__ void apply(int dir, V& v, typename P::real sc, bool flip, float one,
                                               const cpx<typename P::real>* U, cpx<typename P::real> (&acc)[12]) {
    if (P::SCALED && flip) sc = -sc;
    if constexpr (RAW16) {
      hop_dir_h16<DAG>(dir, v, sc, one, U, acc);
    } else if constexpr (RAW64) {
      Site z;
      get(v, z);
      if (flip) negate(z);
      hop_dir<P, DAG>(dir, z, sc, U, acc);
    } else {
      if (!P::SCALED && flip) negate(v);
      hop_dir<P, DAG>(dir, v, sc, U, acc);
    }
  }
  // 1.0 where the compiler cannot fold it (see proj_h16)
  __device__ static __forceinline__ float opaque_one() {
    float one = 1.0f;
    if constexpr (RAW16) asm("s_mov_b32 %0, 1.0" : "=s"(one));
    return one;
  }
};

// Direction of the k-th term (4-7 are the backward hops).  FP64 takes -t first
// and +t last, -t +x -x +y -y +z -z +t: the slice behind was read longest ago,
// the slice ahead is what the next blocks read (17 % fewer L2 misses at
// 32^3 x 16 x 16, CG iteration 3340 -> 3285 us; 16^4 x 16, two right-hand sides,
// 831 -> 811 us).  FP32 spills in this order, FP16 gains nothing from it
// (32^3 x 16 1.6 % slower, 24^4 0.7 % faster): +x -x +y -y +z -z +t -t.
template <class P>
__device__ __forceinline__ int term_dir(int k) {
  if constexpr (sizeof(typename P::real) == 8) return k & 1 ? k >> 1 : 4 + (((k >> 1) + 3) & 3);
  else return (k >> 1) | ((k & 1) << 2);
}

// a block-uniform integer in a scalar register (the compiler does not always
// prove uniformity through the traversal arithmetic)
__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The eight hopping terms of output site j0 + sl of a block that lies inside
// one x-row (half-row length a multiple of the sites per block), summed into
// acc (the factor -1/2 rides on the staged links).  y, z, t and the parity of
// the row are then block-uniform: the seven neighbour rows (own row for the x
// hops, y +- 1, z +- 1, t +- 1) are scalar 64-bit bases, and a lane addresses a
// neighbour as base + one of three 32-bit offsets (own column, x + 1, x - 1)
// + a constant chunk offset, so the loads need almost no vector address
// arithmetic.  Terms are summed in the order of term_dir, the neighbours loaded G at a
// time ahead of their arithmetic.
template <class P, int NS, bool DAG, int G, bool PRE>
__device__ __forceinline__ void hop_sum_row(const HopArgs& a, int j0, int sl, int r, int s, bool valid,
                                            const cpx<typename P::real>* U, cpx<typename P::real> (&acc)[12]) {
  using R = typename P::real;
  constexpr int NCG = 12 / P::CPB;
  const int nrhs = a.nrhs;
  const int L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  const int hx = a.L[0] >> 1;
  const int jb = uniform_int(j0);
  const int row = a.d_hx.div(jb), xh0 = jb - row * hx;
  const int zt = a.d_y.div(row), y = row - zt * L1;
  const int t = a.d_z.div(zt), z = zt - t * L2;
  const int p = (y + z + t + a.out_par) & 1;
  const int yp = y + 1 == L1 ? 0 : y + 1, ym = y == 0 ? L1 - 1 : y - 1;
  const int zp = z + 1 == L2 ? 0 : z + 1, zm = z == 0 ? L2 - 1 : z - 1;
  const int tp = t + 1 == L3 ? 0 : t + 1, tm = t == 0 ? L3 - 1 : t - 1;
  // per lane: half-row column of the own site and of its x neighbours
  // (x + 1 lies in column xi (p = 0) or xi + 1 (p = 1); x - 1 in xi - 1 or xi)
  const int xi = xh0 + sl;
  const int xip = p ? (xi + 1 == hx ? 0 : xi + 1) : xi;
  const int xim = p ? xi : (xi == 0 ? hx - 1 : xi - 1);
  auto boff = [&](int q) { return (unsigned)((((q * nrhs + r) * NCG) * NS + s) * 16); };
  const unsigned off_own = boff(xi), off_xp = boff(xip), off_xm = boff(xim);
  const size_t row_bytes = (size_t)hx * nrhs * NCG * NS * 16;
  auto soff = [&](int q) { return (unsigned)(((q * nrhs + r) * NS + s) * 4); };
  const unsigned soff_own = soff(xi), soff_xp = soff(xip), soff_xm = soff(xim);
  const size_t srow_bytes = (size_t)hx * nrhs * NS * 4;
  const bool flip_f = a.bc_t < 0 && t + 1 == L3;  // forward t hop wraps
  const bool flip_b = a.bc_t < 0 && t == 0;       // backward t hop wraps
  const unsigned char* in = reinterpret_cast<const unsigned char*>(a.in);
  const unsigned char* in_sc = reinterpret_cast<const unsigned char*>(a.in_sc);
  using N = Neighbour<P>;
  using Nb = typename N::V;
  const float one = N::opaque_one();
  // neighbour of direction dir (0-3 forward, 4-7 backward) into v; sc its scale
  auto load_nb = [&](int dir, Nb& v, R& sc) {
    const int mu = dir & 3;
    const bool fwd = dir < 4;
    const int yy = mu == 1 ? (fwd ? yp : ym) : y;
    const int zz = mu == 2 ? (fwd ? zp : zm) : z;
    const int tt = mu == 3 ? (fwd ? tp : tm) : t;
    const int nrow = (tt * L2 + zz) * L1 + yy;  // block-uniform
    const unsigned off = mu == 0 ? (fwd ? off_xp : off_xm) : off_own;
    const unsigned char* base = in + (size_t)nrow * row_bytes;
    u32x4 q[NCG];
#pragma unroll
    for (int cg = 0; cg < NCG; cg++) q[cg] = *reinterpret_cast<const u32x4*>(base + off + cg * NS * 16);
    N::set(v, q);
    if constexpr (P::SCALED) {
      const unsigned so = mu == 0 ? (fwd ? soff_xp : soff_xm) : soff_own;
      sc = *reinterpret_cast<const float*>(in_sc + (size_t)nrow * srow_bytes + so);
    } else {
      sc = R(1);
    }
  };
  auto apply_nb = [&](int dir, Nb& v, R sc) {
    N::template apply<DAG>(dir, v, sc, (dir == 3 && flip_f) || (dir == 7 && flip_b), one, U, acc);
  };
  auto dir_of = [](int k) { return term_dir<P>(k); };
  Nb psi[G];
  R scl[G];
  if (PRE && valid) {
#pragma unroll
    for (int k = 0; k < G; k++) load_nb(dir_of(k), psi[k], scl[k]);
  }
  __syncthreads();  // the staged links
  if (!valid) return;
  // (a rolled loop: unrolled, the compiler issues the loads of later groups
  // early and spills them at the register budget of four waves per SIMD; a
  // software pipeline over two register buffers fits three waves and was
  // slower in the fused kernels)
#pragma unroll 1
  for (int g0 = 0; g0 < 8; g0 += G) {
    if constexpr (!PRE) {
#pragma unroll
      for (int k = 0; k < G; k++) load_nb(dir_of(g0 + k), psi[k], scl[k]);
    }
#pragma unroll
    for (int k = 0; k < G; k++) apply_nb(dir_of(g0 + k), psi[k], scl[k]);
    if constexpr (PRE) {
      if (g0 + G >= 8) break;
#pragma unroll
      for (int k = 0; k < G; k++) load_nb(dir_of(g0 + G + k), psi[k], scl[k]);
    }
  }
}

// The eight hopping terms of output site j, summed into acc (the factor -1/2
// rides on the staged links), for any block shape: the coordinates and the
// neighbour index are formed per lane.
template <class P, int NS, bool DAG, int G, bool PRE, bool PACKED>
__device__ __forceinline__ void hop_sum(const HopArgs& a, uint32_t j, int r, int s, bool valid,
                                        const cpx<typename P::real>* U, cpx<typename P::real> (&acc)[12]) {
  using R = typename P::real;
  const int nrhs = a.nrhs;
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  const int hx = L0 >> 1;
  const int row = a.d_hx.div(j), xh = j - row * hx;
  const int zt = a.d_y.div(row), y = row - zt * L1;
  const int t = a.d_z.div(zt), z = zt - t * L2;
  const int p = (y + z + t + a.out_par) & 1;
  const bool flip_f = a.bc_t < 0 && t + 1 == L3;  // forward t hop wraps
  const bool flip_b = a.bc_t < 0 && t == 0;       // backward t hop wraps
  using N = Neighbour<P, PACKED>;
  using Nb = typename N::V;
  const float one = N::opaque_one();
  Nb psi[G];
  R scl[G];  // per-site scales of the neighbours (scaled formats)
  auto dir_of = [](int k) { return term_dir<P>(k); };
  auto load_nb = [&](int dir, Nb& v, R& sc) {
    const int mu = dir & 3;
    const bool fwd = dir < 4;
    int xx = xh, yy = y, zz = z, tt = t;
    // x + 1 lies in column xh (p = 0) or xh + 1 (p = 1), x - 1 in xh - 1 or xh
    if (mu == 0 && fwd && p) xx = xh + 1 == hx ? 0 : xh + 1;
    if (mu == 0 && !fwd && !p) xx = xh == 0 ? hx - 1 : xh - 1;
    if (mu == 1) yy = fwd ? (y + 1 == L1 ? 0 : y + 1) : (y == 0 ? L1 - 1 : y - 1);
    if (mu == 2) zz = fwd ? (z + 1 == L2 ? 0 : z + 1) : (z == 0 ? L2 - 1 : z - 1);
    if (mu == 3) tt = fwd ? (t + 1 == L3 ? 0 : t + 1) : (t == 0 ? L3 - 1 : t - 1);
    const long nj = (long)((tt * L2 + zz) * L1 + yy) * hx + xx;
    constexpr int NCG = 12 / P::CPB;
    const u32x4* b = reinterpret_cast<const u32x4*>(a.in) + (nj * nrhs + r) * NCG * NS + s;
    u32x4 q[NCG];
#pragma unroll
    for (int cg = 0; cg < NCG; cg++) q[cg] = b[cg * NS];
    N::set(v, q);
    sc = P::SCALED ? R(a.in_sc[(nj * nrhs + r) * NS + s]) : R(1);
  };
  auto apply_nb = [&](int dir, Nb& v, R sc) {
    N::template apply<DAG>(dir, v, sc, (dir == 3 && flip_f) || (dir == 7 && flip_b), one, U, acc);
  };
  if (PRE && valid) {
#pragma unroll
    for (int k = 0; k < G; k++) load_nb(dir_of(k), psi[k], scl[k]);
  }
  __syncthreads();  // the staged links
  if (!valid) return;
#pragma unroll 1
  for (int g0 = 0; g0 < 8; g0 += G) {
    if constexpr (!PRE) {
#pragma unroll
      for (int k = 0; k < G; k++) load_nb(dir_of(g0 + k), psi[k], scl[k]);
    }
#pragma unroll
    for (int k = 0; k < G; k++) apply_nb(dir_of(g0 + k), psi[k], scl[k]);
    if constexpr (PRE) {
      if (g0 + G >= 8) break;
#pragma unroll
      for (int k = 0; k < G; k++) load_nb(dir_of(g0 + G + k), psi[k], scl[k]);
    }
  }
}

// minimum waves per SIMD the register allocation must allow
#ifndef ODWF_HOP_WAVES32
#define ODWF_HOP_WAVES32 4
#endif
#ifndef ODWF_HOP_WAVES64
#define ODWF_HOP_WAVES64 2
#endif
template <class P, int NS, bool PLAIN>
struct HopWaves {
  static constexpr int W =
      sizeof(typename P::real) == 8 ? ODWF_HOP_WAVES64 : ((PLAIN || NS <= DENSE_N) ? ODWF_HOP_WAVES32 : 2);
  static_assert(W >= 2, "above 256 registers the compiler takes accumulation registers (hop_small_kernel)");
};

// alpha of the iteration from the partial sums of an earlier launch, into the
// records' copies that the rest of the iteration works from (the records
// themselves stay: other blocks of this launch read their gates)
__device__ __forceinline__ void fin_block(const HopArgs& a, double* tmp) {
  const double v = partial_sum(a.fin_partial, a.fin_nblocks, a.nrhs, tmp);
  const int r = threadIdx.x;
  if (r >= a.nrhs) return;
  CGScal c = a.fin_scal[r];
  fin_alpha(c, v);
  a.fin_scal[SCAL_COPY + r] = c;
}

// one block's sites; tid: the thread's index in the block
template <class P, int NS, bool DAG, bool PLAIN>
__device__ __forceinline__ void hop_block(const HopArgs& a, uint32_t lb, int tid) {
  using R = typename P::real;
  constexpr bool DENSE = !PLAIN && NS <= DENSE_N;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nrhs = a.nrhs;
  const int col = tid / NS, s = tid - col * NS;  // column (site, right-hand side) of the block, and slice
  const int sl = nrhs == 1 ? col : col / nrhs;
  const int r = col - sl * nrhs;
  const uint32_t j0 = block_first_site(a, lb);
  const int nsb = min(a.spb, a.h - (int)j0);
  // padded threads have sl >= spb >= nsb; gated-off right-hand sides do no work
  const bool valid = sl < nsb && gate_on(a.gate, a.gate_mode, r);

  // LDS: links, programs (dense images or the column buffer), reduction scratch.
  // Links and column buffer are separate, so an x term can be transformed in
  // LDS while the links are staged and used (N_s = 32)
  cpx<R>* lnk = reinterpret_cast<cpx<R>*>(smem);
  R* prog = reinterpret_cast<R*>(lnk + (size_t)a.spb * 8 * 9);
  ProgLds<R> pl = {prog, prog, prog, nullptr};
  R* kap = nullptr;
  stage_links<P>(a.links, j0, nsb, lnk, tid);
  bool x_first = false;
  if constexpr (DENSE) {
    if (a.dn_h.tab) {
      dense_stage<R>(pl.h, a.dn_h.tab, tid);
      prog += DENSE_IMAGE<R>;
    }
    pl.x = prog;
    if (a.dn_x.tab) {
      dense_stage<R>(pl.x, a.dn_x.tab, tid);
      prog += DENSE_IMAGE<R>;
    }
    pl.o = prog;
    if (a.dn_o.tab) {
      dense_stage<R>(pl.o, a.dn_o.tab, tid);
      prog += DENSE_IMAGE<R>;
    }
    pl.scr = prog + (tid >> 6) * DENSE_SCRATCH<R>;
    prog += (blockDim.x >> 6) * DENSE_SCRATCH<R>;
  } else if constexpr (!PLAIN) {
    prog += (size_t)a.spb * nrhs * 12 * (NS + 1) * 2;
    kap = prog;
    prog += MAXRHS;
    if (tid < nrhs) kap[tid] = (R)a.kappa[tid];
    // x term with its own fifth-dimension program: transform it in LDS before the
    // hop, so no column pass runs while the hop accumulators are live
    x_first = a.xin != nullptr && a.prog_x.n > 0;
    if (x_first) {
      cpx<R>* buf = reinterpret_cast<cpx<R>*>(pl.h);
      if (valid) {
        cpx<R> xv[12];
        load_site<P>(a.xin, a.xin_sc, j0 + sl, r, s, nrhs, NS, xv);
#pragma unroll
        for (int c = 0; c < 12; c++) buf[((size_t)(sl * nrhs + r) * 12 + c) * (NS + 1) + s] = xv[c];
      }
      __syncthreads();
      column_pass_lds<R, NS>(buf, nsb, nrhs, a.prog_x, reinterpret_cast<const R*>(a.coef), kap, tid);
    }
  }
  double* red = reinterpret_cast<double*>(prog);

  cpx<R> acc[12];
#pragma unroll
  for (int c = 0; c < 12; c++) acc[c] = {R(0), R(0)};
  {
    const cpx<R>* U = lnk + (size_t)sl * 8 * 9;
    constexpr int G = HopGroup<P>::G;
    constexpr bool PRE = sizeof(R) == 8;
    // (row offsets are 32-bit: a row of a half field is at most 6.3 MB here, 128 sites of 256 FP64 5D sites)
    if (a.rows) hop_sum_row<P, NS, DAG, G, PRE>(a, (int)j0, sl, r, s, valid, U, acc);
    else hop_sum<P, NS, DAG, G, PRE, !PLAIN>(a, j0 + sl, r, s, valid, U, acc);
  }
  if constexpr (PLAIN) {
    if (valid) store_site<P, ODWF_NT_STORE>(a.out, a.out_sc, j0 + sl, r, s, nrhs, NS, acc);
    return;
  }

  // the own-site index again from the block-uniform first site: cheaper than
  // keeping the 64-bit index live through the hop (which spills at 4 waves);
  // the empty asm stops the compiler from reusing the value computed earlier
  int slr = sl;
  asm volatile("" : "+v"(slr));
  cpx<R> xv[12], rv[12];
  const R rho[6] = {};
  const double nval = fused_tail<P, NS, false>(a, first_io(a), acc, valid, (long)j0 + slr, sl, r, s, nsb, pl, kap,
                                               x_first ? X_LDS : X_LOAD, xv, rv, rho, R(0), false, tid);
  if (a.partial) block_reduce_rhs(valid ? nval : 0.0, NS, a.spb, nrhs, red, a.partial, lb, tid);
}

template <class P, int NS, bool DAG, bool PLAIN>
__global__ void __launch_bounds__(256, (HopWaves<P, NS, PLAIN>::W)) hop_kernel(const HopArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t lb = blockIdx.x;
  if constexpr (!PLAIN) {
    if (a.fin_partial) {  // the first block forms the step lengths
      if (lb == 0) {
        fin_block(a, reinterpret_cast<double*>(smem));
        return;
      }
      lb -= 1;
    }
  }
  if (!gate_any(a.gate, a.gate_mode, a.nrhs)) return;  // whole block idle
  hop_block<P, NS, DAG, PLAIN>(a, lb, threadIdx.x);
}

// Launches gated to pending updates find nothing to do in most iterations, and
// then cost the passing of their blocks.  Above the blocks that fit the chip at
// once (a span) a block here walks several, a span apart: up to eight spans in a
// single one, beyond them two to a block, since blocks that walk alone drift apart
// and lose the rows they share in L2.  us a launch with work / without, against
// hop_kernel: 16^4 x 16 (4 spans) 85 / 4.6 and 89 / 4.6; 16^3 x 32 x 16 (8) 168 / 4.6
// and 174 / 4.7; 8^4 x 16 of twelve slots (4) 45 / 4.5 and 43 / 6.2; 32^3 x 16 x 16
// (32) 654 / 4.9 and 623 / 10 (745 / 4.8 in one span, 717 / 4.7 with four to a
// block); 64^3 x 32 x 16 (512) 10750 / 43 and 10460 / 119 (14430 / 4.5, 11750 / 23).
constexpr int LOOP_SPANS = 8, LOOP_STEPS = 2;
__host__ __device__ inline uint32_t loop_span(int threads) { return 256 * (512 / threads); }  // two waves per SIMD
template <class P, int NS, bool DAG>
__global__ void __launch_bounds__(256, (HopWaves<P, NS, false>::W)) hop_loop_kernel(const HopArgs a) {
  if (!gate_any(a.gate, a.gate_mode, a.nrhs)) return;  // whole block idle
  const uint32_t span = loop_span(blockDim.x);
  const uint32_t steps = gridDim.x == span ? LOOP_SPANS : LOOP_STEPS;
  uint32_t lb = blockIdx.x / span * span * steps + blockIdx.x % span;
  for (uint32_t k = 0; k < steps && lb < (uint32_t)a.nblocks; k++, lb += span) {
    // the arguments and the thread's index again for every block: what follows from
    // them would be formed outside the loop and kept through it, and does not fit
    // the registers
    auto* args = __builtin_amdgcn_kernarg_segment_ptr();
    int tid = threadIdx.x;
    asm volatile("" : "+s"(args), "+v"(tid));
    hop_block<P, NS, DAG, false>(*(const HopArgs*)args, lb, tid);
    __syncthreads();  // LDS of these sites is done with
  }
}

// ---------------------------------------------------------------------------
// Small launches: a lattice whose columns do not fill the chip is bound by the
// chain of latencies of one block, not by traffic.  Here four waves share 64
// 5D sites: wave mu takes the forward and the backward hop of direction mu (its
// two neighbours, and its links through LDS of its own, all in flight
// together), the four partial sums meet in LDS at the only barrier, and wave 0,
// which has meanwhile requested what the epilogue reads, runs it.  Against the
// kernel above: a quarter of the hop's arithmetic per wave, one round trip to memory
// instead of six, four times the waves.
// ---------------------------------------------------------------------------
// complex numbers of one wave's links: two of each of the block's sites
template <int NS>
constexpr int SMALL_LINKS = 2 * (64 / NS) * 9;

template <class P, bool DAG, int MU, bool FWD>
__device__ __forceinline__ void small_term(typename Neighbour<P>::V& v, typename P::real sc, bool flip, float one,
                                           const cpx<typename P::real>* U, cpx<typename P::real> (&acc)[12]) {
  constexpr int SIG = FWD != DAG ? +1 : -1;
  using N = Neighbour<P>;
  if (P::SCALED && flip) sc = -sc;
  if constexpr (N::RAW16) {
    hop_one_h16<MU, SIG>(v, sc, one, U, acc);
  } else if constexpr (N::RAW64) {
    typename N::Site z;
    N::get(v, z);
    if (flip) N::negate(z);
    hop_one<MU, SIG>(z, U, acc);
  } else if constexpr (P::SCALED) {
    hop_one_scaled<MU, SIG>(v, sc, U, acc);
  } else {
    if (flip) N::negate(v);
    hop_one<MU, SIG>(v, U, acc);
  }
}
template <class P, bool DAG, int MU>
__device__ __forceinline__ void small_terms(typename Neighbour<P>::V (&v)[2], const typename P::real (&sc)[2], bool flip_f,
                                            bool flip_b, float one, const cpx<typename P::real>* U,
                                            cpx<typename P::real> (&acc)[12]) {
  small_term<P, DAG, MU, true>(v[0], sc[0], flip_f, one, U, acc);
  small_term<P, DAG, MU, false>(v[1], sc[1], flip_b, one, U + 9, acc);
}

// The two links (forward, backward) of direction mu of the block's sites into
// LDS of the calling wave, times -1/2 as in stage_links: matrix 2 site + b.
// load() requests them, store() writes them.
template <class P, int NS>
struct SmallLinks {
  static constexpr bool FULL = LinkFmt<P>::REALS == 18;
  static constexpr int K = FULL ? (2 * (64 / NS) * 9 + 63) / 64 : 3;
  uint4 q[K];
  __device__ static __forceinline__ int clamp_mat(int m, int nsb) { return min(m, 2 * nsb - 1); }
  __device__ __forceinline__ void load(const void* links, uint32_t j0, int nsb, int mu, int l) {
    const uint4* src = reinterpret_cast<const uint4*>(links);
#pragma unroll
    for (int k = 0; k < K; k++) {
      const int m = clamp_mat(FULL ? (l + 64 * k) / 9 : l, nsb), e = FULL ? (l + 64 * k) % 9 : k;
      q[k] = src[(((long)j0 + (m >> 1)) * 8 + mu + 4 * (m & 1)) * (FULL ? 9 : 3) + e];
    }
  }
  __device__ __forceinline__ void store(cpx<typename P::real>* lw, int nsb, int l) const {
    if constexpr (FULL) {
#pragma unroll
      for (int k = 0; k < K; k++) {
        cpx<double> z;
        unpack_chunk<SP64>(q[k], &z);
        if (l + 64 * k < 2 * nsb * 9) lw[l + 64 * k] = cscale(-0.5, z);
      }
    } else if (l < 2 * nsb) {
      cpx<float> u[6];
#pragma unroll
      for (int k = 0; k < 3; k++) unpack_chunk<SP32>(q[k], &u[2 * k]);
      cpx<float>* d = lw + l * 9;
#pragma unroll
      for (int k = 0; k < 6; k++) d[k] = cscale(-0.5f, u[k]);
#pragma unroll
      for (int a0 = 0; a0 < 3; a0++) {
        const int b0 = (a0 + 1) % 3, c0 = (a0 + 2) % 3;
        const cpx<float> t = csub(cmul(u[b0], u[3 + c0]), cmul(u[c0], u[3 + b0]));
        d[6 + a0] = {-0.5f * t.re, 0.5f * t.im};
      }
    }
  }
};

// (two waves per SIMD keep the register budget at 256: above it the compiler puts
// the matrix results of the dense programs into accumulation registers.  Such
// builds gave wrong results, by a cause that was not found; the build refuses them)
template <class P, int NS, bool DAG>
__global__ void __launch_bounds__(256, 2) hop_small_kernel(const HopArgs a) {
  using R = typename P::real;
  using N = Neighbour<P>;
  constexpr int NCG = 12 / P::CPB;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nrhs = a.nrhs;
  const int tid = threadIdx.x;
  uint32_t lb = blockIdx.x;
  if (a.fin_partial) {  // the first block forms the step lengths
    if (lb == 0) {
      fin_block(a, reinterpret_cast<double*>(smem));
      return;
    }
    lb -= 1;
  }
  if (!gate_any(a.gate, a.gate_mode, nrhs)) return;  // whole block idle
  HopIo io = first_io(a);
  if (blockIdx.y) {  // (field by field: an indexed copy of arguments would go through scratch)
    io.in = a.other.in;
    io.in_sc = a.other.in_sc;
    io.links = a.other.links;
    io.xin = a.other.xin;
    io.xin_sc = a.other.xin_sc;
    io.out = a.other.out;
    io.out_sc = a.other.out_sc;
    io.out_par = a.other.out_par;
  }
  const int mu = uniform_int(tid >> 6), l = tid & 63;
  const int col = l / NS, s = l - col * NS;
  const int sl = nrhs == 1 ? col : col / nrhs;
  const int r = col - sl * nrhs;
  const uint32_t j0 = lb * a.spb;
  const int nsb = min(a.spb, a.h - (int)j0);
  const bool valid = sl < nsb && gate_on(a.gate, a.gate_mode, r);
  const uint32_t j = j0 + min(sl, nsb - 1);

  // LDS: partial sums of waves 1-3, wave 0's scratch, programs.  Each wave's
  // links lie where it writes later (its sums, or the scratch)
  R* sum = reinterpret_cast<R*>(smem);
  R* scr = sum + 3 * 24 * 64;
  cpx<R>* lw = reinterpret_cast<cpx<R>*>(mu > 0 ? sum + (mu - 1) * 24 * 64 : scr);
  static_assert(2 * SMALL_LINKS<NS> <= DENSE_SCRATCH<R> && 2 * SMALL_LINKS<NS> <= 24 * 64, "");
  R* prog = scr + DENSE_SCRATCH<R>;

  // the two neighbours and links of this wave's direction
  const int L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  const int hx = a.L[0] >> 1;
  const int row = a.d_hx.div(j), xh = j - row * hx;
  const int zt = a.d_y.div(row), y = row - zt * L1;
  const int t = a.d_z.div(zt), z = zt - t * L2;
  const int p = (y + z + t + io.out_par) & 1;
  typename N::V v[2];
  R sc[2] = {R(1), R(1)};
  SmallLinks<P, NS> lk;
  lk.load(io.links, j0, nsb, mu, l);
  if (valid) {
#pragma unroll
    for (int b = 0; b < 2; b++) {  // forward, backward
      const bool fwd = b == 0;
      int xx = xh, yy = y, zz = z, tt = t;
      // x + 1 lies in column xh (p = 0) or xh + 1 (p = 1), x - 1 in xh - 1 or xh
      if (mu == 0 && fwd && p) xx = xh + 1 == hx ? 0 : xh + 1;
      if (mu == 0 && !fwd && !p) xx = xh == 0 ? hx - 1 : xh - 1;
      if (mu == 1) yy = fwd ? (y + 1 == L1 ? 0 : y + 1) : (y == 0 ? L1 - 1 : y - 1);
      if (mu == 2) zz = fwd ? (z + 1 == L2 ? 0 : z + 1) : (z == 0 ? L2 - 1 : z - 1);
      if (mu == 3) tt = fwd ? (t + 1 == L3 ? 0 : t + 1) : (t == 0 ? L3 - 1 : t - 1);
      const long nj = (long)((tt * L2 + zz) * L1 + yy) * hx + xx;
      const u32x4* src = reinterpret_cast<const u32x4*>(io.in) + (nj * nrhs + r) * NCG * NS + s;
      u32x4 q[NCG];
#pragma unroll
      for (int cg = 0; cg < NCG; cg++) q[cg] = src[cg * NS];
      N::set(v[b], q);
      if constexpr (P::SCALED) sc[b] = io.in_sc[(nj * nrhs + r) * NS + s];
    }
  }
  ProgLds<R> pl = {prog, nullptr, nullptr, nullptr};
  if (a.dn_h.tab) dense_stage<R>(prog, a.dn_h.tab, tid), prog += DENSE_IMAGE<R>;
  pl.x = prog;
  if (a.dn_x.tab) dense_stage<R>(prog, a.dn_x.tab, tid), prog += DENSE_IMAGE<R>;
  pl.o = prog;
  if (a.dn_o.tab) dense_stage<R>(prog, a.dn_o.tab, tid), prog += DENSE_IMAGE<R>;
  pl.scr = scr;
  lk.store(lw, nsb, l);
  wave_lds_order();

  cpx<R> acc[12];
#pragma unroll
  for (int c = 0; c < 12; c++) acc[c] = {R(0), R(0)};
  if (valid) {
    const float one = N::opaque_one();
    const cpx<R>* U = lw + sl * 18;
    const bool flip_f = mu == 3 && a.bc_t < 0 && t + 1 == L3, flip_b = mu == 3 && a.bc_t < 0 && t == 0;
    switch (mu) {
      case 0: small_terms<P, DAG, 0>(v, sc, false, false, one, U, acc); break;
      case 1: small_terms<P, DAG, 1>(v, sc, false, false, one, U, acc); break;
      case 2: small_terms<P, DAG, 2>(v, sc, false, false, one, U, acc); break;
      default: small_terms<P, DAG, 3>(v, sc, flip_f, flip_b, one, U, acc); break;
    }
  }
  cpx<R> xv[12], rv[12];
  R rho[6], alpha = R(0);
  bool cg_update = false;
#pragma unroll
  for (int c = 0; c < 12; c++) xv[c] = rv[c] = {R(0), R(0)};
#pragma unroll
  for (int c = 0; c < 6; c++) rho[c] = R(0);
  // (after the hop: its neighbours, links and these together exceed the registers in FP64)
  if (mu == 0) tail_preload<P, NS>(a, io, valid, j, r, s, xv, rv, rho, alpha, cg_update);
  if (mu > 0) {
    R* d = sum + (mu - 1) * 24 * 64 + l;
#pragma unroll
    for (int c = 0; c < 12; c++) {
      d[(2 * c) * 64] = acc[c].re;
      d[(2 * c + 1) * 64] = acc[c].im;
    }
  }
  __syncthreads();
  if (mu > 0) return;
#pragma unroll
  for (int w = 0; w < 3; w++) {
    const R* d = sum + w * 24 * 64 + l;
#pragma unroll
    for (int c = 0; c < 12; c++) acc[c] = cadd(acc[c], cpx<R>{d[(2 * c) * 64], d[(2 * c + 1) * 64]});
  }
  double nval = fused_tail<P, NS, true>(a, io, acc, valid, j, sl, r, s, nsb, pl, nullptr, X_LOAD, xv, rv, rho, alpha,
                                        cg_update, tid);
  if (a.partial) {  // one wave: LDS of its own, in order
    if (!valid) nval = 0.0;
    for (int m = NS >> 1; m >= 1; m >>= 1) nval += __shfl_xor(nval, m, NS);
    double* tmp = reinterpret_cast<double*>(smem);
    wave_lds_order();
    if (s == 0) tmp[col] = nval;
    wave_lds_order();
    if (l < nrhs) {
      double tot = 0.0;
      for (int k = 0; k < a.spb; k++) tot += tmp[k * nrhs + l];
      a.partial[(long)lb * nrhs + l] = tot;
    }
  }
}

// extra LDS per block (plain / fused kernels): caps the blocks resident per CU
#ifndef ODWF_HOP_SMEM_PAD
#define ODWF_HOP_SMEM_PAD 0
#endif
#ifndef ODWF_HOP_SMEM_PAD_F
#define ODWF_HOP_SMEM_PAD_F 0
#endif
template <class P, int NS>
static size_t hop_smem(const HopArgs& a, bool plain) {
  using R = typename P::real;
  size_t n = (size_t)a.spb * 8 * 9 * 2;  // reals
  if (!plain && NS <= DENSE_N)
    n += (size_t)DENSE_IMAGE<R> * ((a.dn_h.tab != nullptr) + (a.dn_x.tab != nullptr) + (a.dn_o.tab != nullptr)) +
         (size_t)((a.spb * a.nrhs * NS + 63) / 64) * DENSE_SCRATCH<R>;
  else if (!plain)
    n += (size_t)a.spb * a.nrhs * 12 * (NS + 1) * 2 + MAXRHS;
  n = n * sizeof(R) + (plain ? 0 : (size_t)a.spb * a.nrhs * sizeof(double));
  // a launch with a scalar block: one double a thread
  if (a.fin_partial) n = std::max(n, (size_t)256 * sizeof(double));
  return n + (plain ? ODWF_HOP_SMEM_PAD : ODWF_HOP_SMEM_PAD_F);
}

template <class P, int NS>
static hipError_t launch_hop_t(HopArgs a, int dag, hipStream_t st) {
  const int inner = a.nrhs * NS;
  if (inner > 256 || a.nrhs > MAXRHS) return hipErrorInvalidValue;
  if constexpr (NS <= DENSE_N) {
    if (a.small) {
      using R = typename P::real;
      const int np = (a.dn_h.tab != nullptr) + (a.dn_x.tab != nullptr) + (a.dn_o.tab != nullptr);
      const size_t sm = (3 * 24 * 64 + (size_t)np * DENSE_IMAGE<R> + DENSE_SCRATCH<R>) * sizeof(R);
      const dim3 grid(a.nblocks + (a.fin_partial ? 1 : 0), a.pair ? 2 : 1);
      if (dag) hipLaunchKernelGGL((hop_small_kernel<P, NS, true>), grid, dim3(256), sm, st, a);
      else hipLaunchKernelGGL((hop_small_kernel<P, NS, false>), grid, dim3(256), sm, st, a);
      return hipGetLastError();
    }
  }
  const int block = (a.spb * inner + 63) & ~63;  // whole waves, <= 256
  const size_t sm = hop_smem<P, NS>(a, a.plain);
  if constexpr (sizeof(typename P::real) == 8) {
    const int span = loop_span(block);
    if (a.gate_mode == GATE_UPDATE && !a.plain && !a.fin_partial && a.nblocks > span) {
      const int walk = span * (a.nblocks <= span * LOOP_SPANS ? LOOP_SPANS : LOOP_STEPS);  // of a span of blocks
      const dim3 grid((a.nblocks + walk - 1) / walk * span);
      if (dag) hipLaunchKernelGGL((hop_loop_kernel<P, NS, true>), grid, dim3(block), sm, st, a);
      else hipLaunchKernelGGL((hop_loop_kernel<P, NS, false>), grid, dim3(block), sm, st, a);
      return hipGetLastError();
    }
  }
  const dim3 grid(a.nblocks + (a.fin_partial ? 1 : 0));
  if (a.plain) {
    if (dag) hipLaunchKernelGGL((hop_kernel<P, NS, true, true>), grid, dim3(block), sm, st, a);
    else hipLaunchKernelGGL((hop_kernel<P, NS, false, true>), grid, dim3(block), sm, st, a);
    return hipGetLastError();
  }
  if (dag) hipLaunchKernelGGL((hop_kernel<P, NS, true, false>), grid, dim3(block), sm, st, a);
  else hipLaunchKernelGGL((hop_kernel<P, NS, false, false>), grid, dim3(block), sm, st, a);
  return hipGetLastError();
}

template <class P>
static hipError_t launch_hop_p(const HopArgs& a, int Ns, int dag, hipStream_t st) {
  switch (Ns) {
    case 4: return launch_hop_t<P, 4>(a, dag, st);
    case 8: return launch_hop_t<P, 8>(a, dag, st);
    case 16: return launch_hop_t<P, 16>(a, dag, st);
    case 32: return launch_hop_t<P, 32>(a, dag, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace odwf
