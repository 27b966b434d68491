// Device-side building blocks shared by the HIP kernels of libodwf:
// complex arithmetic, spinor storage policies (FP64 / FP32 / FP16+scale /
// BF16+scale), link formats, fifth-dimension programs and deterministic
// per-right-hand-side block reductions.
//
// Internal spinor layout of one parity half (h = V/2 sites), per site j,
// right-hand side r, fifth-dimension slice s and spin-colour component
// c = spin*3 + colour (12 complex per 5D site):
//     chunk (j, r, cg, s) of CPB consecutive complex numbers, cg = c / CPB,
//     address = ((j * nrhs + r) * NCG + cg) * Ns + s   (in 16-byte chunks),
// so the Ns lanes of one (site, rhs) read consecutive 16-byte chunks and the
// chunk stride within a 5D site is the compile-time Ns.  The
// reduced-precision formats keep one float scale per 5D site (j, r, s) at
// (j * nrhs + r) * Ns + s; stored values are component / scale with scale the
// largest |real| or |imag| part of the 24 reals.
#pragma once
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "odwf_types.h"

namespace odwf {

template <class R>
struct cpx {
  R re, im;
};

template <class R>
__device__ __forceinline__ cpx<R> cadd(cpx<R> a, cpx<R> b) { return {a.re + b.re, a.im + b.im}; }
template <class R>
__device__ __forceinline__ cpx<R> csub(cpx<R> a, cpx<R> b) { return {a.re - b.re, a.im - b.im}; }
template <class R>
__device__ __forceinline__ cpx<R> cscale(R f, cpx<R> a) { return {f * a.re, f * a.im}; }
// a * b
template <class R>
__device__ __forceinline__ cpx<R> cmul(cpx<R> a, cpx<R> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// acc + a * b
template <class R>
__device__ __forceinline__ cpx<R> cfma(cpx<R> a, cpx<R> b, cpx<R> acc) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
  return acc;
}
// i * a
template <class R>
__device__ __forceinline__ cpx<R> cmuli(cpx<R> a) { return {-a.im, a.re}; }
template <class R>
__device__ __forceinline__ R cnorm2(cpx<R> a) { return a.re * a.re + a.im * a.im; }

// ---------------------------------------------------------------------------
// storage policies
// ---------------------------------------------------------------------------

struct SP64 {
  using real = double;
  static constexpr int CPB = 1;  // complex per 16-byte chunk
  static constexpr bool SCALED = false;
  static constexpr int BYTES = 16;  // bytes per complex
};
struct SP32 {
  using real = float;
  static constexpr int CPB = 2;
  static constexpr bool SCALED = false;
  static constexpr int BYTES = 8;
};
struct SP16 {
  using real = float;
  static constexpr int CPB = 4;
  static constexpr bool SCALED = true;
  static constexpr int BYTES = 4;
};
struct SPB16 {
  using real = float;
  static constexpr int CPB = 4;
  static constexpr bool SCALED = true;
  static constexpr int BYTES = 4;
};

// BF16 stores through the hardware conversion (1, default) or the integer
// rounding of f_to_bf16 (0); both round to nearest even
#ifndef ODWF_HW_BF16_CVT
#define ODWF_HW_BF16_CVT 1
#endif
__device__ __forceinline__ float bf16_to_f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f_to_bf16(float f) {
  // round to nearest even; inputs are finite and bounded by 1 after scaling
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// A 16-byte load that stays one: where only the two doubles of a chunk are used,
// the compiler takes two loads of 8 bytes, each of which passes the same cache
// lines through L1 again.  The empty asm uses the chunk as a whole, at the point
// where its value is needed.  FP64 hops (230 -> 129 vector memory instructions a
// wave): 32^3 x 16 x 16 755 / 784 -> about 640 us, normal operator of
// 16^4 x 16 495 -> 448 us a call.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 whole_chunk(u32x4 w) {
  asm("" : "+v"(w));
  return make_uint4(w.x, w.y, w.z, w.w);
}

// unpack one 16-byte chunk into CPB complex values
template <class P>
__device__ __forceinline__ void unpack_chunk(const uint4 q, cpx<typename P::real>* v);

template <>
__device__ __forceinline__ void unpack_chunk<SP64>(const uint4 q, cpx<double>* v) {
  v[0].re = __hiloint2double((int)q.y, (int)q.x);
  v[0].im = __hiloint2double((int)q.w, (int)q.z);
}
template <>
__device__ __forceinline__ void unpack_chunk<SP32>(const uint4 q, cpx<float>* v) {
  v[0] = {__uint_as_float(q.x), __uint_as_float(q.y)};
  v[1] = {__uint_as_float(q.z), __uint_as_float(q.w)};
}
template <>
__device__ __forceinline__ void unpack_chunk<SP16>(const uint4 q, cpx<float>* v) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int k = 0; k < 4; k++) {
    __half2 hh = *reinterpret_cast<const __half2*>(&w[k]);
    float2 f = __half22float2(hh);
    v[k] = {f.x, f.y};
  }
}
template <>
__device__ __forceinline__ void unpack_chunk<SPB16>(const uint4 q, cpx<float>* v) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int k = 0; k < 4; k++) v[k] = {bf16_to_f((uint16_t)(w[k] & 0xffffu)), bf16_to_f((uint16_t)(w[k] >> 16))};
}

template <class P>
__device__ __forceinline__ uint4 pack_chunk(const cpx<typename P::real>* v, typename P::real inv);

template <>
__device__ __forceinline__ uint4 pack_chunk<SP64>(const cpx<double>* v, double) {
  uint4 q;
  q.x = (uint32_t)__double2loint(v[0].re);
  q.y = (uint32_t)__double2hiint(v[0].re);
  q.z = (uint32_t)__double2loint(v[0].im);
  q.w = (uint32_t)__double2hiint(v[0].im);
  return q;
}
template <>
__device__ __forceinline__ uint4 pack_chunk<SP32>(const cpx<float>* v, float) {
  return make_uint4(__float_as_uint(v[0].re), __float_as_uint(v[0].im), __float_as_uint(v[1].re),
                    __float_as_uint(v[1].im));
}
template <>
__device__ __forceinline__ uint4 pack_chunk<SP16>(const cpx<float>* v, float inv) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; k++) {
    __half2 hh = __floats2half2_rn(v[k].re * inv, v[k].im * inv);
    w[k] = *reinterpret_cast<uint32_t*>(&hh);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}
template <>
__device__ __forceinline__ uint4 pack_chunk<SPB16>(const cpx<float>* v, float inv) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; k++) {
#if ODWF_HW_BF16_CVT
    // one v_cvt_pk_bf16_f32 per complex (gfx950): round to nearest even, as f_to_bf16
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 f = {v[k].re * inv, v[k].im * inv};
    w[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
#else
    w[k] = (uint32_t)f_to_bf16(v[k].re * inv) | ((uint32_t)f_to_bf16(v[k].im * inv) << 16);
#endif
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// Spinor half-field view
template <class P>
struct HalfView {
  const uint4* __restrict__ base;
  const float* __restrict__ scale;
};

// load the 12 components of 5D site (j, r, s); NT = 1: nontemporal loads
// (a stream read once, which should not displace re-used rows from L2); NOW:
// the values are needed at once (else they may travel on behind this call)
template <class P, int NT = 0, bool NOW = true>
__device__ __forceinline__ void load_site(const void* base, const float* scale, long j, int r, int s,
                                          int nrhs, int Ns, cpx<typename P::real> (&v)[12]) {
  constexpr int NCG = 12 / P::CPB;
  const u32x4* b = reinterpret_cast<const u32x4*>(base);
  const long off = ((j * nrhs + r) * NCG) * Ns + s;
  u32x4 q[NCG];
#pragma unroll
  for (int cg = 0; cg < NCG; cg++) {
    if constexpr (NT) q[cg] = __builtin_nontemporal_load(b + off + cg * Ns);
    else q[cg] = b[off + cg * Ns];
  }
#pragma unroll
  for (int cg = 0; cg < NCG; cg++) {
    if constexpr (NOW && P::CPB == 1) unpack_chunk<P>(whole_chunk(q[cg]), &v[cg * P::CPB]);
    else unpack_chunk<P>(make_uint4(q[cg].x, q[cg].y, q[cg].z, q[cg].w), &v[cg * P::CPB]);
  }
  if constexpr (P::SCALED) {
    float sc = scale[(j * nrhs + r) * Ns + s];
#pragma unroll
    for (int c = 0; c < 12; c++) v[c] = cscale(sc, v[c]);
  }
}

// NT = 1: nontemporal stores (written once, not re-read by this launch)
#ifndef ODWF_NT_STORE
#define ODWF_NT_STORE 0
#endif
#ifndef ODWF_NT_LINKS
#define ODWF_NT_LINKS 0
#endif
template <class P, int NT = 0>
__device__ __forceinline__ void store_site(void* base, float* scale, long j, int r, int s, int nrhs,
                                           int Ns, const cpx<typename P::real> (&v)[12]) {
  using R = typename P::real;
  constexpr int NCG = 12 / P::CPB;
  uint4* b = reinterpret_cast<uint4*>(base);
  const long off = ((j * nrhs + r) * NCG) * Ns + s;
  R inv = R(1);
  if constexpr (P::SCALED) {
    float m = 0.f;
#pragma unroll
    for (int c = 0; c < 12; c++) m = fmaxf(m, fmaxf(fabsf(v[c].re), fabsf(v[c].im)));
    if constexpr (NT) __builtin_nontemporal_store(m, scale + (j * nrhs + r) * Ns + s);
    else scale[(j * nrhs + r) * Ns + s] = m;
    inv = m > 0.f ? 1.0f / m : 0.f;
  }
#pragma unroll
  for (int cg = 0; cg < NCG; cg++) {
    const uint4 q = pack_chunk<P>(&v[cg * P::CPB], inv);
    if constexpr (NT) {
      const u32x4 w = {q.x, q.y, q.z, q.w};
      __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(b + off + cg * Ns));
    } else {
      b[off + cg * Ns] = q;
    }
  }
}

// ---------------------------------------------------------------------------
// spin projection in the chiral basis (shared by the hopping and force kernels)
// ---------------------------------------------------------------------------

// multiplication by f in {+1, -1, +i, -i} (codes 0..3)
template <int CODE, class R>
__device__ __forceinline__ cpx<R> mulf(cpx<R> z) {
  if constexpr (CODE == 0) return z;
  if constexpr (CODE == 1) return {-z.re, -z.im};
  if constexpr (CODE == 2) return {-z.im, z.re};
  return {z.im, -z.re};
}
template <int CODE>
struct ConjCode {
  static constexpr int v = CODE == 2 ? 3 : (CODE == 3 ? 2 : CODE);
};

// chiral basis: gamma_mu = [[0, B_mu], [B_mu^dag, 0]], row a of B_mu has one
// entry f_a at column p_a:
//   mu = x: p = (1, 0), f = (-i, -i);   mu = y: p = (1, 0), f = (-1, +1)
//   mu = z: p = (0, 1), f = (-i, +i);   mu = t: p = (0, 1), f = (+1, +1)
template <int MU>
struct GammaB;
template <>
struct GammaB<0> {
  static constexpr int p0 = 1, p1 = 0, f0 = 3, f1 = 3;
};
template <>
struct GammaB<1> {
  static constexpr int p0 = 1, p1 = 0, f0 = 1, f1 = 0;
};
template <>
struct GammaB<2> {
  static constexpr int p0 = 0, p1 = 1, f0 = 3, f1 = 2;
};
template <>
struct GammaB<3> {
  static constexpr int p0 = 0, p1 = 1, f0 = 0, f1 = 0;
};

// (1 - SIG gamma_mu) psi = [h; -SIG B^dag h], h = psi_up - SIG B psi_dn.
// Computes the half spinor h (2 spins x 3 colours).
template <int MU, int SIG, class R>
__device__ __forceinline__ void project(const cpx<R> (&psi)[12], cpx<R> (&h)[6]) {
  using B = GammaB<MU>;
#pragma unroll
  for (int c = 0; c < 3; c++) {
    cpx<R> t0 = mulf<B::f0>(psi[(2 + B::p0) * 3 + c]);
    cpx<R> t1 = mulf<B::f1>(psi[(2 + B::p1) * 3 + c]);
    if constexpr (SIG > 0) {
      h[c] = csub(psi[c], t0);
      h[3 + c] = csub(psi[3 + c], t1);
    } else {
      h[c] = cadd(psi[c], t0);
      h[3 + c] = cadd(psi[3 + c], t1);
    }
  }
}

// Orders what the lanes of one wave exchange through LDS: writes before, reads (and
// later writes) behind.  The hardware takes a wave's LDS operations in order, so
// this costs no instruction; the fences keep the compiler from moving accesses
// across (wave_barrier alone orders the instructions it schedules, not the memory).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// is right-hand side r selected by the gate?
__device__ __forceinline__ bool gate_on(const CGScal* g, int mode, int r) {
  if (!g || mode == GATE_NONE) return true;
  return mode == GATE_ACTIVE ? g[r].active != 0 : g[r].update != 0;
}
// does any right-hand side of the launch pass the gate? (block-uniform)
__device__ __forceinline__ bool gate_any(const CGScal* g, int mode, int nrhs) {
  if (!g || mode == GATE_NONE) return true;
  bool any = false;
  for (int r = 0; r < nrhs; r++) any |= gate_on(g, mode, r);
  return any;
}

// ---------------------------------------------------------------------------
// fifth-dimension programs on one column y[0..NS-1] (one 4D site, one
// right-hand side, one spin-colour component), in the chirality-local order:
// chirality + (spins 0, 1) uses s as is, chirality - (spins 2, 3) uses the
// mirrored index NS-1-s, in which L_- takes the same lower-shift form as L_+.
// ---------------------------------------------------------------------------

// coefficient table coef[chi][id][s] in global memory; the column passes
// make chi wave-uniform so the coefficients come in through scalar loads
template <class R, int NS>
__device__ __forceinline__ void m5_run(const M5Prog& prog, cpx<R> (&y)[NS], const R* __restrict__ cf,
                                       R kappa) {
  for (int k = 0; k < prog.n; k++) {
    const M5Op op = prog.op[k];
    const R* d = cf + op.d * NS;
    const R* e = cf + op.e * NS;
    switch (op.type) {
      case M5_SCALE: {
#pragma unroll
        for (int s = 0; s < NS; s++) y[s] = cscale(d[s], y[s]);
      } break;
      case M5_MUL_LO: {  // z_s = d_s y_s + e_s y_{s-1};  z_0 = d_0 y_0 + kappa e_0 y_{NS-1}
        cpx<R> last = y[NS - 1];
#pragma unroll
        for (int s = NS - 1; s >= 1; s--) y[s] = cadd(cscale(d[s], y[s]), cscale(e[s], y[s - 1]));
        y[0] = cadd(cscale(d[0], y[0]), cscale(kappa * e[0], last));
      } break;
      case M5_MUL_UP: {  // z_s = d_s y_s + e_s y_{s+1};  z_{NS-1} = d y + kappa e_{NS-1} y_0
        cpx<R> first = y[0];
#pragma unroll
        for (int s = 0; s < NS - 1; s++) y[s] = cadd(cscale(d[s], y[s]), cscale(e[s], y[s + 1]));
        y[NS - 1] = cadd(cscale(d[NS - 1], y[NS - 1]), cscale(kappa * e[NS - 1], first));
      } break;
      case M5_SOLVE_LO: {  // inverse of MUL_LO; d holds 1/d
        // y_s = p_s + q_s y_{N-1}; p by forward substitution, q recomputed
        R q = -kappa * e[0] * d[0];
        y[0] = cscale(d[0], y[0]);
#pragma unroll
        for (int s = 1; s < NS; s++) {
          q = -e[s] * q * d[s];
          y[s] = cscale(d[s], csub(y[s], cscale(e[s], y[s - 1])));
        }
        const cpx<R> vl = cscale(R(1) / (R(1) - q), y[NS - 1]);
        y[NS - 1] = vl;
        q = -kappa * e[0] * d[0];
#pragma unroll
        for (int s = 0; s < NS - 1; s++) {
          if (s > 0) q = -e[s] * q * d[s];
          y[s] = cadd(y[s], cscale(q, vl));
        }
      } break;
      case M5_SOLVE_UP: {  // inverse of MUL_UP; d holds 1/d
        R q = -kappa * e[NS - 1] * d[NS - 1];
        y[NS - 1] = cscale(d[NS - 1], y[NS - 1]);
#pragma unroll
        for (int s = NS - 2; s >= 0; s--) {
          q = -e[s] * q * d[s];
          y[s] = cscale(d[s], csub(y[s], cscale(e[s], y[s + 1])));
        }
        const cpx<R> v0 = cscale(R(1) / (R(1) - q), y[0]);
        y[0] = v0;
        q = -kappa * e[NS - 1] * d[NS - 1];
#pragma unroll
        for (int s = NS - 1; s >= 1; s--) {
          if (s < NS - 1) q = -e[s] * q * d[s];
          y[s] = cadd(y[s], cscale(q, v0));
        }
      } break;
      default: break;
    }
  }
}

// the same programs applied in place to one LDS column (element s at
// col[chi ? NS - 1 - s : s]), streaming through it with O(1) registers
template <class R, int NS>
__device__ __forceinline__ void m5_run_lds(const M5Prog& prog, cpx<R>* col, int chi,
                                           const R* __restrict__ cf, R kappa) {
  const int st = chi ? -1 : 1;
  cpx<R>* c0 = col + (chi ? NS - 1 : 0);  // element s at c0[s * st]
  for (int k = 0; k < prog.n; k++) {
    const M5Op op = prog.op[k];
    const R* d = cf + op.d * NS;
    const R* e = cf + op.e * NS;
    switch (op.type) {
      case M5_SCALE: {
#pragma unroll 4
        for (int s = 0; s < NS; s++) c0[s * st] = cscale(d[s], c0[s * st]);
      } break;
      case M5_MUL_LO: {
        const cpx<R> last = c0[(NS - 1) * st];
        cpx<R> hi = last;
#pragma unroll 4
        for (int s = NS - 1; s >= 1; s--) {
          const cpx<R> lo = c0[(s - 1) * st];
          c0[s * st] = cadd(cscale(d[s], hi), cscale(e[s], lo));
          hi = lo;
        }
        c0[0] = cadd(cscale(d[0], hi), cscale(kappa * e[0], last));
      } break;
      case M5_MUL_UP: {
        const cpx<R> first = c0[0];
        cpx<R> lo = first;
#pragma unroll 4
        for (int s = 0; s < NS - 1; s++) {
          const cpx<R> hi = c0[(s + 1) * st];
          c0[s * st] = cadd(cscale(d[s], lo), cscale(e[s], hi));
          lo = hi;
        }
        c0[(NS - 1) * st] = cadd(cscale(d[NS - 1], lo), cscale(kappa * e[NS - 1], first));
      } break;
      case M5_SOLVE_LO: {
        R q = -kappa * e[0] * d[0];
        cpx<R> prev = cscale(d[0], c0[0]);
        c0[0] = prev;
#pragma unroll 4
        for (int s = 1; s < NS; s++) {
          q = -e[s] * q * d[s];
          prev = cscale(d[s], csub(c0[s * st], cscale(e[s], prev)));
          c0[s * st] = prev;
        }
        const cpx<R> vl = cscale(R(1) / (R(1) - q), prev);
        c0[(NS - 1) * st] = vl;
        q = -kappa * e[0] * d[0];
#pragma unroll 4
        for (int s = 0; s < NS - 1; s++) {
          if (s > 0) q = -e[s] * q * d[s];
          c0[s * st] = cadd(c0[s * st], cscale(q, vl));
        }
      } break;
      case M5_SOLVE_UP: {
        R q = -kappa * e[NS - 1] * d[NS - 1];
        cpx<R> prev = cscale(d[NS - 1], c0[(NS - 1) * st]);
        c0[(NS - 1) * st] = prev;
#pragma unroll 4
        for (int s = NS - 2; s >= 0; s--) {
          q = -e[s] * q * d[s];
          prev = cscale(d[s], csub(c0[s * st], cscale(e[s], prev)));
          c0[s * st] = prev;
        }
        const cpx<R> v0 = cscale(R(1) / (R(1) - q), prev);
        c0[0] = v0;
        q = -kappa * e[NS - 1] * d[NS - 1];
#pragma unroll 4
        for (int s = NS - 1; s >= 1; s--) {
          if (s < NS - 1) q = -e[s] * q * d[s];
          c0[s * st] = cadd(c0[s * st], cscale(q, v0));
        }
      } break;
      default: break;
    }
  }
}

// ---------------------------------------------------------------------------
// dense programs on the matrix cores (N_s <= 16).  A wave holds 64 5D sites:
// four sets (lane / 16) of 16 slice slots (lane % 16; one column of N_s = 16
// slices, or 16 / N_s columns side by side with a block-diagonal matrix), 24
// reals per lane.  v_mfma_*_16x16x4 contracts over lane / 16, so the slots have
// to move there: each wave passes its reals through LDS of its own (one b32 /
// b64 write per real, the four slots of a lane's operand element back in one or
// two b128 reads, rows padded so that neither side meets bank conflicts; LDS
// operations of one wave are in order, so there is no barrier), takes the
// data as the first operand (row = set and real, k = lane / 16 for the slots
// 4 k .. 4 k + 3) and the transposed matrix as the second, and finds the result
// in the lanes and registers it started from.  Every output row depends on its
// own input row only.
// Replaces a serial recurrence through LDS columns (FP64: 190-224 VGPRs, two
// barriers per program) or a log-depth scan over DPP rows (FP32: 350 vector
// instructions per program, now 70; 16-bit storage the same).  Fused launches,
// before and after: FP64 32^3 x 16 x 16 1064 / 920 -> 755 / 784 us, 4^4 x 8
// 21.8 / 18.6 -> 16.1 / 15.5 us; FP32 32^3 x 16 x 16 302 / 310 -> 303 / 302 us;
// FP16S 24^4 x 16 167 / 157 -> 165 / 152 us (DPP quads for the transposition,
// without LDS, took 172 / 157 us: 280 vector instructions per program).
// ---------------------------------------------------------------------------
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));
typedef double mfma_f64x4 __attribute__((ext_vector_type(4)));
template <class R>
struct Mfma;
template <>
struct Mfma<float> {
  using V = mfma_f32x4;
  static constexpr int ROW = 20;           // reals between two rows of 16 slots, scratch and matrix
  static constexpr int SET = 12 * ROW;     // reals between two sets
  __device__ static __forceinline__ int swap(int) { return 0; }
  // register v of lane group g is result row 4 g + v: row = 4 set + real
  __device__ static __forceinline__ int set_of(int row) { return row >> 2; }
  __device__ static __forceinline__ int real_of(int row) { return row & 3; }
  __device__ static __forceinline__ V mul(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<double> {
  using V = mfma_f64x4;
  static constexpr int ROW = 18;
  static constexpr int SET = 12 * ROW + 24;
  // sets 2 and 3 keep the halves of a row swapped: sets 0 / 2 and 1 / 3, which lie
  // on the same banks, are read together
  __device__ static __forceinline__ int swap(int set) { return (set & 2) << 2; }
  // register v of lane group g is result row 4 v + g: row = 4 real + set
  __device__ static __forceinline__ int set_of(int row) { return row & 3; }
  __device__ static __forceinline__ int real_of(int row) { return row >> 2; }
  __device__ static __forceinline__ V mul(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
// reals of LDS scratch per wave
template <class R>
constexpr int DENSE_SCRATCH = 4 * Mfma<R>::SET;

// LDS image of a program: its table (M0, u, w per chirality) in the arithmetic
// type.  Nothing in it depends on the mass, so one image serves every
// right-hand side of a launch.
template <class R>
constexpr int DENSE_IMAGE_CHI = DENSE_N * Mfma<R>::ROW + 2 * DENSE_N;  // rows padded against bank conflicts (0.5 - 1.2 % of a solve)
template <class R>
constexpr int DENSE_IMAGE = 2 * DENSE_IMAGE_CHI<R>;
template <class R>
__device__ __forceinline__ void dense_stage(R* m, const double* __restrict__ tab, int tid) {
  constexpr int K = (DENSE_LEN + 255) / 256;  // a thread's elements in flight together (256 threads)
  constexpr int NN = DENSE_N * DENSE_N;
  for (int i0 = tid; i0 < DENSE_LEN; i0 += K * blockDim.x) {
    double v[K];
#pragma unroll
    for (int k = 0; k < K; k++) v[k] = tab[min(i0 + k * (int)blockDim.x, DENSE_LEN - 1)];
#pragma unroll
    for (int k = 0; k < K; k++) {
      const int i = i0 + k * blockDim.x, chi = i / DENSE_CHI, e = i - chi * DENSE_CHI;
      const int at = e < NN ? (e / DENSE_N) * Mfma<R>::ROW + e % DENSE_N : DENSE_N * Mfma<R>::ROW + e - NN;
      if (i < DENSE_LEN) m[chi * DENSE_IMAGE_CHI<R> + at] = (R)v[k];
    }
  }
}

template <class R>
__device__ __forceinline__ R dense_lim(const DenseArg& a) { return sizeof(R) == 8 ? (R)a.lim64 : (R)a.lim32; }

// Inputs that must not meet other columns in a row of the matrix instructions, by
// real part and imaginary part of a component (each a row of its own).  One that is
// not finite in any slice of the lane's column becomes zero, and its flag makes the
// column's results NaN; so does a rho that is not finite (a singular mass; lim is NaN
// then), for its chirality.  A column that holds a finite value near lim or above is scaled by a power of
// two, taken back from its results (flag 31).
template <class R>
constexpr R QUARANTINE_SCALE = sizeof(R) == 8 ? R(0x1p-512) : R(0x1p-64);
template <class R>
__device__ __forceinline__ bool finite(R v) { return fabs(v) <= (sizeof(R) == 8 ? (R)__DBL_MAX__ : (R)__FLT_MAX__); }
template <int NS, class R>
__device__ __forceinline__ uint32_t quarantine(cpx<R> (&y)[12], R lim, int lane) {
  const uint64_t column = ((uint64_t(1) << NS) - 1) << (lane / NS * NS);
  uint32_t aside = 0;
  bool big = false;
#pragma unroll
  for (int c = 0; c < 24; c++) {
    R& v = c & 1 ? y[c >> 1].im : y[c >> 1].re;
    if (__ballot(!finite(v)) & column) aside |= 1u << c;
    v = finite(v) ? v : R(0);
    big = big || fabs(v) >= lim / 32;
  }
  if (__ballot(big) & column) {
    aside |= 1u << 31;
#pragma unroll
    for (int c = 0; c < 12; c++) y[c] = cscale(QUARANTINE_SCALE<R>, y[c]);
  }
  return aside;
}
template <class R>
__device__ __forceinline__ void release(cpx<R> (&y)[12], uint32_t aside, R rho_p, R rho_m) {
  if (!finite(rho_p)) aside |= 0xfffu;
  if (!finite(rho_m)) aside |= 0xfff000u;
  const R f = aside >> 31 ? R(1) / QUARANTINE_SCALE<R> : R(1);
#pragma unroll
  for (int c = 0; c < 24; c++) {
    R& v = c & 1 ? y[c >> 1].im : y[c >> 1].re;
    v = (aside >> c) & 1 ? (R)__builtin_nan("") : f * v;
  }
}

// y <- M y for the 12 components of every lane's 5D site; m: LDS image; scr:
// DENSE_SCRATCH reals of this wave (16-byte aligned); rho_p / rho_m: rho of the
// lane's right-hand side per chirality; lim: that of the program
// (DenseArg); tid: the thread's index in its block.  The rank-1 term rho u w^T rides on a
// fifth matrix instruction: lane group k contributes rho times its part of
// w . x (slots 4 k .. 4 k + 3) as element k of the operand row, and u in every
// row of the second operand sums the parts.  Right-hand sides of any masses
// share the instruction, and each one's result is the same bits whatever the
// others are.  Called by whole waves: the matrix instructions ignore the lane
// mask.
// Below 16 slices the zeros between the columns of a row do not stop a value that
// is not finite (0 * Inf is NaN), nor a product rho * t that is not: such inputs are
// set aside (quarantine).  (One test ahead of it all: tests on the way keep the two
// chiralities from overlapping.)  With 16 slices such a value may reach every slice
// of its own column, which is all that its row holds.
// FP64 with 16 slices takes two sums of eight terms (and the rank-1 term): the error
// against extended precision is below that of the recurrences (D 1.40 -> 1.37,
// normal operator 3.96 -> 3.32 units of 2^-53; one sum of sixteen 1.60 and 4.18), and
// the shorter chains take 1 % off an iteration.  TIGHT: one after the other, for a
// caller short of registers (hop_small_kernel, which spills 28 otherwise).
template <int NS, bool TIGHT = false, class R>
__device__ __forceinline__ void dense_apply(cpx<R> (&y)[12], const R* m, R* scr, R rho_p, R rho_m, R lim, int tid) {
  using M = Mfma<R>;
  using V = typename M::V;
  constexpr int NN = DENSE_N * M::ROW;
  const int lane = tid & 63, slot = lane & 15, k = lane >> 4;
  R* put = scr + k * M::SET + (slot ^ M::swap(k));
  const int set_i = M::set_of(slot);
  const R* get = scr + set_i * M::SET + M::real_of(slot) * M::ROW + ((4 * k) ^ M::swap(set_i));
  const int src = 16 * set_i + 4 * k;  // a lane of the operand element's column
  const bool same = slot / NS == 4 * k / NS;  // result slot and operand slots belong to one column
  uint32_t aside = 0;
  if constexpr (NS < DENSE_N) {
    R sum[2] = {R(0), R(0)};
#pragma unroll
    for (int c = 0; c < 12; c++) {
      sum[0] += fabs(y[c].re);
      sum[1] += fabs(y[c].im);
    }
    if (__any(!(sum[0] + sum[1] < lim))) aside = quarantine<NS>(y, lim, lane);
  }
  R rho[2] = {__shfl(rho_p, src, 64), __shfl(rho_m, src, 64)};
  if (NS < DENSE_N) rho[0] = finite(rho[0]) ? rho[0] : R(0), rho[1] = finite(rho[1]) ? rho[1] : R(0);
#pragma unroll
  for (int chi = 0; chi < 2; chi++) {
    const R* mc = m + chi * DENSE_IMAGE_CHI<R>;
    wave_lds_order();
#pragma unroll
    for (int c = 0; c < 6; c++) {
      put[(2 * c) * M::ROW] = y[6 * chi + c].re;
      put[(2 * c + 1) * M::ROW] = y[6 * chi + c].im;
    }
    wave_lds_order();
    R b[4], w[4];
#pragma unroll
    for (int e = 0; e < 4; e++) b[e] = mc[slot * M::ROW + 4 * k + e];
#pragma unroll
    for (int e = 0; e < 4; e++) w[e] = mc[NN + DENSE_N + 4 * k + e];
    const R u = same ? mc[NN + slot] : R(0);
#pragma unroll
    for (int g = 0; g < 3; g++) {
      R x[4];
#pragma unroll
      for (int e = 0; e < 4; e++) x[e] = get[4 * g * M::ROW + e];
      R t = w[0] * x[0];
#pragma unroll
      for (int e = 1; e < 4; e++) t = fma(w[e], x[e], t);
      V d = {R(0), R(0), R(0), R(0)};
      if constexpr (sizeof(R) == 8 && NS == DENSE_N) {
        V d2 = M::mul(rho[chi] * t, u, d);
#pragma unroll
        for (int e = 0; e < 2; e++) d = M::mul(x[e], b[e], d);
        if constexpr (TIGHT) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 2; e < 4; e++) d2 = M::mul(x[e], b[e], d2);
        d = d + d2;
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++) d = M::mul(x[e], b[e], d);
        d = M::mul(rho[chi] * t, u, d);
      }
      y[6 * chi + 2 * g] = {d[0], d[1]};
      y[6 * chi + 2 * g + 1] = {d[2], d[3]};
    }
  }
  if constexpr (NS < DENSE_N)
    if (__any(aside != 0) || !(lim > R(0))) release(y, aside, rho_p, rho_m);
}

// ---------------------------------------------------------------------------
// column pass: buf holds [site][rhs][12 components][NS + 1] values; every
// column (site, rhs, component) of NS values is transformed by prog.  Items
// are ordered (chirality, site, rhs, component-of-chirality) with each
// chirality padded to a multiple of 64, so chirality is uniform per wave.
// blockDim.x must be a multiple of 64.  Caller synchronises around it.
// ---------------------------------------------------------------------------
template <class R, int NS>
__device__ __forceinline__ void column_pass_lds(cpx<R>* buf, int nsb, int nrhs, const M5Prog& prog,
                                                const R* coef, const R* kap, int tid) {
  constexpr int NSP = NS + 1;
  const int per = nsb * nrhs * 6;
  const int ipc = (per + 63) & ~63;
  const int lane = tid & 63;
  for (int base = tid & ~63; base < 2 * ipc; base += blockDim.x) {
    const int chi = __builtin_amdgcn_readfirstlane(base / ipc);
    const int q = base - chi * ipc + lane;
    if (q < per) {
      const int c6 = q % 6;
      const int sr = q / 6;  // sl * nrhs + r
      const int rr = sr % nrhs;
      cpx<R>* col = buf + ((size_t)sr * 12 + chi * 6 + c6) * NSP;
      if constexpr (sizeof(R) == 8) {
        // FP64: a column in registers (2 NS doubles per component) would cap the
        // fused hopping kernel at one wave per SIMD; streamed through LDS it
        // runs two (measured 5 % faster for the normal operator)
        m5_run_lds<R, NS>(prog, col, chi, coef + chi * NCOEF * NS, kap[rr]);
      } else {
        // FP32 arithmetic: the register column is faster than streaming
        cpx<R> yv[NS];
#pragma unroll
        for (int s = 0; s < NS; s++) yv[s] = col[chi ? NS - 1 - s : s];
        m5_run<R, NS>(prog, yv, coef + chi * NCOEF * NS, kap[rr]);
#pragma unroll
        for (int s = 0; s < NS; s++) col[chi ? NS - 1 - s : s] = yv[s];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// deterministic per-right-hand-side block reduction of one double per lane.
// A lane's column is col = site slot * nrhs + right-hand side, its slice s; the
// Ns lanes of a column are consecutive in one wave (Ns a power of two).  They
// add their values by a fixed xor butterfly of cross-lane moves (no LDS
// traffic; every lane ends with the same bits, each pairwise addition being
// commutative); lane s = 0 puts the sum in tmp[col]; one lane per right-hand
// side then adds the nsl site sums in site order and writes
// partial[slot * nrhs + r].
// All threads of the block call it; padded threads (col >= nsl * nrhs) pass 0.
// tmp: LDS of at least nsl * nrhs doubles.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void block_reduce_rhs(double v, int Ns, int nsl, int nrhs, double* tmp,
                                                 double* partial, long slot, int tid) {
  for (int m = Ns >> 1; m >= 1; m >>= 1) v += __shfl_xor(v, m, Ns);
  const int g = tid / Ns;
  __syncthreads();  // tmp may alias LDS the block used before
  if ((tid & (Ns - 1)) == 0 && g < nsl * nrhs) tmp[g] = v;
  __syncthreads();
  if (tid < nrhs) {
    double acc = 0.0;
    for (int k = 0; k < nsl; k++) acc += tmp[k * nrhs + tid];
    partial[slot * nrhs + tid] = acc;
  }
}

// ---------------------------------------------------------------------------
// CG scalars from partial sums: the sum in a fixed order, and the update of a
// right-hand side's record
// ---------------------------------------------------------------------------
// sum over blocks of partial[b * nrhs + r]; thread r < nrhs returns right-hand
// side r's.  Threads take consecutive doubles (a thread keeps one right-hand
// side), then a fixed tree.  Every thread of the block calls it; tmp: LDS of
// blockDim.x doubles.
__device__ __forceinline__ double partial_sum(const double* __restrict__ partial, int nblocks, int nrhs, double* tmp) {
  const int tid = threadIdx.x;
  int n = blockDim.x / nrhs;
  const int used = n * nrhs;
  double acc = 0.0;
  if (tid < used) {
    const long total = (long)nblocks * nrhs;
    long i = tid;
    for (; i + 7L * used < total; i += 8L * used) {  // eight loads in flight
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = partial[i + (long)u * used];
#pragma unroll
      for (int u = 0; u < 8; u++) acc += v[u];
    }
    for (; i < total; i += used) acc += partial[i];
  }
  __syncthreads();  // tmp may alias LDS the block used before
  tmp[tid] = acc;
  __syncthreads();
  while (n > 1) {
    const int half = (n + 1) / 2;
    if (tid < (n - half) * nrhs) tmp[tid] += tmp[tid + half * nrhs];
    __syncthreads();
    n = half;
  }
  return tmp[tid];
}

__device__ __forceinline__ void fin_alpha(CGScal& c, double v) {  // v = <p, N p>
  c.pAp = v;
  c.alpha = 0.0;
  if (!c.active) return;
  if (!isfinite(v) || !(v > 0.0)) {
    c.nan = !isfinite(v);
    c.active = 0;
  } else {
    c.alpha = c.rr / v;
  }
}

__device__ __forceinline__ void fin_beta(CGScal& c, double v) {  // v = |r|^2 after the step
  c.beta = 0.0;
  if (!c.active) return;
  c.iters += 1;
  if (!isfinite(v)) {
    c.nan = 1;
    c.active = 0;
    return;
  }
  c.beta = v / c.rr;
  c.rr = v;
  if (v > c.rmax2) c.rmax2 = v;
  const bool met = v <= c.tol2 * c.f2;
  const bool capped = c.iters >= c.maxiter;
  if (c.confirm) {
    // the decision is left to the true residual of the update that follows
    if (met || capped) c.update = 1;
    if (capped) c.active = 0;
  } else if (met) {
    c.converged = 1;
    c.active = 0;
  } else if (capped) {
    c.active = 0;
  }
  if (c.delta2 > 0.0 && v < c.delta2 * c.rmax2) c.update = 1;
}

}  // namespace odwf
